// MFMA form of the incremental predictor for the paper's own network (16 and 32 hidden channels; architecture
// table of the appendix "Implement Details").  Same method as predict_inc_reg_body (predict_inc8.h): per
// column, the state of the interior rows moves by (row entering) - (row leaving) and the four border rows are
// evaluated afresh; waves 0,1 = top half, waves 2,3 = bottom half.
//
// Only columns that can contribute are evaluated, as in predict_inc8.h: an instance's columns are cut into passes of up to 252, a
// thread stages one column (all ten rows) and says for either half whether one of the five values is other than zero, and the list a half
// works off holds the outputs with such a value within two columns, the tile's ends, and their direct neighbours, ascending.
// The list goes in chunks of 128 entries, of which the first and the last are neighbours: 126 outputs; its blocks of 32 are dealt to the two
// waves of a half, and blocks beyond the list's end are left out.  With dense rows the list is every column.
// Measured (us; before: every column, tiles of 124), histories of 64 selected blocks in runs: 2048 instances x 2050 columns 128 (295), 256 x 1251 17
// (32), 8 x 2050 8.7 (9.1); all rows dense 327 (301), 31 (32.5), 8.8 (7.9); all zero 64 (293).  With a dense row every 32 steps one half
// is dense in ten of 32.  With rows 0..3 dense and the newest ones sparse, the steps after a prefill, 282 (275). Dense: as many MFMAs as before and
// 8 % more vector instructions (stages, lists and addresses), neither unit full (38 and 44 % of the SIMDs' cycles): a chunk's layers wait for each other at
// barriers; sparse: the passes' serial part.  Two waves per SIMD, 242 VGPRs: 261 of them, and one workgroup a CU,
// cost 70 %; without a straight path through both blocks of a wave, or with the lists made by scalar instructions, 30-100 % more on sparse rows.
//
// v_mfma_f32_32x32x16_f16: D[32 x 32] += A[32 x 16] * B[16 x 32]; lane l supplies row/column l % 32 and K
// entries 8 (l / 32) .. + 7, and receives D rows 8 (v / 4) + 4 (l / 32) + v % 4 (v = 0..15) of column l % 32.
//   layer 1: rows = (y1 row q, c1): two row blocks (q = 0,1 and q = 2,3); K = 16 = (x row 0..4, kw 0..2) + one
//            unused slot; columns = 32 y1 columns.  x is scaled by 2^12 and split into f16 hi + lo (two MFMAs; the
//            split is done once, when a pass's rows are staged),
//            the weights are f16 scaled by 2^-4, the accumulator starts at 2^8 b1: the result is 2^8 y1 before
//            the ReLU.  It is rounded to f16 (the scale keeps y1 up to 255 inside the f16 range), clamped at 0
//            and stored as [half][q][channel half][column] x 8 channels, so a layer-2 operand is one 16-byte read.
//   layer 2: one row block (32 output channels) per output o; K-step = (q, kw) with its 16 input channels.
//            Each output only meets the y1 rows it taps (3 + 3 + 2), 24 MFMAs per column block instead of 36.
//            The staged rows and outputs of the bottom half are numbered so that both halves have the same
//            (q, o) structure; which kernel row a pair stands for is in the operand table built on the host:
//              q0 -> o0     q1 -> o0, o1, o2     q2 -> o0, o2     q3 -> o1, o2        (o0 = the moving row)
//              top:    q0..q3 = x[-1..1] formula, y1[1], y1[2], y1[0]      o1, o2 = rows 0, 1
//              bottom: q0..q3 = y1[H-4], y1[H-2], y1[H-3], y1[H-1]         o1, o2 = rows H-1, H-2
//            Accumulators start at 2^8 b2; the head weights carry the 2^-8.
// The moving row of the bottom half and that of the top half sum their taps in different orders, so the value
// that leaves the state is the one that entered only up to fp32 rounding; callers re-base now and then anyway.
#pragma once

#include "predict_inc8.h"

namespace ap {
namespace {

constexpr int kP16Staged = 256;                   // staged columns of a pass, one a thread: kP16Halo more than outputs on either side
constexpr int kP16Halo = 2, kP16Cols = kP16Staged - 2 * kP16Halo;   // most output columns per pass
constexpr int kP16Outs = 126;                     // outputs of a chunk of 128 list entries
constexpr int kP16YW = 130;                       // y1 entries per plane (layer-2 reads run 2 past the 128 written)
constexpr int kP16BitWords = 20;                  // read by the sixteen lanes of a row, and one further on either side
constexpr int kP16XBuf = 10 * kP16Staged + 4;
constexpr int kP16Y1Floats = 2 * 4 * 2 * kP16YW * 4;
// A1 | 2^8 init1 | 2^-8 w3 | x offsets | 2^8 init2 of (half, row type all / border) | 2^8 lo2 of the same | 2^8 lo1 (f16)
constexpr int kP16ConstFloats = 2 * 2 * kWave * 4 + 2 * 16 + 2 * 16 + 2 * 8 + 2 * 2 * 2 * 16 + 2 * 2 * 2 * 16 + 2 * 4;
// y1 | two passes' x | partial sums [half][staged column] (moving, border) | lists | two passes' bits [half] | constants
constexpr int kPred16LdsFloats = kP16Y1Floats + 2 * kP16XBuf + 4 * kP16Staged + kP16Staged + 4 * kP16BitWords + kP16ConstFloats;
static_assert(kPred16LdsFloats * sizeof(float) <= 65536, "LDS of a workgroup");

// A workgroup of 256 threads takes a run of consecutive passes of all instances (PassPlan); smem: kPred16LdsFloats floats, 16-byte aligned.
__device__ __forceinline__ void predict_inc_mfma16_body(const float* __restrict__ hist,
                                                        const float* __restrict__ wts_global, int R, int H,
                                                        int newest_slot, int nb_cur, int nb_cap, int inst0,
                                                        const PassPlan& plan, int advance, float* __restrict__ pstate,
                                                        float* __restrict__ pred, float* smem) {
  constexpr int C1 = 16, C2 = 32, XW = kP16Staged, YW = kP16YW, XBUF = kP16XBuf;
  constexpr float kXScale = 4096.f, kAccScale = 256.f;
  half8* s_y1 = reinterpret_cast<half8*>(smem);          // [half 2][q 4][channel half 2][YW] x 8 f16
  uint32_t* s_xb = reinterpret_cast<uint32_t*>(smem + kP16Y1Floats);   // 2 buffers of [10][XW] (+4) hi|lo words
  float* s_part = reinterpret_cast<float*>(s_xb + 2 * XBUF);           // [half 2][XW][moving | border]
  uint16_t* s_lists = reinterpret_cast<uint16_t*>(s_part + 4 * XW);    // [half 2][XW] staged column | kRiIsOutput
  uint32_t* s_bits = reinterpret_cast<uint32_t*>(s_lists + 2 * XW);    // [buffer 2][half 2][a zero word | column / 32 | zero words]
  // Per-lane operands that only one phase of a chunk needs live here and are re-read in that phase, which
  // keeps the kernel at two waves per SIMD next to the 96 registers of layer-2 weights:
  half8* s_a1 = reinterpret_cast<half8*>(s_bits + 4 * kP16BitWords);      // [half 2][row block 2][lane 64]
  float* s_b1 = reinterpret_cast<float*>(s_a1 + 2 * 2 * kWave);   // [lane half 2][16] accumulator start of layer 1
  float* s_w3 = s_b1 + 2 * 16;                           // [lane half 2][16] head weight of accumulator entry v
  int* s_xoff = reinterpret_cast<int*>(s_w3 + 2 * 16);   // [lane half 2][8]  x offset of layer-1 K slot e
  // Difference form (ap_internal.h): where the accumulators of the second layer start and where they are clamped,
  // for the outputs that meet all three kernel rows (o0, o2) and for the half's border row (o1: row 0 or row H-1).
  float* s_i2 = reinterpret_cast<float*>(s_xoff + 2 * 8);   // [half 2][all | border][lane half 2][16]
  float* s_l2 = s_i2 + 2 * 2 * 2 * 16;                      // the same layout
  half4* s_l1 = reinterpret_cast<half4*>(s_l2 + 2 * 2 * 2 * 16);   // [channel half pl 2][lane half 2] clamp of the first layer

  const int g_begin = blockIdx.x * plan.per_wg, g_end = min(plan.total, g_begin + plan.per_wg);
  if (g_begin >= g_end) return;                          // (the whole workgroup)
  int at_inst = g_begin, at_pass = 0;
  if (plan.n_pass > 1) {
    at_inst = __umulhi((uint32_t)g_begin, plan.inv_pass);
    at_pass = g_begin - at_inst * plan.n_pass;
    if (at_pass < 0) { --at_inst; at_pass += plan.n_pass; }
  }
  int inst = inst0 + at_inst, c0 = at_pass * plan.cols;

  const int tid = threadIdx.x, lane = tid & (kWave - 1);
  const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  const int hf = wave >> 1, wsub = wave & 1;
  const int n = lane & 31, hsel = lane >> 5;

  // Operand tables and constants.
  const half8* tab = reinterpret_cast<const half8*>(wts_global + kMfma16TableFloatOffset);
  const half8* tab2 = tab + (size_t)hf * 24 * kWave;     // [pair 8][kw 3][lane]
  half8 A2[24];
#pragma unroll
  for (int i = 0; i < 24; ++i) A2[i] = tab2[i * kWave + lane];
  const float* b2 = wts_global + 10 * C1 + 9 * C1 * C2;
  const float* dc = wts_global + delta_const_offset(C1, C2);
  s_a1[tid] = tab[2 * 24 * kWave + tid];
  if (tid < 32) {
    const int h = tid >> 4, v = tid & 15, row = 8 * (v / 4) + 4 * h + v % 4;   // D row of accumulator entry v
    s_b1[tid] = kAccScale * dc[row % C1];
    s_w3[tid] = b2[C2 + row] * (1.f / kAccScale);
  }
  if (tid < 128) {
    const int half = tid >> 6, border = (tid >> 5) & 1, h = (tid >> 4) & 1, v = tid & 15;
    const int row = 8 * (v / 4) + 4 * h + v % 4;
    const int type = border ? (half == 0 ? kRowTop : kRowBot) : kRowAll;
    s_i2[tid] = kAccScale * dc[2 * C1 + type * C2 + row];
    s_l2[tid] = kAccScale * dc[2 * C1 + (4 + type) * C2 + row];
  }
  if (tid < 4) {
    const int pl = tid >> 1, h = tid & 1;
    half4 l;
#pragma unroll
    for (int c = 0; c < 4; ++c) l[c] = (_Float16)(kAccScale * dc[C1 + 8 * pl + 4 * h + c]);
    s_l1[tid] = l;
  }
  if (tid < 16) {   // layer-1 K slot 8 h + e is (x row, kw) = divmod(8 h + e, 3); slot 15 has zero weights
    const int k = tid;
    s_xoff[tid] = k < 15 ? (k / 3) * XW + k % 3 : 0;
  }
  if (tid < 4) s_xb[XBUF - 4 + tid] = s_xb[2 * XBUF - 4 + tid] = 0u;

  // Staging: thread tid fetches staged column tid (tile column c0 - kP16Halo + tid) of all ten rows, a pass ahead into registers; staged rows
  // 0..4 are history rows -1..3, staged rows 5..9 are rows H-5..H-1.
  uint32_t row_off[10];                                  // (wave-uniform, byte offsets into an instance's ring)
#pragma unroll
  for (int r = 0; r < 10; ++r)
    row_off[r] = (uint32_t)__builtin_amdgcn_readfirstlane(ring_slot(newest_slot, H, R, r < 5 ? r - 1 : H - 10 + r)) * (uint32_t)nb_cap * 4u;
  float xpre[10], pst_cur = 0.f, pst_next = 0.f;
  // Loads are unconditional on clamped addresses; the raw values stay untouched in registers until `stash`
  // masks them, so nothing waits on them while the current pass is computed.
  auto fetch = [&](int in, int at, float& pst) __attribute__((always_inline)) {
    const char* src = reinterpret_cast<const char*>(hist + (size_t)in * R * nb_cap);
    const uint32_t j = (uint32_t)min(max(at - kP16Halo + tid, 0), nb_cur - 1);
#pragma unroll
    for (int i = 0; i < 10; ++i) xpre[i] = *reinterpret_cast<const float*>(src + (row_off[i] + j * 4u));
    pst = (pstate + (size_t)in * nb_cap)[j];
  };
  // The words of a pass, and a bit per column and half: is one of its five values other than zero.
  auto stash = [&](int at, int buf) __attribute__((always_inline)) {
    const int j = at - kP16Halo + tid;
    const bool inside = j >= 0 && j < nb_cur;
    uint32_t* s_x = s_xb + buf * XBUF + tid;
#pragma unroll
    for (int h2 = 0; h2 < 2; ++h2) {
      uint32_t any = 0u;
#pragma unroll
      for (int r = 0; r < 5; ++r) {
        const uint32_t w = split_hi_lo(inside ? xpre[h2 * 5 + r] * kXScale : 0.f);
        any |= w;
        s_x[(h2 * 5 + r) * XW] = w;
      }
      const unsigned long long m = __ballot((any & 0x7fff7fffu) != 0u);
      if (lane < 2) s_bits[(buf * 2 + h2) * kP16BitWords + 1 + 2 * wave + lane] = (uint32_t)(m >> (32 * lane));
    }
  };
  float inf = INFINITY;                 // opaque, so that med3(a, 0, inf) stays one instruction
  asm volatile("" : "+v"(inf));
  for (int i = tid; i < 4 * kP16BitWords; i += 256) s_bits[i] = 0u;     // (the words around a row stay zero)
  fetch(inst, c0, pst_cur);
  __syncthreads();
  stash(c0, 0);
  __syncthreads();

  int buf = 0;
#pragma unroll 1
  for (int left = g_end - g_begin; left > 0; --left, buf ^= 1) {
    const int len = min(nb_cur - c0, plan.cols);         // output columns, from staged column kP16Halo on
    const uint32_t* s_x = s_xb + buf * XBUF;
    const bool more = left > 1;
    int inst_next = inst, c0_next = c0 + plan.cols;
    if (c0_next >= nb_cur) { ++inst_next; c0_next = 0; }
    if (more) fetch(inst_next, c0_next, pst_next);

    // The halves' lists, as in predict_inc8.h: lane w of a row of 16 works on columns 32 w .. 32 w + 31, the even rows on the top half,
    // the odd ones on the bottom half; then wave w writes the entries of columns 64 w .. 64 w + 63 of both.
    int count[2];
    bool output[2];                                      // is this thread's column an output of the half
    {
      const int w = lane & 15;
      const uint32_t* bits = s_bits + (buf * 2 + ((lane >> 4) & 1)) * kP16BitWords + 1 + w;
      const uint32_t a0 = bits[0], whole = bit_range(kP16Halo, kP16Halo + len, w);
      count[0] = count[1] = len + 2;
      output[0] = output[1] = true;                      // (in the columns of the pass)
      if ((uint32_t)__ballot((a0 & whole) == whole) != ~0u) {          // has not every column of the pass a value in either half?
        const uint32_t am = bits[-1], ap = bits[1];
        // column i takes the bits of columns i - 2 .. i + 2
        uint32_t out = a0 | __builtin_amdgcn_alignbit(a0, am, 31) | __builtin_amdgcn_alignbit(a0, am, 30) |
                       __builtin_amdgcn_alignbit(ap, a0, 1) | __builtin_amdgcn_alignbit(ap, a0, 2);
        out &= whole;
        if (c0 == 0) out |= bit_range(kP16Halo, kP16Halo + 1, w);      // (beside the tile y1 = 0 stands for d1 = lo1)
        if (c0 + len == nb_cur) out |= bit_range(kP16Halo + len - 1, kP16Halo + len, w);
        const uint32_t prev = dpp_all<0x111>(out), next = dpp_all<0x101>(out);      // row_shr:1: word w - 1; row_shl:1: word w + 1
        const uint32_t listed = out | __builtin_amdgcn_alignbit(out, prev, 31) | __builtin_amdgcn_alignbit(next, out, 1);
        const uint32_t own = (uint32_t)__builtin_popcount(listed);
        uint32_t incl = own;                               // inclusive sums over each row of 16 lanes
        incl += dpp_all<0x111>(incl);
        incl += dpp_all<0x112>(incl);
        incl += dpp_all<0x114>(incl);
        incl += dpp_all<0x118>(incl);
#pragma unroll
        for (int h2 = 0; h2 < 2; ++h2) {
          const int at = h2 * 16 + 2 * wave;
          count[h2] = __builtin_amdgcn_readlane(incl, h2 * 16 + 15);
          const uint32_t lo = __builtin_amdgcn_readlane(listed, at), hi = __builtin_amdgcn_readlane(listed, at + 1);
          const uint32_t olo = __builtin_amdgcn_readlane(out, at), ohi = __builtin_amdgcn_readlane(out, at + 1);
          output[h2] = __builtin_amdgcn_inverse_ballot_w64(((unsigned long long)ohi << 32) | olo);
          const uint32_t rank = __builtin_amdgcn_mbcnt_hi(hi, __builtin_amdgcn_mbcnt_lo(lo, __builtin_amdgcn_readlane(incl - own, at)));
          if (__builtin_amdgcn_inverse_ballot_w64(((unsigned long long)hi << 32) | lo))
            s_lists[h2 * XW + rank] = (uint16_t)(tid | (output[h2] ? kRiIsOutput : 0u));
        }
      }
    }
    if (count[0] != len + 2 || count[1] != len + 2) __syncthreads();   // (dense lists are not looked at; the same for every wave)
    const uint16_t* s_list = s_lists + hf * XW;
    const int cnt = hf ? count[1] : count[0], longest = max(count[0], count[1]);
    const bool dense = cnt == len + 2;                   // every column: entry e is column kP16Halo - 1 + e, an output but for
                                                         // the ends (and what is read beyond them is staged, too)
    auto entry_at = [&](int e) __attribute__((always_inline)) { return (uint32_t)s_list[min(e, cnt - 1)]; };

#pragma unroll 1
    for (int e_chunk = 0; e_chunk + 2 < longest; e_chunk += kP16Outs) {       // (the same for every wave)
    int fresh = 0;                      // opaque zero: the phase operands are read again in every chunk
    asm volatile("" : "+v"(fresh));

    // Layer 1.
    {
      const uint32_t* xs = s_x + hf * 5 * XW;
      const half8 A1a = s_a1[fresh + (hf * 2 + 0) * kWave + lane], A1b = s_a1[fresh + (hf * 2 + 1) * kWave + lane];
      float16v b1acc;
      int xoff[8];
#pragma unroll
      for (int v = 0; v < 16; ++v) b1acc[v] = s_b1[fresh + hsel * 16 + v];
#pragma unroll
      for (int e = 0; e < 8; ++e) xoff[e] = s_xoff[fresh + hsel * 8 + e];
      const half4 lo1a = s_l1[fresh + 0 * 2 + hsel], lo1b = s_l1[fresh + 1 * 2 + hsel];
      auto block = [&](int blk, int col) __attribute__((always_inline)) {
        const int yc = (blk * 2 + wsub) * 32 + n;        // entry 0..127 of the chunk
        uint4v whi, wlo;
#pragma unroll
        for (int e = 0; e < 8; e += 2) {
          const uint32_t wa = xs[col - 1 + xoff[e]], wb = xs[col - 1 + xoff[e + 1]];
          whi[e / 2] = __builtin_amdgcn_perm(wb, wa, 0x05040100u);
          wlo[e / 2] = __builtin_amdgcn_perm(wb, wa, 0x07060302u);
        }
        const half8 Bhi = __builtin_bit_cast(half8, whi), Blo = __builtin_bit_cast(half8, wlo);
        const int j = c0 - kP16Halo + col;
        const bool outside = j < 0 || j >= nb_cur;
#pragma unroll
        for (int rb = 0; rb < 2; ++rb) {
          float16v acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(rb ? A1b : A1a, Bhi, b1acc, 0, 0, 0);
          acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(rb ? A1b : A1a, Blo, acc, 0, 0, 0);
          // entry v: y1 row q = 2 rb + v / 8, channel 8 (v / 4 % 2) + 4 hsel + v % 4
#pragma unroll
          for (int ql = 0; ql < 2; ++ql)
#pragma unroll
            for (int p = 0; p < 2; ++p) {
              half4 h;
#pragma unroll
              for (int c = 0; c < 4; ++c) h[c] = (_Float16)acc[8 * ql + 4 * p + c];
              h = __builtin_elementwise_max(h, p ? lo1b : lo1a);
              reinterpret_cast<half4*>(s_y1 + ((hf * 4 + 2 * rb + ql) * 2 + p) * YW + yc)[hsel] = h;
            }
        }
        if (outside) {                                   // layer-2 padding: y1 = 0 beside the tile, d1 = lo1
#pragma unroll
          for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int p = 0; p < 2; ++p)
              reinterpret_cast<half4*>(s_y1 + ((hf * 4 + q) * 2 + p) * YW + yc)[hsel] = p ? lo1b : lo1a;
        }
      };
      // (both blocks without a branch between them, where the list is long enough: their chains hide each other's latency)
      const int e = e_chunk + wsub * 32 + n;
      if (e_chunk + (2 + wsub) * 32 < cnt) {
        if (dense) {
          block(0, kP16Halo - 1 + e);
          block(1, kP16Halo - 1 + e + 64);
        } else {
          const int col0 = entry_at(e) & ~kRiIsOutput, col1 = entry_at(e + 64) & ~kRiIsOutput;
          block(0, col0);
          block(1, col1);
        }
      } else if (e_chunk + wsub * 32 < cnt) {
        block(0, dense ? kP16Halo - 1 + e : entry_at(e) & ~kRiIsOutput);
      }
    }
    __syncthreads();

    // Layer 2 and the head.
    float16v b2acc, b2bor;                // accumulator starts: rows with all kernel rows (o0, o2), the border row (o1)
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      b2acc[v] = s_i2[fresh + ((hf * 2 + 0) * 2 + hsel) * 16 + v];
      b2bor[v] = s_i2[fresh + ((hf * 2 + 1) * 2 + hsel) * 16 + v];
    }
    auto block = [&](int blk) __attribute__((always_inline)) {
      const int cb = (blk * 2 + wsub) * 32;              // outputs cb .. cb + 31: entries cb + 1 ..
      const half8* yq = s_y1 + ((size_t)hf * 4 * 2 + hsel) * YW + cb + n;   // + q * 2 * YW + kw
      float16v acc0, acc1, acc2;
#pragma unroll
      for (int kw = 0; kw < 3; ++kw) {
        const half8 B = yq[0 * 2 * YW + kw];
        acc0 = __builtin_amdgcn_mfma_f32_32x32x16_f16(A2[0 * 3 + kw], B, kw == 0 ? b2acc : acc0, 0, 0, 0);
      }
#pragma unroll
      for (int kw = 0; kw < 3; ++kw) {
        const half8 B = yq[1 * 2 * YW + kw];
        acc0 = __builtin_amdgcn_mfma_f32_32x32x16_f16(A2[1 * 3 + kw], B, acc0, 0, 0, 0);
        acc1 = __builtin_amdgcn_mfma_f32_32x32x16_f16(A2[2 * 3 + kw], B, kw == 0 ? b2bor : acc1, 0, 0, 0);
        acc2 = __builtin_amdgcn_mfma_f32_32x32x16_f16(A2[3 * 3 + kw], B, kw == 0 ? b2acc : acc2, 0, 0, 0);
      }
#pragma unroll
      for (int kw = 0; kw < 3; ++kw) {
        const half8 B = yq[2 * 2 * YW + kw];
        acc0 = __builtin_amdgcn_mfma_f32_32x32x16_f16(A2[4 * 3 + kw], B, acc0, 0, 0, 0);
        acc2 = __builtin_amdgcn_mfma_f32_32x32x16_f16(A2[5 * 3 + kw], B, acc2, 0, 0, 0);
      }
#pragma unroll
      for (int kw = 0; kw < 3; ++kw) {
        const half8 B = yq[3 * 2 * YW + kw];
        acc1 = __builtin_amdgcn_mfma_f32_32x32x16_f16(A2[6 * 3 + kw], B, acc1, 0, 0, 0);
        acc2 = __builtin_amdgcn_mfma_f32_32x32x16_f16(A2[7 * 3 + kw], B, acc2, 0, 0, 0);
      }
      float t0 = 0.f, t1 = 0.f, t2 = 0.f;
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const float w = s_w3[fresh + hsel * 16 + v];
        const float la = s_l2[fresh + ((hf * 2 + 0) * 2 + hsel) * 16 + v], lb = s_l2[fresh + ((hf * 2 + 1) * 2 + hsel) * 16 + v];
        t0 = fmaf(w, __builtin_amdgcn_fmed3f(acc0[v], la, inf), t0);
        t1 = fmaf(w, __builtin_amdgcn_fmed3f(acc1[v], lb, inf), t1);
        t2 = fmaf(w, __builtin_amdgcn_fmed3f(acc2[v], la, inf), t2);
      }
      // Sum the two channel halves: afterwards lanes 0..31 hold the moving row, lanes 32..63 the two border rows.
      const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(t0), __float_as_uint(t1 + t2), false, false);
      const int e = e_chunk + cb + n + 1;
      const uint32_t entry = dense ? (uint32_t)(kP16Halo - 1 + e) | kRiIsOutput : entry_at(e);
      if (cb + n < kP16Outs && e < cnt - 1 && (entry & kRiIsOutput))
        s_part[(hf * XW + (entry & ~kRiIsOutput)) * 2 + hsel] = __uint_as_float(sw[0]) + __uint_as_float(sw[1]);
    };
    if (e_chunk + (2 + wsub) * 32 + 2 < cnt) { block(0); block(1); }
    else if (e_chunk + wsub * 32 + 2 < cnt) block(0);
    if (e_chunk + kP16Outs + 2 < longest) __syncthreads();               // (the next chunk overwrites what was read)
    }
    // The next pass's words go to the other buffer; this barrier is also the one before its lists and y1 overwrite this pass's.
    if (more) stash(c0_next, buf ^ 1);
    __syncthreads();
    if (tid >= kP16Halo && tid < kP16Halo + len) {
      const float2* part = reinterpret_cast<const float2*>(s_part);
      float2 top = make_float2(0.f, 0.f), bot = make_float2(0.f, 0.f);       // (a column that is no output has no partial sums)
      if (output[0]) top = part[tid];
      if (output[1]) bot = part[XW + tid];
      const size_t o = (size_t)inst * nb_cap + (c0 - kP16Halo + tid);
      float st = pst_cur;
      if (advance && (output[0] || output[1])) {
        st = (st - top.x) + bot.x;
        pstate[o] = st;
      }
      pred[o] = (st + (top.y + bot.y)) / (float)H;
    }
    pst_cur = pst_next;
    inst = inst_next;
    c0 = c0_next;
  }
}

}  // namespace
}  // namespace ap
