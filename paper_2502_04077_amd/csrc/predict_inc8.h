// Incremental predictor for 8/8 channels on MFMA with both layers held in registers (see predict.hip for the
// method: the interior state moves by (row entering) - (row leaving), the four border rows are evaluated afresh).
//
// Only columns that can contribute are evaluated.  In the difference form of ap_internal.h a history that is zero
// around a column gives exactly zero there (d1 = max(min(b1, 0), -max(b1, 0)) = 0, and the same for d2), and the rows
// that sparse steps push are zero outside the selection.  So a pass of up to kRiPassCols columns starts with one bit per
// column and half of the method: is one of the half's five values other than zero.  An output column has such a
// value within two columns, or lies at an end of the tile (where y1 = 0 beside the tile stands for d1 = lo1); the
// list a wave then works off holds the outputs and their direct neighbours, in ascending order, so that lanes next to
// each other hold neighbouring columns wherever an output needs them: of 2050 columns with 64 selected in runs, some
// 200 a half.  With dense rows it would hold every column and is not written at all.
//
// A wave owns 32 list entries at a time (lane l: entry n = l % 32, channel half h = l / 32) and works one half of the
// method on them: waves 0,1 the top half (leaving row, rows 0, 1), waves 2,3 the bottom half (entering row, rows H-2,
// H-1; the outputs of a half are numbered so that 1 is the row whose window leaves the history: row 0, row H-1).
// v_mfma_f32_32x32x16_f16 computes D[32 x 32] += A[32 x 16] * B[16 x 32]; lane l supplies row / column l % 32 and
// K entries 8 (l / 32) .. + 7 and receives D rows 8 (v / 4) + 4 (l / 32) + v % 4 (v = 0..15) of column l % 32.  What
// makes the registers enough:
//   layer 1  rows = (staged y1 row q, channel c1), K = 16 = 15 (x row, tap) pairs + a constant 1 that carries the
//            accumulator start.  The ten history rows of a pass of columns go from global memory straight to LDS
//            (global_load_lds, no registers), asked for a whole pass ahead into the other of two buffers; at the start
//            of a pass a column's values are scaled by 2^12 and rounded to f16 once, in place, into the words that the
//            K slots are made of.
//   layer 2  the result of layer 1 is, per lane, channels 4h .. 4h+3 of the four y1 rows of its own column: exactly
//            half of the K entries of a layer-2 step whose 16 entries are two (y1 row, tap) pairs of 8 channels.
//            The centre tap takes those registers as they are, the outer taps the same registers moved by one
//            lane with DPP wave shifts (16 moves): K = 96 in six steps, no LDS and no barrier.
//   head     fp32: clamp (the ReLU in difference form), weight, sum the four channels of the lane, and one
//            half-wave swap adds the two channel halves.
// The entries at either end of the 32 get wrong neighbours, so a piece yields 30 outputs and pieces overlap by two.
// All arithmetic is in the difference form of ap_internal.h: accumulators start at 2^8 init, the ReLUs are clamps at
// 2^8 lo, y1 is kept as f16 of 2^8 d1.  f16 operands, fp32 accumulation.
// The two halves of a column meet once per pass, through LDS: the state and pred are written by a short epilogue after
// the pass's second barrier (the first one is between the bits and the lists).  The
// leaving row is evaluated by the same instruction sequence on the same values as when it entered, so it cancels exactly.
//
// Measured at 2048 instances x 2050 columns (0.20 GB to move: 31 us at the rate a plain read reaches), histories of 64
// selected blocks in runs: 45.5 us, with all columns evaluated 67-69; an all-zero history 37 us (66), 128 instances x 8194
// columns 14.2 us (22.9).  Where both halves have a value in every column of a pass (the first five steps after a prefill) nothing is
// looked up and the pieces inside the tile take a loop of their own, without a test or an address of their own: 76 us (up to 90 in the
// launches right after a prefill), against 73
// for a kernel that only knows dense histories and reads the f16 words of row 2 in pairs (82-84 us with the lists made in any
// case); there the SIMDs are full of vector instructions (62 a piece at four cycles) and MFMAs, which overlap in part
// only.  A single pass per workgroup, 1 to 8 instances, takes 0.2 us longer than in that kernel: bits, barrier, list.
#pragma once

#include <type_traits>

#include "predict_body.h"

namespace ap {
namespace {

constexpr int kRiOut = 30;                              // outputs per 32 list entries
constexpr int kRiRawSegs = 6;                           // a raw history row of a pass arrives in wave-wide pieces
constexpr int kRiRawStride = kRiRawSegs * kWave;        // staged history columns of a pass, four more than outputs on either side
constexpr int kRiPassCols = kRiRawStride - 8;           // most output columns per pass (four workgroups' LDS fits a CU)
// LDS words: two buffers of ten raw history rows [row][kRiRawStride], the pass at hand and the next one; the partial
// sums [half][column of the pass][moving | border]; the waves' column lists (16 bits an entry); one bit per staged
// column [half][2 zero words | column / 32 | zero words]; two masks of output columns; and a constant
constexpr int kRiRawWords = 10 * kRiRawStride;
constexpr int kRiPartWords = 2 * kRiPassCols * 2;
constexpr int kRiListWords = kRiRawStride / 2;
constexpr int kRiBitWords = 20;
constexpr int kPredRegLdsFloats = 2 * kRiRawWords + kRiPartWords + 4 * kRiListWords + 2 * kRiBitWords + 16 + 2 * 16 + 2 * kRiOut + 1;
static_assert(2 * kRiRawSegs <= 16 && 2 + 16 + 1 <= kRiBitWords, "a lane of a row of 16 per 32 columns");
constexpr uint32_t kRiIsOutput = 0x8000u;               // list entry: staged column | this if it is an output

// Every lane is written (a lane without a source lane gets 0), so no previous value has to be set up.
template <int CTRL> __device__ __forceinline__ uint32_t dpp_all(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, CTRL, 0xF, 0xF, true);
}
constexpr int kWaveShr1 = 0x138, kWaveShl1 = 0x130;     // lane l reads lane l - 1 / l + 1 of the whole wave

// 64 consecutive floats of LDS starting at `dst` (wave-uniform) are filled from global memory, lane l from
// base[byte_off / 4] of its own choosing, without passing through registers; completion is counted by vmcnt.
__device__ __forceinline__ void load_to_lds(const float* base, uint32_t byte_off, float* dst) {
  typedef const __attribute__((address_space(1))) void* gptr_t;
  typedef __attribute__((address_space(3))) void* lptr_t;
  __builtin_amdgcn_global_load_lds((gptr_t)(reinterpret_cast<const char*>(base) + byte_off), (lptr_t)dst, 4, 0, 0);
}

// Bits [lo, hi) of a row of bits, as far as they lie in its 32-bit word w.
__device__ __forceinline__ uint32_t bits_from(int n) { return n <= 0 ? ~0u : n >= 32 ? 0u : ~0u << n; }
__device__ __forceinline__ uint32_t bit_range(int lo, int hi, int w) { return bits_from(lo - 32 * w) & ~bits_from(hi - 32 * w); }

// Workgroup barrier for data in LDS only: __syncthreads() would also wait for the loads in flight (vmcnt), among
// them the next pass's rows.
__device__ __forceinline__ void lds_barrier() {
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

// Every instance's columns are cut into n_pass passes of equal length (at most kRiPassCols columns); a workgroup of
// 256 threads takes a run of consecutive passes of all instances, so that the operands are fetched and the first
// rows waited for once per workgroup.  (Divisions would be a tenth of a call that has one pass a workgroup: the host makes them.)
struct PassPlan {
  int n_pass, cols;                                      // passes per instance, columns of a pass
  int total, per_wg;                                     // passes of all instances, of a workgroup
  uint32_t inv_pass;                                     // ceil(2^32 / n_pass) where n_pass > 1: quotients at most one too large
};

// smem: kPredRegLdsFloats floats.
__device__ __forceinline__ void predict_inc_reg_body(const float* __restrict__ hist, const float* __restrict__ wts_global,
                                                     int R, int H, int newest_slot, int nb_cur, int nb_cap, int inst0,
                                                     const PassPlan& plan, int advance, float* __restrict__ pstate,
                                                     float* __restrict__ pred, float* smem) {
  constexpr int C = 8;
  constexpr float kXScale = 4096.f, kAccScale = 256.f;
  typedef _Float16 half2v __attribute__((ext_vector_type(2)));

  const int pass_cols = plan.cols;
  const int tid_all = threadIdx.x;
  int tid = tid_all, lane = tid & (kWave - 1);
  const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  const int hf = wave >> 1, wsub = wave & 1;
  const int n = lane & 31, hsel = lane >> 5;

  // Ring rows of the ten staged x rows, as byte offsets into an instance's ring: staged rows 0..4 of the top half are history
  // rows -1..3, of the bottom half H-5..H-1.  (Wave-uniform: they live in scalar registers.)  Without an advance no row leaves, and row -1 is
  // not looked at, whatever it may hold: row 0 stands in for it.
  uint32_t row_off[2][5];
#pragma unroll
  for (int h2 = 0; h2 < 2; ++h2)
#pragma unroll
    for (int r = 0; r < 5; ++r)
      row_off[h2][r] = (uint32_t)__builtin_amdgcn_readfirstlane(ring_slot(newest_slot, H, R, h2 ? H - 5 + r : max(r - 1, advance ? -1 : 0))) * (uint32_t)nb_cap * 4u;
  // The raw rows of a pass are asked for a whole pass ahead and go straight to LDS: of the six pieces of 64 columns
  // wave w brings piece w of all ten rows and piece 4 + w / 2 of one half's rows (every address is clamped into the
  // tile; what lies outside only reaches lanes that mask it).  Staged column i is history column c0 - 4 + i.
  auto fetch_pass = [&](int inst, int c0, float* s_raw) __attribute__((always_inline)) {
    const int n_staged = min(nb_cur - c0, pass_cols) + 8;
    const float* hist_inst = hist + (size_t)inst * R * nb_cap;
    if (wave * kWave < n_staged) {                         // (wave-uniform)
      const uint32_t off = (uint32_t)min(max(c0 - 4 + wave * kWave + lane, 0), nb_cur - 1) * 4u;
#pragma unroll
      for (int h2 = 0; h2 < 2; ++h2)
#pragma unroll
        for (int r = 0; r < 5; ++r)
          load_to_lds(hist_inst, off + row_off[h2][r], s_raw + (h2 * 5 + r) * kRiRawStride + wave * kWave);
    }
    const int k = 4 + hf;
    if (k * kWave < n_staged) {
      const uint32_t off = (uint32_t)min(max(c0 - 4 + k * kWave + lane, 0), nb_cur - 1) * 4u;
#pragma unroll
      for (int r = 0; r < 5; ++r)
        load_to_lds(hist_inst, off + (wsub ? row_off[1][r] : row_off[0][r]), s_raw + (wsub * 5 + r) * kRiRawStride + k * kWave);
    }
  };
  const int g_begin = blockIdx.x * plan.per_wg, g_end = min(plan.total, g_begin + plan.per_wg);
  if (g_begin >= g_end) return;                          // (the whole workgroup: no barrier is skipped by part of it)
  int at_inst = g_begin, at_pass = 0;
  if (plan.n_pass > 1) {
    at_inst = __umulhi((uint32_t)g_begin, plan.inv_pass);
    at_pass = g_begin - at_inst * plan.n_pass;
    if (at_pass < 0) { --at_inst; at_pass += plan.n_pass; }
  }
  int inst = inst0 + at_inst, c0 = at_pass * pass_cols;
  fetch_pass(inst, c0, smem);

  // Operand tables and per-lane constants.
  const half8* tab2 = reinterpret_cast<const half8*>(wts_global + kMfmaTableFloatOffset) + (size_t)hf * 6 * kWave;
  const half8* tab1 = reinterpret_cast<const half8*>(wts_global + kMfmaTableFloatOffset) + 2 * 6 * kWave + hf * kWave;
  half8 A2[6];
#pragma unroll
  for (int s = 0; s < 6; ++s) A2[s] = tab2[s * kWave + lane];
  const half8 A1 = tab1[lane];
  // (constants come four channels at a time: every group of four starts on 16 bytes)
  static_assert(delta_const_offset(C, C) % 4 == 0 && (10 * C + 9 * C * C + C) % 4 == 0, "16-byte constants");
  const float4* dc = reinterpret_cast<const float4*>(wts_global + delta_const_offset(C, C)) + hsel;
  auto scaled = [](float4 v, float* dst) __attribute__((always_inline)) {
    dst[0] = kAccScale * v.x; dst[1] = kAccScale * v.y; dst[2] = kAccScale * v.z; dst[3] = kAccScale * v.w;
  };
  float16v b2init;                                       // entry v is D row 8 (v / 4) + c, c = 4 hsel + v % 4
  half4 lo1h;
  float lo2v[8], w3v[4];                                 // (outputs 0 and 2 share their clamps)
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    const int ty = k != 1 ? kRowAll : hf ? kRowBot : kRowTop;
    float start[4];
    scaled(dc[(2 * C + ty * C) / 4], start);
    if (k < 2) scaled(dc[(2 * C + (4 + ty) * C) / 4], lo2v + 4 * k);
#pragma unroll
    for (int j = 0; j < 4; ++j) b2init[4 * k + j] = start[j];
  }
#pragma unroll
  for (int j = 12; j < 16; ++j) b2init[j] = 0.f;
  {
    float lo1[4];
    scaled(dc[C / 4], lo1);
    const float4 w3 = reinterpret_cast<const float4*>(wts_global + 10 * C + 9 * C * C + C)[hsel];
    w3v[0] = w3.x; w3v[1] = w3.y; w3v[2] = w3.z; w3v[3] = w3.w;
#pragma unroll
    for (int j = 0; j < 4; ++j) lo1h[j] = (_Float16)lo1[j];
  }
  float inf = INFINITY;                                  // opaque, so that med3(a, lo, inf) stays one instruction
  asm volatile("" : "+v"(inf));
  const float inv_H = 1.f / (float)H;                    // the time mean as a multiplication
  constexpr float kUnscale = 1.f / kAccScale;            // the head sums come out times 2^8 (exact to undo)

  float2* s_part = reinterpret_cast<float2*>(smem + 2 * kRiRawWords);   // [half][column]: (moving, border)
  uint16_t* s_list = reinterpret_cast<uint16_t*>(smem + 2 * kRiRawWords + kRiPartWords) + wave * kRiRawStride;
  uint32_t* s_bits = reinterpret_cast<uint32_t*>(smem + 2 * kRiRawWords + kRiPartWords + 4 * kRiListWords);
  uint32_t* s_outs = s_bits + 2 * kRiBitWords;           // the outputs of a whole pass, one bit per staged column
  uint32_t* s_epi = s_outs + 16;                         // [half][column / 32]: the outputs of the pass at hand
  // f16 1 in the place of a row-2 word, for the lane half whose K slot is the constant (read with an offset of two pieces too)
  uint32_t* s_one = s_epi + 32;
  if (tid <= 2 * kRiOut) s_one[tid] = 0x3c00u;
  if (tid < 2 * kRiBitWords) s_bits[tid] = 0u;           // (the words around a row stay zero)
  if (tid < 16) s_outs[tid] = bit_range(4, 4 + pass_cols, tid);
  __builtin_amdgcn_s_waitcnt(0x0F70);                    // vmcnt(0): this wave's pieces of the first pass are in LDS
  __syncthreads();


  int buf = 0;
#pragma unroll 1
  for (int left = g_end - g_begin; left > 0; --left, buf ^= 1) {
    // (worked out again in every pass: what follows from them would otherwise sit in registers through all of it)
    tid = tid_all;
    asm volatile("" : "+v"(tid));
    lane = tid & (kWave - 1);
    const int w = lane & 15, w_half = (lane >> 4) & 1;   // the word of bits this lane works on, and its half
    const int len = min(nb_cur - c0, pass_cols);         // output columns of the pass: staged columns 4 .. 4 + len - 1
    // Staged columns lie beyond the tile: the pass holds an end of it, or the last pass is shorter than what is staged beside
    // this one.
    const bool at_end = c0 == 0 || c0 + len + 4 > nb_cur;
    float* pstate_pass = pstate + ((size_t)inst * nb_cap + c0);
    float* pred_pass = pred + ((size_t)inst * nb_cap + c0);
    // Every wave has seen its own pieces of this pass's rows arrive before the last barrier, and is done with the
    // pass before: the other buffer is free.  The next pass's rows and the state of this thread's columns are asked
    // for now and have the whole pass to arrive in.
    float* s_raw = smem + buf * kRiRawWords;
    int inst_next = inst, c0_next = c0 + pass_cols;
    if (c0_next >= nb_cur) { ++inst_next; c0_next = 0; }
    if (left > 1) fetch_pass(inst_next, c0_next, smem + (buf ^ 1) * kRiRawWords);
    constexpr int kPerThread = (kRiPassCols + 255) / 256;
    float pst[kPerThread];
#pragma unroll
    for (int i = 0; i < kPerThread; ++i) pst[i] = pstate_pass[(uint32_t)min(tid + 256 * i, len - 1)];

    // One bit per staged column and half: is one of the five values other than zero.  Where one of 64 columns has such
    // a value they are turned into what layer 1 reads, in place (a thread touches its own column only): f16 of 2^12 x,
    // zero outside the tile, rows (0 | 1) in the place of row 0, (3 | 4) in that of row 1, (2 | 0) in that of row 2.
    // Zeros are that already.  (Six pieces of 64 columns, two halves: three of these for every wave.)
#pragma unroll
    for (int u = 0; u < kRiRawSegs / 2; ++u) {
      const int seg = u * 2 + hf, h2 = wsub;             // (wave-uniform)
      const int i = seg * kWave + lane;
      float* x = s_raw + h2 * 5 * kRiRawStride + i;
      const float x0 = x[0], x1 = x[kRiRawStride], x2 = x[2 * kRiRawStride], x3 = x[3 * kRiRawStride], x4 = x[4 * kRiRawStride];
      const uint32_t any = (__float_as_uint(x0) | __float_as_uint(x1) | __float_as_uint(x2) | __float_as_uint(x3) |
                            __float_as_uint(x4)) << 1;
      const unsigned long long nonzero = __ballot(any != 0u);
      unsigned long long m = nonzero;
      float sc = kXScale;
      if (at_end) {
        const bool inside = (uint32_t)(c0 - 4 + i) < (uint32_t)nb_cur;
        m &= __ballot(inside);
        sc = inside ? kXScale : 0.f;
      }
      if (nonzero != 0ull) {                             // (with a column outside the tile, too)
        const half2v a01 = {(_Float16)(x0 * sc), (_Float16)(x1 * sc)}, a34 = {(_Float16)(x3 * sc), (_Float16)(x4 * sc)};
        const half2v a2 = {(_Float16)(x2 * sc), (_Float16)0};
        x[0] = __builtin_bit_cast(float, a01);
        x[kRiRawStride] = __builtin_bit_cast(float, a34);
        x[2 * kRiRawStride] = __builtin_bit_cast(float, a2);
      }
      if (lane < 2) s_bits[h2 * kRiBitWords + 2 + seg * 2 + lane] = (uint32_t)(m >> (32 * lane));
    }
    lds_barrier();
    // Which columns are outputs, which are listed, and how many come before: lane w of a row of 16 lanes works on
    // columns 32 w .. 32 w + 31, the even rows on the top half, the odd ones on the bottom half.
    // First of all: has every column of the pass a value in either half?  Then there is nothing to look up.
    int count = len + 2;
    bool dense = true;                                   // every column of the pass: entry e is column 3 + e, an output but for the ends
    const uint32_t* bits = s_bits + w_half * kRiBitWords + 2 + w;
    const uint32_t a0 = bits[0], whole = at_end ? bit_range(4, 4 + len, w) : s_outs[w];
    const bool all_dense = (uint32_t)__ballot((a0 & whole) == whole) == ~0u;     // (lanes 0 .. 31: the words of both halves)
    if (!all_dense) {
      const uint32_t am = bits[-1], ap = bits[1];
      // column i takes the bits of columns i - 2 .. i + 2
      uint32_t out = a0 | __builtin_amdgcn_alignbit(a0, am, 31) | __builtin_amdgcn_alignbit(a0, am, 30) |
                     __builtin_amdgcn_alignbit(ap, a0, 1) | __builtin_amdgcn_alignbit(ap, a0, 2);
      out &= whole;
      if (at_end) {
        if (c0 == 0) out |= bit_range(4, 5, w);
        if (c0 + len == nb_cur) out |= bit_range(4 + len - 1, 4 + len, w);
      }
      const uint32_t prev = __builtin_amdgcn_update_dpp(0, out, 0x111, 0xF, 0xF, true);   // row_shr:1: word w - 1
      const uint32_t next = __builtin_amdgcn_update_dpp(0, out, 0x101, 0xF, 0xF, true);   // row_shl:1: word w + 1
      if (wave == 0 && lane < 32) s_epi[lane] = out;       // (read after the pass's last barrier)
      const uint32_t listed = out | __builtin_amdgcn_alignbit(out, prev, 31) | __builtin_amdgcn_alignbit(next, out, 1);
      const int own = __builtin_popcount(listed);
      int incl = own;                                    // inclusive sums over each row of 16 lanes
      incl += __builtin_amdgcn_update_dpp(0, incl, 0x111, 0xF, 0xF, true);
      incl += __builtin_amdgcn_update_dpp(0, incl, 0x112, 0xF, 0xF, true);
      incl += __builtin_amdgcn_update_dpp(0, incl, 0x114, 0xF, 0xF, true);
      incl += __builtin_amdgcn_update_dpp(0, incl, 0x118, 0xF, 0xF, true);
      const int row0 = hf * 16;                          // first lane of this wave's half
      count = __builtin_amdgcn_readlane(incl, row0 + 15);
      dense = count == len + 2;
      if (!dense && count != 0) {
#pragma unroll
        for (int s = 0; s < kRiRawSegs; ++s) {
          const uint32_t lo = __builtin_amdgcn_readlane(listed, row0 + 2 * s), hi = __builtin_amdgcn_readlane(listed, row0 + 2 * s + 1);
          if ((lo | hi) == 0u) continue;
          const uint32_t olo = __builtin_amdgcn_readlane(out, row0 + 2 * s), ohi = __builtin_amdgcn_readlane(out, row0 + 2 * s + 1);
          const int base = __builtin_amdgcn_readlane(incl - own, row0 + 2 * s);
          const uint32_t rank = __builtin_amdgcn_mbcnt_hi(hi, __builtin_amdgcn_mbcnt_lo(lo, base));
          const uint32_t col = s * kWave + lane;
          if (__builtin_amdgcn_inverse_ballot_w64(((unsigned long long)hi << 32) | lo))
            s_list[rank] = (uint16_t)(__builtin_amdgcn_inverse_ballot_w64(((unsigned long long)ohi << 32) | olo) ? col | kRiIsOutput : col);
        }
      }
    }
    asm volatile("" ::: "memory");                       // a wave reads what it has just written, in order

    // 32 list entries: this lane's staged column `at` (3 .. 4 + len, or, beyond the end of a dense list, anything finite
    // to read that no output depends on), whose words the pointers stand for (moved by `off`).  One of them may lie beside
    // the tile, where y1 = 0 (d1 = lo1).  INNER: none does, and entries 1 .. 30 are all outputs.
    struct Words { const uint32_t *rows, *side, *mid; float* part; };
    auto words_of = [&](int at) __attribute__((always_inline)) {
      const uint32_t* x = reinterpret_cast<const uint32_t*>(s_raw) + hf * 5 * kRiRawStride + at;
      // rows (0 | 1) or (3 | 4); row 2, column - 1 or + 1; row 2 or the constant
      return Words{x + hsel * kRiRawStride, x + 2 * kRiRawStride + 2 * hsel - 1, hsel ? s_one : x + 2 * kRiRawStride,
                   reinterpret_cast<float*>(s_part) + (hf * kRiPassCols + at - 4) * 2 + hsel};
    };
    auto piece = [&](const Words& ptr, int off, int col, bool output, auto inner_tag) __attribute__((always_inline)) {
      constexpr bool BORDER = !decltype(inner_tag)::value;
      // Layer 1 operand: the K slots of this lane half (ri_slot_row / ri_slot_kw).
      uint4v b1;
#pragma unroll
      for (int kw = 0; kw < 3; ++kw) b1[kw] = ptr.rows[off + kw - 1];
      b1[3] = __builtin_amdgcn_perm(ptr.mid[off], ptr.side[off], 0x05040100u);         // (side | column), or (side | 1)
      float16v acc = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
      acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(A1, __builtin_bit_cast(half8, b1), acc, 0, 0, 0);
      // y1 row q, channels 4 hsel .. + 3 of this lane's column: f16 of 2^8 d1
      const bool inside = !BORDER || (col >= 0 && col < nb_cur);
      half4 y[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        half4 h;
#pragma unroll
        for (int c = 0; c < 4; ++c) h[c] = (_Float16)acc[4 * q + c];
        y[q] = __builtin_elementwise_max(h, lo1h);
        if (BORDER) y[q] = inside ? y[q] : lo1h;         // layer-2 padding: y1 = 0 beside the tile
      }

      // Layer 2: centre taps from the registers as they are, outer taps moved by a lane.
      typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
      uint4v bc[2], bm[2], bp[2];                        // steps (q0, q1) and (q2, q3) of tap 1, 0, 2
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const u32x2 w = __builtin_bit_cast(u32x2, y[q]);
#pragma unroll
        for (int r = 0; r < 2; ++r) {
          bc[q >> 1][2 * (q & 1) + r] = w[r];
          bm[q >> 1][2 * (q & 1) + r] = dpp_all<kWaveShr1>(w[r]);
          bp[q >> 1][2 * (q & 1) + r] = dpp_all<kWaveShl1>(w[r]);
        }
      }
      acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(A2[0], __builtin_bit_cast(half8, bc[0]), b2init, 0, 0, 0);
      acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(A2[1], __builtin_bit_cast(half8, bc[1]), acc, 0, 0, 0);
      acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(A2[2], __builtin_bit_cast(half8, bm[0]), acc, 0, 0, 0);
      acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(A2[3], __builtin_bit_cast(half8, bm[1]), acc, 0, 0, 0);
      acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(A2[4], __builtin_bit_cast(half8, bp[0]), acc, 0, 0, 0);
      acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(A2[5], __builtin_bit_cast(half8, bp[1]), acc, 0, 0, 0);
      float p[3];                                        // 2^8 x the head-weighted sums of this lane's four channels
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        float t = 0.f;
#pragma unroll
        for (int jj = 0; jj < 4; ++jj) t = fmaf(w3v[jj], __builtin_amdgcn_fmed3f(acc[4 * k + jj], lo2v[4 * (k & 1) + jj], inf), t);
        p[k] = t;
      }
      // Sum the two channel halves: afterwards lanes 0..31 hold the moving row, lanes 32..63 the two border rows.
      const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(p[0]), __float_as_uint(p[1] + p[2]), false, false);
      const float total = __uint_as_float(sw[0]) + __uint_as_float(sw[1]);
      if (n >= 1 && n <= kRiOut && output)
        ptr.part[2 * off] = total;
    };
    // (The first and the last entry of a list that is not empty are neighbours, not outputs.)
    int e0 = wsub * kRiOut, e_next = e0 + 2 * kRiOut;
    if (dense) {                                           // (the same for the whole wave)
      const bool head = c0 == 0 && wsub == 0;              // its first piece holds the column beside the tile
      int e = head ? e_next : e0;
      const int last = min(count, nb_cur - c0 + 1) - 32;   // first entry of the last piece inside the tile and the list
      Words ptr = words_of(3 + e + n);
#pragma unroll 1
      for (; e + 2 * kRiOut <= last; e += 4 * kRiOut) {
        piece(ptr, 0, 0, true, std::true_type{});
        piece(ptr, 2 * kRiOut, 0, true, std::true_type{});
        ptr.rows += 4 * kRiOut;
        ptr.side += 4 * kRiOut;
        ptr.mid += hsel ? 0 : 4 * kRiOut;
        ptr.part += 8 * kRiOut;
      }
      if (e <= last) {
        piece(ptr, 0, 0, true, std::true_type{});
        e += 2 * kRiOut;
      }
      if (head) e_next = e;
      else { e0 = e; e_next = e + 2 * kRiOut; }
    }
#pragma unroll 1
    for (; e0 + 2 < count; e0 = e_next, e_next += 2 * kRiOut) {
      const int e = e0 + n;
      const uint32_t entry = dense ? (uint32_t)min(3 + e, 4 + len) | (e > 0 ? kRiIsOutput : 0u) : s_list[min(e, count - 1)];
      const int at = entry & ~kRiIsOutput;
      piece(words_of(at), 0, c0 - 4 + at, e < count - 1 && (entry & kRiIsOutput), std::false_type{});
    }
    __builtin_amdgcn_s_waitcnt(0x0F70);                  // vmcnt(0): this wave's pieces of the next pass are in LDS
    __syncthreads();
#pragma unroll
    for (int i = 0; i < kPerThread; ++i) {
      const uint32_t rel = tid + 256 * i;
      if (rel < (uint32_t)len) {
        float2 top = s_part[rel], bot = s_part[kRiPassCols + rel];
        bool has_top = true, has_bot = true;
        if (!all_dense) {                                // a column that is no output has no partial sums
          const uint32_t word = (rel + 4) >> 5, bit = (rel + 4) & 31;
          has_top = (s_epi[word] >> bit) & 1u;
          has_bot = (s_epi[16 + word] >> bit) & 1u;
          if (!has_top) top = make_float2(0.f, 0.f);
          if (!has_bot) bot = make_float2(0.f, 0.f);
        }
        float st = pst[i];
        if (advance && (has_top || has_bot)) {
          st = (st - top.x * kUnscale) + bot.x * kUnscale;
          pstate_pass[rel] = st;
        }
        pred_pass[rel] = (st + (top.y + bot.y) * kUnscale) * inv_H;
      }
    }
    inst = inst_next;
    c0 = c0_next;
  }
}

}  // namespace
}  // namespace ap
