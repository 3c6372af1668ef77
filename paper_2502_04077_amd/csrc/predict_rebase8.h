// The interior state of the incremental predictor from scratch, 8/8 channels on MFMA: what a re-base or a first prediction needs,
//   state[j] = sum_{r=2}^{H-3} sum_c w3[c] * (relu(y2[c][r][j]) - relu(B2[c]))      (difference form, ap_internal.h).
// The border rows 0, 1, H-2, H-1 and pred are then added by the incremental kernel run without an advance.  Same operands as there (x as one
// f16 of 2^12 x, fp32 accumulation, y1 kept as f16 of 2^8 d1), so a re-based state continues the advanced one without a step.
//
// The time axis is walked in strips of three output rows, with v_mfma_f32_32x32x16_f16: D[32 x 32] += A[32 x 16] * B[16 x 32]; lane l
// supplies row / column l % 32 and K entries 8 (l / 32) .. + 7 and receives D rows 8 (v / 4) + 4 (l / 32) + v % 4 of column l % 32.
//   pass p    layer 1 for y1 rows 1+3p .. 3+3p from x rows 3p .. 3p+4: rows = (y1 row, channel), 8 of 32 idle; K = 15 (x row, tap) pairs.
//             A column's x rows lie in LDS as f16 in threes: a word with rows 3p, 3p+1 and a half word with row 3p+2
//   strip s   layer 2 for output rows 2+3s .. 4+3s from the y1 rows of passes s and s+1, of which the wave keeps six in LDS:
//             rows = (output row, channel), K = 15 (y1 row, tap) chunks of 8 channels in 8 steps, each operand one 16-byte read
//   head      fp32: clamp, weight, the four channels of a lane, into a running sum; the two channel halves meet at the end
// Order is part of the result: an MFMA adds its K entries in two groups of eight, the second onto what the first gave (the order inside a
// group does not matter), so a y2 value is nine groups of 8 channels in the order of the taps, and a column's sum goes row by row.  A column is
// evaluated by one item, from its first strip to its last, whatever its neighbours in the tile need: equal windows
// have equal states, bit for bit, wherever they lie, and blocks whose scores coincide are told apart by their order alone.  (Sums taken in another order - two
// rows at a time, dense and sparse strips apart - are no further from the exact ones, but decide near ties another way now and then.)
//
// Only what can contribute is evaluated: where the five columns around an output are zero in the seven rows around a strip, its
// terms are exactly zero.  Every column has a bit per three x rows, so a word per column says which strips matter.  A row that a sparse step pushed
// is zero outside the selection, a row of a prefill or a calibration nowhere: strips that matter in more than half of a tile's columns
// are dense.  The columns in which another strip matters are listed with their neighbours, as in predict_inc8.h, and an item
// of 32 entries, 30 outputs, walks the dense strips and those that matter in one of its columns; items of consecutive columns walk the
// dense strips for the others (or all that matter in one of theirs, where most columns would be listed).
// A tile's rows are read once, straight into f16 words.
//
// Measured at 2048 instances x 2050 columns, H = 64, state and pred, 33 to 77 us of it the border rows and pred (before: every strip of every
// column, rows staged by every wave for itself): histories of 64 selected blocks in runs with a dense row every 32 steps 539 us (866),
// without dense rows 444 (955), all rows dense 884 (1012), all zero 305 (950); 8 instances 18 us (18).  Reading the 1.09 GB of rows and
// listing take 213 us without arithmetic (155 at a plain read's rate).  Dense strips are bound by issue (63 % of the SIMDs' cycles vector
// instructions, 54 % MFMAs), selected columns by a strip's chain in the one wave that has the list: nine MFMAs of which eight build on each other, y1
// into LDS and back, the head.
// Measured and not kept: operands asked for a strip ahead but their addresses kept in a register each (spills: 588 us instead of 539), 66
// rows on their way at a time (no difference), the same sums by 16x16x32 MFMAs, two output rows at a time and half the
// MFMA cycles (533, all dense 911).  Strips of two rows summed in an order of their own, dense and listed ones apart, take 369 us.
#pragma once

#include "predict_body.h"

namespace ap {
namespace {

constexpr int kRbOut = 30;                              // outputs per item
constexpr int kRbCols = 8 * kRbOut;                     // most output columns per tile (two items a wave)
constexpr int kRbStrips = 21;                           // most strips per segment of the time axis
constexpr int kRbHalo = 4;                              // staged columns on either side of a tile's outputs
constexpr int kRbYW = 34;                               // y1 columns of a row (32 written, reads run 2 further)

// Tiles of cols columns (staged: 64, 128 or 256, at least cols + 8), the time axis in segments of at most kRbStrips strips.
struct RebasePlan { int cols, seg_strips; };

// LDS words: y1 [wave][6 rows][kRbYW] x 8 f16 | x rows in threes: two in a word, the third in a half word |
// sums [channel half][column], before that masks of x rows per thread | strips per column | active columns per wave and strip, then
// the list (bytes) | listed columns per wave | next item
constexpr int kRbY1Words = 4 * 6 * kRbYW * 4;
constexpr int rebase_lds_words(int staged, int seg_strips) {
  return kRbY1Words + (seg_strips + 2) * staged * 3 / 2 + 512 + staged + 4 * 32 + 8 + 4;
}
static_assert(rebase_lds_words(256, kRbStrips) * 4 * 3 <= 160 * 1024, "three workgroups a CU");

// Workgroup of 256 threads, SW staged columns; smem: rebase_lds_words(..) words, 16-byte aligned.
template <int SW>
__device__ __forceinline__ void predict_rebase8_body(const float* __restrict__ hist, const float* __restrict__ wts_global, int R,
                                                     int H, int newest_slot, int nb_cur, int nb_cap, int inst, int tile,
                                                     const RebasePlan& plan, float* __restrict__ pstate, uint32_t* smem) {
  constexpr int C = 8;
  constexpr float kXScale = 4096.f, kAccScale = 256.f;
  typedef _Float16 half2v __attribute__((ext_vector_type(2)));
  const int tid = threadIdx.x, lane = tid & (kWave - 1);
  const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  const int n = lane & 31, h = lane >> 5;
  constexpr int kParts = 256 / SW;                       // threads per staged column
  constexpr int kBatch = SW == 64 ? 6 : 11;              // threes of x rows of a column on their way at a time
  const int c0 = tile * plan.cols, len = min(nb_cur - c0, plan.cols);
  const float* hist_inst = hist + (size_t)inst * R * nb_cap;

  half8* s_y1 = reinterpret_cast<half8*>(smem) + wave * 6 * kRbYW;             // [6][kRbYW]
  const int n_threes = plan.seg_strips + 2;
  uint32_t* s_x01 = smem + kRbY1Words;                                         // [n_threes][SW]
  _Float16* s_x2 = reinterpret_cast<_Float16*>(s_x01 + n_threes * SW);         // [n_threes][SW]
  uint32_t* s_rest = s_x01 + n_threes * SW * 3 / 2;
  float* s_sum = reinterpret_cast<float*>(s_rest);                             // [2][SW]
  unsigned long long* s_mask = reinterpret_cast<unsigned long long*>(s_rest);  // [256]
  uint32_t* s_act = s_rest + 512;                                              // [SW]
  uint32_t* s_cnt = s_act + SW;                                                // [wave 4][32]
  uint8_t* s_list = reinterpret_cast<uint8_t*>(s_cnt);                         // [SW]
  unsigned long long* s_out = reinterpret_cast<unsigned long long*>(s_cnt + 4 * 32);   // [wave 4]
  int* s_next = reinterpret_cast<int*>(s_out + 4);       // next item

  const int n_rows = H - 4, n_strips = (n_rows + 2) / 3; // interior rows 2 .. H-3
  const int col = tid & (SW - 1), part = __builtin_amdgcn_readfirstlane(tid / SW);   // staged column, and which of its x rows
  const int j_col = c0 - kRbHalo + col;                  // its column of the tile
  const bool is_out = part == 0 && col >= kRbHalo && col < kRbHalo + len;
  float total[2] = {0.f, 0.f};                           // of this thread's column, by channel halves

#pragma unroll 1
  for (int t0 = 0; t0 < n_strips; t0 += plan.seg_strips) {
    const int n_seg = min(plan.seg_strips, n_strips - t0);
    const uint32_t seg_mask = (1u << n_seg) - 1u;
    // x rows 3 t0 .. 3 (t0 + n_seg) + 5: f16 of 2^12 x, zero outside the window and the tile, and two bits for every three: is one of
    // them other than zero, and is the first.  A thread takes a run of its column's rows, up to 33 on their way at a time.
    {
      const int per = (n_seg + 2 + kParts - 1) / kParts, i_begin = part * per, i_end = min(n_seg + 2, i_begin + per);
      const bool inside = j_col >= 0 && j_col < nb_cur;
      // (rows as scalar byte offsets into the instance's ring, walked from slot to slot)
      const uint32_t j_load = (uint32_t)min(max(j_col, 0), nb_cur - 1) * 4u, row_bytes = (uint32_t)nb_cap * 4u;
      int row = 3 * (t0 + i_begin), slot = ring_slot(newest_slot, H, R, min(row, H - 1));
      unsigned long long mask = 0;
#pragma unroll 1
      for (int i0 = i_begin; i0 < i_end; i0 += kBatch) {
        float x[kBatch][3];
#pragma unroll
        for (int u = 0; u < kBatch; ++u) {
#pragma unroll
          for (int r = 0; r < 3; ++r) {                  // (past the last row the last one again)
            x[u][r] = *reinterpret_cast<const float*>(reinterpret_cast<const char*>(hist_inst) + (j_load + (uint32_t)slot * row_bytes));
            if (++row < H && ++slot == R) slot = 0;
          }
        }
#pragma unroll
        for (int u = 0; u < kBatch; ++u)               // (all on their way before the first is used)
          asm volatile("" : "+v"(x[u][0]), "+v"(x[u][1]), "+v"(x[u][2]));
        uint32_t some = 0u, first = 0u;
#pragma unroll
        for (int u = 0; u < kBatch; ++u) {
          if (i0 + u >= i_end) break;
          const int i = i0 + u, left = H - 3 * (t0 + i);      // rows of the three that exist
          const half2v x01 = {(_Float16)(x[u][0] * kXScale), (_Float16)(x[u][1] * kXScale)};
          const _Float16 x2 = (_Float16)(x[u][2] * kXScale);
          const uint32_t keep = left >= 2 ? ~0u : left == 1 ? 0xffffu : 0u;
          const uint32_t w = inside ? __builtin_bit_cast(uint32_t, x01) & keep : 0u;
          const uint16_t w2 = inside && left >= 3 ? __builtin_bit_cast(uint16_t, x2) : (uint16_t)0;
          s_x01[i * SW + col] = w;
          s_x2[i * SW + col] = __builtin_bit_cast(_Float16, w2);
          some |= ((w & 0x7fff7fffu) | (w2 & 0x7fffu)) != 0u ? 1u << u : 0u;
          first |= (w & 0x7fffu) != 0u ? 1u << u : 0u;
        }
        mask |= (unsigned long long)(some << i0) | ((unsigned long long)(first << i0) << 32);
      }
      s_mask[tid] = mask;
    }
    __syncthreads();
    // Operand tables and per-lane constants (asked for here, where the staged rows have left the registers).
    const float* wts = wts_global;
    asm volatile("" : "+s"(wts));
    const half8* tab = reinterpret_cast<const half8*>(wts + kMfmaTableFloatOffset) + kMfmaTableHalfs / 8;
    half8 A2[8];
#pragma unroll
    for (int st = 0; st < 8; ++st) A2[st] = tab[st * kWave + lane];
    const half8 A1 = tab[8 * kWave + lane];
    const float* dc = wts + delta_const_offset(C, C);
    float16v b1acc, b2acc;                                 // entry v is D row 8 (v / 4) + c, c = 4 h + v % 4
    float w3v[4], lo2v[4];
    half4 lo1h;
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      b1acc[v] = v < 12 ? kAccScale * dc[4 * h + v % 4] : 0.f;
      b2acc[v] = v < 12 ? kAccScale * dc[2 * C + kRowAll * C + 4 * h + v % 4] : 0.f;
    }
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      w3v[c] = wts[10 * C + 9 * C * C + C + 4 * h + c] * (1.f / kAccScale);
      lo2v[c] = kAccScale * dc[2 * C + (4 + kRowAll) * C + 4 * h + c];
      lo1h[c] = (_Float16)(kAccScale * dc[C + 4 * h + c]);
    }
    float inf = INFINITY;                                  // opaque, so that med3(a, lo, inf) stays one instruction
    asm volatile("" : "+v"(inf));
    // The strips that matter to an output column: those that a value within two columns reaches (strip s: x rows 3s .. 3s+6).
    uint32_t act = 0u;
    if (is_out) {
      unsigned long long m = 0;
      for (int p = 0; p < kParts; ++p)
#pragma unroll
        for (int d = -2; d <= 2; ++d) m |= s_mask[p * SW + col + d];
      const uint32_t some = (uint32_t)m, first = (uint32_t)(m >> 32);
      act = (some | (some >> 1) | (first >> 2)) & seg_mask;
      if (j_col == 0 || j_col == nb_cur - 1) act = seg_mask;       // (beside the tile y1 = 0 stands for d1 = lo1)
    }
    uint32_t active = 0u;                                // lane t: columns of this wave to which strip t matters
#pragma unroll
    for (int t = 0; t < kRbStrips; ++t) {
      const uint32_t c = (uint32_t)__popcll(__ballot((int)(act << (31 - t)) < 0));
      asm("v_writelane_b32 %0, %1, %2" : "+v"(active) : "s"(c), "n"(t));
    }
    if (lane < 32) s_cnt[wave * 32 + lane] = active;
    __syncthreads();
    uint32_t in_all = 0u;
    if (lane < 32) in_all = (s_cnt[lane] + s_cnt[32 + lane]) + (s_cnt[2 * 32 + lane] + s_cnt[3 * 32 + lane]);
    const uint32_t dense = (uint32_t)__ballot(2 * (int)in_all > len) & seg_mask;
    if (part == 0) {
      s_sum[col] = total[0];                             // (the masks have been read)
      s_sum[SW + col] = total[1];
      s_act[col] = act & ~dense;
    }
    {
      const unsigned long long o = __ballot((act & ~dense) != 0u);
      if (lane == 0) s_out[wave] = o;
      if (tid == 0) *s_next = 0;
    }
    __syncthreads();
    int n_list = 0;
    if (dense != seg_mask) {                             // (the same for every wave)
      unsigned long long before = 0, mine = 0;           // the wave's 64 columns, and the outputs of the wave before
#pragma unroll
      for (int w = 0; w < 4; ++w) {
        const unsigned long long o = s_out[w], prev = w > 0 ? s_out[w - 1] : 0ull, next = w < 3 ? s_out[w + 1] : 0ull;
        const unsigned long long listed = o | (o << 1) | (o >> 1) | (prev >> 63) | (next << 63);
        const int c = __popcll(listed);
        if (w < wave) before += c;
        if (w == wave) mine = listed;
        n_list += c;
      }
      n_list = __builtin_amdgcn_readfirstlane(n_list);
      if ((mine >> lane) & 1ull)
        s_list[(int)before + __builtin_amdgcn_mbcnt_hi((uint32_t)(mine >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mine, 0u))] = (uint8_t)tid;
    }
    __syncthreads();

    // Most columns listed: items of consecutive columns take their strips along.
    const bool together = 4 * n_list > 3 * len;
    const int n_row = dense != 0u || together ? (len + kRbOut - 1) / kRbOut : 0;       // items of consecutive columns
    const int n_listed = !together && n_list > 2 ? (n_list - 2 + kRbOut - 1) / kRbOut : 0;
    // (the listed ones first: they are the longer ones; a wave takes the next one when it is done with one)
#pragma unroll 1
    for (;;) {
      int item = 0;
      if (lane == 0) item = atomicAdd(s_next, 1);
      item = __builtin_amdgcn_readfirstlane(item);
      if (item >= n_listed + n_row) break;
      const bool listed = item < n_listed;
      const int e0 = (listed ? item : item - n_listed) * kRbOut;
      // Entry n is this lane's column of the first layer, entry n + 1 that of its output (lanes 0 .. 29).
      int at, at_out;
      bool output = n < kRbOut;
      uint32_t S = 0u;
      if (listed) {
        at = s_list[min(e0 + n, n_list - 1)];
        at_out = s_list[min(e0 + n + 1, n_list - 1)];
        const uint32_t a = s_act[at_out];
        output = output && e0 + n + 1 < n_list - 1 && a != 0u;
        S = output ? a : 0u;
      } else {
        at = min(kRbHalo - 1 + e0 + n, SW - 2);
        at_out = min(kRbHalo + e0 + n, SW - 2);
        const uint32_t a = s_act[at_out];
        output = output && e0 + n < len && (together || a == 0u);
        S = output && together ? a : 0u;
        if (!__any(output)) continue;
      }
#pragma unroll
      for (int i = 16; i > 0; i >>= 1) S |= __shfl_xor(S, i, kWave);
      S = __builtin_amdgcn_readfirstlane(S) | dense;     // (both halves of the wave hold the same columns)
      const int j_y1 = c0 - kRbHalo + at;
      const bool outside = j_y1 < 0 || j_y1 >= nb_cur, border = __any(outside);
      float sum = s_sum[h * SW + at_out];

      // Layer-1 operand of pass p: K entries of half h = (rows 3h, 3h+1) x three taps, and row 2's outer taps by halves
      // (the last one of half 1 has no weight and is the tap beside it once more).
      const uint32_t* x01 = s_x01 + h * SW + at - 1;
      const uint16_t* x2a = reinterpret_cast<const uint16_t*>(s_x2) + at - 1 + 2 * h;
      const uint16_t* x2b = reinterpret_cast<const uint16_t*>(s_x2) + at + h;
      auto x_of = [&](int p) __attribute__((always_inline)) {
        uint4v w;
#pragma unroll
        for (int kw = 0; kw < 3; ++kw) w[kw] = x01[p * SW + kw];
        w[3] = (uint32_t)x2a[p * SW] | ((uint32_t)x2b[p * SW] << 16);
        return w;
      };
      auto first_layer = [&](uint4v w) __attribute__((always_inline)) {
        return __builtin_amdgcn_mfma_f32_32x32x16_f16(A1, __builtin_bit_cast(half8, w), b1acc, 0, 0, 0);
      };
      auto put = [&](const float16v& acc, auto parity_tag) __attribute__((always_inline)) {
        half4 y[3];
#pragma unroll
        for (int q = 0; q < 3; ++q) {
#pragma unroll
          for (int c = 0; c < 4; ++c) y[q][c] = (_Float16)acc[4 * q + c];
          y[q] = __builtin_elementwise_max(y[q], lo1h);
        }
        if (border) {                                    // layer-2 padding: y1 = 0 beside the tile, d1 = lo1
#pragma unroll
          for (int q = 0; q < 3; ++q) y[q] = outside ? lo1h : y[q];
        }
#pragma unroll
        for (int q = 0; q < 3; ++q) reinterpret_cast<half4*>(s_y1 + (3 * decltype(parity_tag)::value + q) * kRbYW + n)[h] = y[q];
      };
      // Operand of step st of a strip whose first pass is of parity P: y1 row q < 3 is of that pass, the others of the next one
      // (chunk 15 has no weight).  The second half of the wave reads the next chunk: a tap or a row further, or from the ring's start.
      const half8 *y_tap = s_y1 + n + h, *y_row = s_y1 + n + h * (kRbYW - 2), *y_turn = s_y1 + n - h * (5 * kRbYW + 2), *y_same = s_y1 + n;
      auto operand = [&](int st, auto parity_tag) __attribute__((always_inline)) {
        constexpr int P = decltype(parity_tag)::value;
        const int q = 2 * st / 3, kw = 2 * st % 3, slot = q < 3 ? 3 * P + q : 3 * (1 - P) + q - 3;
        const half8* y = st == 7 ? y_same : kw < 2 ? y_tap : slot == 5 ? y_turn : y_row;
        return y[slot * kRbYW + kw];
      };
      // Strip t, whose two passes are in LDS and the first four operands (B) on their way; w: the x words of the pass after those, which is
      // made meanwhile (at a run's end for nothing).  One wave reads what it has just written: the LDS keeps a wave's accesses in
      // order, the compiler has to as well.
      uint4v w;
      half8 B[8];
      auto strip = [&](int t, auto parity_tag, auto other_tag) __attribute__((always_inline)) {
#pragma unroll
        for (int st = 4; st < 6; ++st) B[st] = operand(st, parity_tag);
        const float16v d = first_layer(w);
        w = x_of(min(t + 3, n_seg));
        float16v acc;
#pragma unroll
        for (int st = 0; st < 4; ++st) acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(A2[st], B[st], st == 0 ? b2acc : acc, 0, 0, 0);
        asm volatile("" ::: "memory");
        put(d, parity_tag);
        asm volatile("" ::: "memory");
#pragma unroll
        for (int st = 6; st < 8; ++st) B[st] = operand(st, parity_tag);
#pragma unroll
        for (int st = 4; st < 8; ++st) acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(A2[st], B[st], acc, 0, 0, 0);
#pragma unroll
        for (int st = 0; st < 4; ++st) B[st] = operand(st, other_tag);
        const int left = n_rows - 3 * (t0 + t);          // output rows of this strip that exist
        float v[3];
#pragma unroll
        for (int o = 0; o < 3; ++o) {
          v[o] = 0.f;
#pragma unroll
          for (int c = 0; c < 4; ++c) v[o] = fmaf(w3v[c], __builtin_amdgcn_fmed3f(acc[4 * o + c], lo2v[c], inf), v[o]);
        }
        if (left < 3) {
          v[2] = 0.f;                                    // (adds nothing)
          if (left < 2) v[1] = 0.f;
        }
        sum = ((sum + v[0]) + v[1]) + v[2];
      };
      constexpr std::integral_constant<int, 0> kEven{};
      constexpr std::integral_constant<int, 1> kOdd{};
#pragma unroll 1
      while (S != 0u) {                                  // a run of consecutive strips
        int t = __builtin_ctz(S);
        {
          const float16v d0 = first_layer(x_of(t)), d1 = first_layer(x_of(t + 1));
          w = x_of(min(t + 2, n_seg));
          if (t & 1) {
            put(d0, kOdd);
            put(d1, kEven);
            asm volatile("" ::: "memory");
#pragma unroll
            for (int st = 0; st < 4; ++st) B[st] = operand(st, kOdd);
          } else {
            put(d0, kEven);
            put(d1, kOdd);
            asm volatile("" ::: "memory");
#pragma unroll
            for (int st = 0; st < 4; ++st) B[st] = operand(st, kEven);
          }
        }
        auto more = [&]() __attribute__((always_inline)) {
          S &= S - 1u;
          ++t;
          return S != 0u && (int)__builtin_ctz(S) == t;
        };
#pragma unroll 1
        for (;;) {
          if (!(t & 1)) {
            strip(t, kEven, kOdd);
            if (!more()) break;
          }
          strip(t, kOdd, kEven);
          if (!more()) break;
        }
      }
      if (output) s_sum[h * SW + at_out] = sum;
    }
    __syncthreads();
    if (part == 0) {
      total[0] = s_sum[col];
      total[1] = s_sum[SW + col];
    }
    if (t0 + n_seg < n_strips) __syncthreads();          // (the next segment's masks lie where the sums are)
  }
  if (is_out) pstate[(size_t)inst * nb_cap + j_col] = total[0] + total[1];
}

}  // namespace
}  // namespace ap
