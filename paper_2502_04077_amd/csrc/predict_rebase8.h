// The predictor over the full history tile for 8/8 channels on MFMA: what a re-base or a first prediction needs.  Writes the
// interior state of the incremental form,
//   state[j] = sum_{r=2}^{H-3} sum_c w3[c] * (relu(y2[c][r][j]) - relu(B2[c]))      (difference form, ap_internal.h),
// and pred, which adds the border rows 0, 1, H-2, H-1.  Same arithmetic as the incremental kernel (x as one f16 of 2^12 x,
// fp32 accumulation, y1 kept as f16 of 2^8 d1), so a re-based state continues the advanced one without a step.
//
// The time axis is walked in strips of two output rows: strip t is rows 2t, 2t+1, which meet y1 rows 2t-1 .. 2t+2, i.e. the
// y1 pairs t and t+1 (pair t: rows 2t-1, 2t), and pair t meets the x pairs t-1 and t (x pair p: rows 2p, 2p+1; one word of LDS a
// column, zeros outside the window).  v_mfma_f32_16x16x16_f16 and _16x16x32_f16: D[16 x 16] += A[16 x K] * B[K x 16], lane l
// supplies row / column l % 16 and K entries K/4 (l / 16) .. and receives D rows 4 (l / 16) + v of column l % 16.
//   layer 1  rows = (y1 row of the pair, channel), K = 16 = 4 lane groups x 2 words: x pair t-1 (groups 0, 1) or t (2, 3) of
//            columns j-1, j (groups 0, 2) or j, j+1 (1, 3; the first with weight 0)
//   layer 2  rows = (output row, channel), K = 32 = two y1 pairs x 2 rows x 8 channels for one column tap: the result of
//            layer 1 is, per lane, four channels of one y1 row of its own column, which is what its lane group supplies.  The
//            centre tap takes those registers as they are, the outer taps the same moved by one lane with DPP moves; a
//            pair is used twice, as the later and as the earlier one.  Three MFMAs a strip.
//   head     fp32: clamp, weight, into a running sum per lane; lane groups are added up once per item.
// An item is 32 columns (two blocks of 16, the inner lanes at the seam exchanged), whose first and last have wrong neighbours: 30
// outputs.  (Blocks of 32 columns with three output rows of 32 D rows, as before, fill 42 % of their MFMAs, these 75 %.)
//
// Only what can contribute is evaluated: where the five columns around an output are zero in the six rows around a strip, its
// terms are exactly zero.  Every column has a bit per x pair, so a word per column says which strips matter.  A row that a sparse step pushed
// is zero outside the selection, a row of a prefill or a calibration nowhere: strips that matter in more than half of a tile's columns
// are evaluated in all of them, and for the other strips the columns in which one matters are listed with
// their neighbours, as in predict_inc8.h, and an item walks those strips that matter in one of its columns.
// A tile's rows are read once, straight into f16 words; four workgroups a CU, so that some read while others compute.
//
// Measured at 2048 instances x 2050 columns, H = 64, state and pred (before: three output rows to 32 D rows, every strip of every
// column, the border rows and pred by a second launch over ten rows): histories of 64 selected blocks in runs with a dense row every 32 steps 381 us
// (913), without dense rows 302 (972), all rows dense 695 (991), all zero 233 (965); 8 instances 10 us (15.8).  The 1.09 GB of rows are 155 us
// at a plain read's rate, and 205 us with the masks and lists and no arithmetic; dense strips are bound by issue: 160 cycles of vector instructions
// (twelve DPP moves, sixteen of the head, eight of the first layer's results) and 128 of MFMAs a strip and item, 240 together.
// Measured and not kept: strips with border rows inside the runs (381 -> 415: branches in every strip), all 64 rows of a column on their
// way at once (255 -> 360 on zeros: registers), an instance's tiles on one XCD (no difference).
#pragma once

#include "predict_body.h"

namespace ap {
namespace {

constexpr int kRbOut = 30;                              // outputs per item
constexpr int kRbCols = 8 * kRbOut;                     // most output columns per tile (two items a wave)
constexpr int kRbStrips = 32;                           // most strips per segment of the time axis (one bit each)
constexpr int kRbBatch = 16;                            // x pairs of a column on their way at a time
constexpr int kRbHalo = 4;                              // staged columns on either side of a tile's outputs

// Tiles of cols columns (staged: 64, 128 or 256, at least cols + 8), the time axis in segments.
struct RebasePlan { int cols, seg_strips; };

// LDS words: x pairs | sums [dense, listed][column] (interior, border), before that a mask of x pairs per thread |
// strips per column | list (bytes), before that active columns per wave and strip |
// outputs per wave | where the second layer starts and is clamped, per row type
constexpr int rebase_sum_words(int staged) { return 4 * staged > 512 ? 4 * staged : 512; }
constexpr int rebase_lds_words(int staged, int seg_strips) {
  return (seg_strips + 2) * staged + rebase_sum_words(staged) + staged + 4 * kRbStrips + 8 + 8 * 8;
}

typedef float rb_float4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ float add_lane_groups(float v) {      // sum over the four rows of 16 lanes, in every lane
  const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  v = __uint_as_float(a[0]) + __uint_as_float(a[1]);
  const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return __uint_as_float(b[0]) + __uint_as_float(b[1]);
}

// Moved by a lane within rows of 16: lane n gets lane n - 1 / n + 1; at the row's end what `other` has at its far end (a block's
// neighbour), or, without one, anything.
template <int CTRL> __device__ __forceinline__ uint32_t dpp_row(uint32_t old, uint32_t v) {
  return (uint32_t)__builtin_amdgcn_update_dpp((int)old, (int)v, CTRL, 0xF, 0xF, false);
}
constexpr int kRowShl1 = 0x101, kRowShr1 = 0x111, kRowRor1 = 0x121, kRowRor15 = 0x12F;

// Workgroup of 256 threads, SW staged columns; smem: rebase_lds_words(..) words.
template <int SW>
__device__ __forceinline__ void predict_rebase8_body(const float* __restrict__ hist, const float* __restrict__ wts_global, int R,
                                                     int H, int newest_slot, int nb_cur, int nb_cap, int inst, int tile,
                                                     const RebasePlan& plan, float* __restrict__ pstate,
                                                     float* __restrict__ pred, uint32_t* smem) {
  constexpr int C = 8;
  constexpr float kXScale = 4096.f, kAccScale = 256.f;
  typedef _Float16 half2v __attribute__((ext_vector_type(2)));
  const int tid = threadIdx.x, lane = tid & (kWave - 1);
  const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  const int n = lane & 15, g = lane >> 4;
  constexpr int kParts = 256 / SW;                       // threads per staged column
  const int c0 = tile * plan.cols, len = min(nb_cur - c0, plan.cols);
  const float* hist_inst = hist + (size_t)inst * R * nb_cap;

  uint32_t* s_x = smem;                                                        // [seg_strips + 2][SW]
  float2* s_sum = reinterpret_cast<float2*>(smem + (plan.seg_strips + 2) * SW);   // [2][SW]
  unsigned long long* s_mask = reinterpret_cast<unsigned long long*>(s_sum);   // [256]
  uint32_t* s_act = smem + (plan.seg_strips + 2) * SW + rebase_sum_words(SW);  // [SW]
  uint32_t* s_cnt = s_act + SW;                                                // [wave 4][kRbStrips]
  uint8_t* s_list = reinterpret_cast<uint8_t*>(s_cnt);                         // [SW]
  unsigned long long* s_out = reinterpret_cast<unsigned long long*>(s_cnt + 4 * kRbStrips);   // [wave 4]

  const rb_float4* s_dc = reinterpret_cast<rb_float4*>(s_out + 4) + (g & 1);   // [start, clamp][row type 4][channel half 2]

  // Operand tables and per-lane constants.
  const half8* tab2 = reinterpret_cast<const half8*>(wts_global + kMfmaTableFloatOffset) + kMfmaTableHalfs / 8;
  half8 A2[2][3];                                        // [which half of B holds the earlier pair][tap]
#pragma unroll
  for (int o = 0; o < 2; ++o)
#pragma unroll
    for (int kw = 0; kw < 3; ++kw) A2[o][kw] = tab2[(o * 3 + kw) * kWave + lane];
  const half4 A1 = reinterpret_cast<const half4*>(tab2 + 6 * kWave)[lane];
  const rb_float4* dc = reinterpret_cast<const rb_float4*>(wts_global + delta_const_offset(C, C)) + (g & 1);   // channels 4 (g % 2) ..
  const rb_float4 b1acc = kAccScale * dc[0], b2all = kAccScale * dc[(2 * C + kRowAll * C) / 4];
  const rb_float4 lo2all = kAccScale * dc[(2 * C + (4 + kRowAll) * C) / 4];
  const rb_float4 w3v = (1.f / kAccScale) * reinterpret_cast<const rb_float4*>(wts_global + 10 * C + 9 * C * C + C)[g & 1];
  half4 lo1h;
  {
    const rb_float4 lo1 = kAccScale * dc[C / 4];
#pragma unroll
    for (int c = 0; c < 4; ++c) lo1h[c] = (_Float16)lo1[c];
  }
  if (tid < 8 * C) reinterpret_cast<float*>(s_out + 4)[tid] = kAccScale * wts_global[delta_const_offset(C, C) + 2 * C + tid];
  float inf = INFINITY;                                  // opaque, so that med3(a, lo, inf) stays one instruction
  asm volatile("" : "+v"(inf));

  const int n_strips = (H + 1) / 2;
  const int col = tid & (SW - 1), part = __builtin_amdgcn_readfirstlane(tid / SW);   // staged column, and which of its x pairs
  const int j_col = c0 - kRbHalo + col;                  // its column of the tile
  const bool is_out = part == 0 && col >= kRbHalo && col < kRbHalo + len;
  float total_int = 0.f, total_bor = 0.f;                // of this thread's column

#pragma unroll 1
  for (int t0 = 0; t0 < n_strips; t0 += plan.seg_strips) {
    const int n_seg = min(plan.seg_strips, n_strips - t0);
    const uint32_t seg_mask = n_seg == 32 ? ~0u : (1u << n_seg) - 1u;
    // x pairs t0 - 1 .. t0 + n_seg: f16 of 2^12 x, zero outside the window and the tile, and a bit for each that is not zero.
    // A thread takes a run of its column's pairs, sixteen rows on their way at a time.
    {
      const bool last_seg = t0 + n_seg == n_strips;
      const int lo = t0 == 0 ? 1 : 0, hi = n_seg + 2 - (last_seg ? 1 : 0), per = (hi - lo + kParts - 1) / kParts;
      const int i_begin = lo + part * per, i_end = min(hi, i_begin + per);
      const uint32_t keep = j_col >= 0 && j_col < nb_cur ? ~0u : 0u;
      // (rows as scalar byte offsets into the instance's ring, walked from slot to slot)
      const uint32_t j_load = (uint32_t)min(max(j_col, 0), nb_cur - 1) * 4u, row_bytes = (uint32_t)nb_cap * 4u;
      int row = 2 * (t0 - 1 + i_begin), slot = ring_slot(newest_slot, H, R, min(row, H - 1));
      if (part == 0 && t0 == 0) s_x[col] = 0u;
      if (part == 0 && last_seg) s_x[(n_seg + 1) * SW + col] = 0u;
      unsigned long long mask = 0;
#pragma unroll 1
      for (int i0 = i_begin; i0 < i_end; i0 += kRbBatch) {
        float x[kRbBatch][2];
#pragma unroll
        for (int u = 0; u < kRbBatch; ++u) {
#pragma unroll
          for (int r = 0; r < 2; ++r) {                  // (past the last row the last one again)
            x[u][r] = *reinterpret_cast<const float*>(reinterpret_cast<const char*>(hist_inst) + (j_load + (uint32_t)slot * row_bytes));
            if (++row < H && ++slot == R) slot = 0;
          }
        }
#pragma unroll
        for (int u = 0; u < kRbBatch; ++u)               // (all on their way before the first is used)
          asm volatile("" : "+v"(x[u][0]), "+v"(x[u][1]));
        uint32_t bits = 0u;
#pragma unroll
        for (int u = 0; u < kRbBatch; ++u) {
          if (i0 + u >= i_end) break;
          const int i = i0 + u;
          const half2v h = {(_Float16)(x[u][0] * kXScale), (_Float16)(x[u][1] * kXScale)};
          const uint32_t rows = 2 * (t0 + i) > H ? 0xffffu : ~0u;      // (the second row is row H)
          const uint32_t w = __builtin_bit_cast(uint32_t, h) & (keep & rows);
          s_x[i * SW + col] = w;
          bits |= (w & 0x7fff7fffu) != 0u ? 1u << u : 0u;
        }
        mask |= (unsigned long long)bits << i0;
      }
      s_mask[tid] = mask;
    }
    __syncthreads();
    // The strips that matter to an output column: those that a value within two columns reaches.
    uint32_t act = 0u;
    if (is_out) {
      unsigned long long m = 0;
      for (int p = 0; p < kParts; ++p)
#pragma unroll
        for (int d = -2; d <= 2; ++d) m |= s_mask[p * SW + col + d];
      act = (uint32_t)(m | (m >> 1) | (m >> 2)) & seg_mask;
      if (j_col == 0 || j_col == nb_cur - 1) act = seg_mask;       // (beside the tile y1 = 0 stands for d1 = lo1)
    }
    uint32_t active = 0u;                                // lane t: columns of this wave to which strip t matters
#pragma unroll
    for (int t = 0; t < kRbStrips; ++t) {
      const uint32_t c = (uint32_t)__popcll(__ballot((int)(act << (kRbStrips - 1 - t)) < 0));
      asm("v_writelane_b32 %0, %1, %2" : "+v"(active) : "s"(c), "n"(t));
    }
    if (lane < kRbStrips) s_cnt[wave * kRbStrips + lane] = active;
    __syncthreads();
    uint32_t in_all = 0u;
    if (lane < kRbStrips) in_all = (s_cnt[lane] + s_cnt[kRbStrips + lane]) + (s_cnt[2 * kRbStrips + lane] + s_cnt[3 * kRbStrips + lane]);
    const uint32_t dense = (uint32_t)__ballot(2 * (int)in_all > len) & seg_mask;        // strips evaluated in every column
    if (part == 0) {
      s_sum[col] = s_sum[SW + col] = make_float2(0.f, 0.f);        // (the masks have been read)
      s_act[col] = act & ~dense;
    }
    {
      const unsigned long long o = __ballot((act & ~dense) != 0u);
      if (lane == 0) s_out[wave] = o;
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

    const int n_dense = dense ? (len + kRbOut - 1) / kRbOut : 0;
    // Few listed columns: two waves take an item's strips by halves (their two sums are added in either order with the same result).
    const int n_listed = n_list > 2 ? (n_list - 2 + kRbOut - 1) / kRbOut : 0, halves = n_listed <= 2 ? 1 : 0;
    const int n_items = n_dense + (n_listed << halves);
#pragma unroll 1
    for (int item = wave; item < n_items; item += 4) {
      const bool listed = item >= n_dense;
      const int e0 = (listed ? (item - n_dense) >> halves : item) * kRbOut;
      int at[2];                                         // this lane's staged columns
      bool output[2], outside[2];
      uint32_t S = 0u;
#pragma unroll
      for (int b = 0; b < 2; ++b) {
        const int p = 16 * b + n, e = e0 + p;
        output[b] = p >= 1 && p <= kRbOut;
        if (listed) {
          at[b] = s_list[min(e, n_list - 1)];
          const uint32_t a = s_act[at[b]];
          output[b] = output[b] && e < n_list - 1 && a != 0u;
          S |= output[b] ? a : 0u;
        } else {
          at[b] = min(kRbHalo - 1 + e, SW - 3);
          output[b] = output[b] && at[b] < kRbHalo + len;
        }
        const int j = c0 - kRbHalo + at[b];
        outside[b] = j < 0 || j >= nb_cur;
      }
      if (listed) {
        S |= dpp_row<0xB1>(0u, S);                       // quad_perm [1,0,3,2]
        S |= dpp_row<0x4E>(0u, S);                       // quad_perm [2,3,0,1]
        S |= dpp_row<0x141>(0u, S);                      // row_half_mirror
        S |= dpp_row<0x140>(0u, S);                      // row_mirror
        S = __builtin_amdgcn_readfirstlane(S);           // (the rows of 16 lanes hold the same columns)
        if (halves) {
          const uint32_t early = (1u << (n_seg / 2)) - 1u;
          S &= ((item - n_dense) & 1) ? ~early : early;
        }
      } else {
        S = dense;
      }
      const bool border = __any(outside[0] || outside[1]);
      // Where this lane's two words of x pair t0 - 1 (or t0) begin.
      const uint32_t* xa[2];
#pragma unroll
      for (int b = 0; b < 2; ++b) xa[b] = s_x + at[b] - 1 + (g & 1) + (g >> 1) * SW;

      typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
      auto words = [&](int b, int j) __attribute__((always_inline)) { return u32x2{xa[b][j * SW], xa[b][j * SW + 1]}; };
      auto first_layer = [&](u32x2 w) __attribute__((always_inline)) {
        return __builtin_amdgcn_mfma_f32_16x16x16f16(A1, __builtin_bit_cast(half4, w), b1acc, 0, 0, 0);
      };
      // y1 pair from its result: this lane's four channels of one of the two rows, in two registers.
      auto clamped = [&](int b, rb_float4 acc, auto border_tag) __attribute__((always_inline)) {
        half4 h;
#pragma unroll
        for (int c = 0; c < 4; ++c) h[c] = (_Float16)acc[c];
        h = __builtin_elementwise_max(h, lo1h);
        if (decltype(border_tag)::value) h = outside[b] ? lo1h : h;    // layer-2 padding: y1 = 0 beside the tile, d1 = lo1
        return __builtin_bit_cast(u32x2, h);
      };
      // Layer-2 operands of the two blocks, per tap: the pair in half `half` of the K entries.
      uint4v centre[2], left[2], right[2];
      auto put = [&](const u32x2 (&y)[2], auto half_tag) __attribute__((always_inline)) {
        constexpr int o = 2 * decltype(half_tag)::value;
#pragma unroll
        for (int r = 0; r < 2; ++r) {
#pragma unroll
          for (int b = 0; b < 2; ++b) centre[b][o + r] = y[b][r];
          left[0][o + r] = dpp_all<kRowRor1>(y[0][r]);                 // (lane 0: its own column 15, wanted by block 1)
          left[1][o + r] = dpp_row<kRowShr1>(left[0][o + r], y[1][r]);
          right[1][o + r] = dpp_all<kRowRor15>(y[1][r]);               // (lane 15: its own column 0)
          right[0][o + r] = dpp_row<kRowShl1>(right[1][o + r], y[0][r]);
        }
      };
      // Layer 2 and the head: four weighted channels of one output row of each block.
      auto second_layer = [&](rb_float4 start, rb_float4 lo, float (&sum)[2], auto order_tag) __attribute__((always_inline)) {
        constexpr int o = decltype(order_tag)::value;
        rb_float4 acc[2];
#pragma unroll
        for (int b = 0; b < 2; ++b) acc[b] = __builtin_amdgcn_mfma_f32_16x16x32_f16(A2[o][1], __builtin_bit_cast(half8, centre[b]), start, 0, 0, 0);
#pragma unroll
        for (int b = 0; b < 2; ++b) acc[b] = __builtin_amdgcn_mfma_f32_16x16x32_f16(A2[o][0], __builtin_bit_cast(half8, left[b]), acc[b], 0, 0, 0);
#pragma unroll
        for (int b = 0; b < 2; ++b) acc[b] = __builtin_amdgcn_mfma_f32_16x16x32_f16(A2[o][2], __builtin_bit_cast(half8, right[b]), acc[b], 0, 0, 0);
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
          for (int c = 0; c < 4; ++c) sum[b] = fmaf(w3v[c], __builtin_amdgcn_fmed3f(acc[b][c], lo[c], inf), sum[b]);
      };
      constexpr std::integral_constant<int, 0> kFirst{};
      constexpr std::integral_constant<int, 1> kSecond{};
      float sum_int[2] = {0.f, 0.f}, sum_bor[2] = {0.f, 0.f};

      // Strips that hold a border row: y1 rows outside the window are no terms at all, rows 0 and H-1 have constants of their own.
      uint32_t edges = 0u;
      if (t0 == 0) edges |= 1u;
      for (int t = max((H - 2) / 2, t0); t < t0 + n_seg; ++t) edges |= 1u << (t - t0);
      uint32_t E = S & edges;
      S &= ~edges;
#pragma unroll 1
      while (E != 0u) {
        const int j = __builtin_ctz(E);
        E &= E - 1u;
        const int t = t0 + j, row = 2 * t + (g >> 1);    // this lane's output row
#pragma unroll
        for (int k = 0; k < 2; ++k) {
          const int row1 = 2 * (t + k) - 1 + (g >> 1);   // its y1 row of pair t + k
          u32x2 y[2];
#pragma unroll
          for (int b = 0; b < 2; ++b) {
            y[b] = clamped(b, first_layer(words(b, j + k)), std::true_type{});
            if (row1 < 0 || row1 >= H) y[b] = u32x2{0u, 0u};
          }
          if (k == 0) put(y, kFirst); else put(y, kSecond);
        }
        const int type = row == 0 ? kRowTop : row == H - 1 ? kRowBot : kRowAll;
        float s[2] = {0.f, 0.f};
        second_layer(s_dc[type * 2], s_dc[(4 + type) * 2], s, kFirst);
#pragma unroll
        for (int b = 0; b < 2; ++b) {
          if (row >= 2 && row <= H - 3) sum_int[b] += s[b];
          else if (row < H) sum_bor[b] += s[b];
        }
      }
      // The others, in runs of consecutive strips; the pair a strip and the next one share is evaluated once.  The first layer of
      // the pair after the next and its words are under way while a strip is worked on (at a run's end for nothing).
      auto runs = [&](auto border_tag) __attribute__((always_inline)) {
#pragma unroll 1
        while (S != 0u) {
          int j = __builtin_ctz(S);
          rb_float4 d1[2];
          u32x2 y[2], w[2];
#pragma unroll
          for (int b = 0; b < 2; ++b) { y[b] = clamped(b, first_layer(words(b, j)), border_tag); d1[b] = first_layer(words(b, j + 1)); w[b] = words(b, j + 2); }
          put(y, kFirst);
          auto strip = [&](auto half_tag, auto order_tag) __attribute__((always_inline)) {
#pragma unroll
            for (int b = 0; b < 2; ++b) y[b] = clamped(b, d1[b], border_tag);
            put(y, half_tag);
#pragma unroll
            for (int b = 0; b < 2; ++b) { d1[b] = first_layer(w[b]); w[b] = words(b, j + 3); }
            second_layer(b2all, lo2all, sum_int, order_tag);
            S &= S - 1u;
            ++j;
            return S != 0u && (int)__builtin_ctz(S) == j;
          };
#pragma unroll 1
          for (;;) {
            if (!strip(kSecond, kFirst)) break;
            if (!strip(kFirst, kSecond)) break;
          }
        }
      };
      if (border) runs(std::true_type{}); else runs(std::false_type{});
#pragma unroll
      for (int b = 0; b < 2; ++b) {
        const float si = add_lane_groups(sum_int[b]), sb = add_lane_groups(sum_bor[b]);
        if (g == 0 && output[b]) {
          float2* to = s_sum + (listed ? SW : 0) + at[b];
          atomicAdd(&to->x, si);                         // (onto zero: the same as a store, but for an item in halves)
          atomicAdd(&to->y, sb);
        }
      }
    }
    __syncthreads();
    if (part == 0) {
      const float2 d = s_sum[col], l = s_sum[SW + col];
      total_int += d.x + l.x;
      total_bor += d.y + l.y;
    }
    if (t0 + n_seg < n_strips) __syncthreads();          // (the next segment's masks lie where the sums are)
  }
  if (is_out) {
    const size_t o = (size_t)inst * nb_cap + j_col;
    pstate[o] = total_int;
    pred[o] = (total_int + total_bor) * (1.f / (float)H);
  }
}

}  // namespace
}  // namespace ap
