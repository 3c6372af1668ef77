// Block-sparse GQA decode attention and dense calibration for gfx950.
//
// Two forms.  The streaming one (sparse_stream_body; calibrate_stream_kernel in attention.hip) is described where it stands.
// The phased one - sparse decode of whole bf16 lists with g <= 4 and of fp32 lists, fp32 calibration - goes through
//   1. logits  l[h][tok] = (q_h . K_tok) / sqrt(d) for the tokens of a list of blocks, fp32
//      accumulate, written to LDS (tokens at or beyond t_cur get -inf);
//   2. per head: M = max l, p = exp(l - M) in place, L = sum p; per (head, block) the max p.
// Sparse decode continues with  3. acc[h][:] = sum_tok p[h][tok] * V_tok  and either finishes
// (one workgroup per instance) or leaves (M, L, acc, block maxima) for the merge: by the last workgroup of the instance to finish or
// by the combine kernel (merge_inside in attention.hip).
// Softmax definition: Sec. 3.1; block max-pooling of the probabilities: Algorithm 1 steps 1-2
// (softmax is monotone, so the pooled probability of a block is exp(max logit - M) / L).
//
// Memory access: a K or V row is d * sizeof(T) bytes (256 B for bf16, d = 128).  LPT = row bytes / 16
// adjacent lanes read one row with one 16-byte load each, so every load instruction of a wave covers
// 64 / LPT whole rows = 1 KiB of contiguous memory inside a block.
#pragma once

#include <type_traits>

#include "select_body.h"

namespace ap {
namespace {


struct bf16_t { uint16_t bits; };
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float float4v __attribute__((ext_vector_type(4)));

template <typename T> struct KvT;
template <> struct KvT<float> { static constexpr int E = 4; };
template <> struct KvT<bf16_t> { static constexpr int E = 8; };

__device__ __forceinline__ void unpack16(const uint4& w, float (&f)[4], float) {
  f[0] = __uint_as_float(w.x); f[1] = __uint_as_float(w.y);
  f[2] = __uint_as_float(w.z); f[3] = __uint_as_float(w.w);
}
__device__ __forceinline__ void unpack16(const uint4& w, float (&f)[8], bf16_t) {
  f[0] = __uint_as_float(w.x << 16); f[1] = __uint_as_float(w.x & 0xffff0000u);
  f[2] = __uint_as_float(w.y << 16); f[3] = __uint_as_float(w.y & 0xffff0000u);
  f[4] = __uint_as_float(w.z << 16); f[5] = __uint_as_float(w.z & 0xffff0000u);
  f[6] = __uint_as_float(w.w << 16); f[7] = __uint_as_float(w.w & 0xffff0000u);
}

// V rows and bf16 K rows are read once per call, a whole row per load instruction (the K rows through a staged
// tile, see qk_logits): 16-byte non-temporal loads, which stream faster than plain ones and keep the rows
// from displacing data that is re-used from cache.
template <typename T> __device__ __forceinline__ uint4 ld_stream(const T* p) {
  typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
  const u32x4 v = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(p));
  return make_uint4(v.x, v.y, v.z, v.w);
}

template <int CTRL> __device__ __forceinline__ float dpp_move(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xF, 0xF, true));
}

// Sum over the LPT adjacent lanes that share one token; every lane of the group gets the total.
template <int LPT> __device__ __forceinline__ float lane_group_sum(float v) {
  v += dpp_move<0xB1>(v);                       // quad_perm [1,0,3,2]
  v += dpp_move<0x4E>(v);                       // quad_perm [2,3,0,1]
  if (LPT >= 8) v += dpp_move<0x141>(v);        // row_half_mirror: pairs the two quads of 8 lanes
  if (LPT >= 16) v += dpp_move<0x140>(v);       // row_mirror: pairs the two halves of 16 lanes
  if (LPT >= 32) v += __shfl_xor(v, 16, 64);
  return v;
}

// Reductions over the 64 lanes on DPP moves - shifts within the rows of 16 lanes, then the last lane of row 0 / 2
// combined into row 1 / 3 and the last lane of row 1 into rows 2 and 3 - so that lane 63 holds the result, which a
// scalar read hands to every lane: register moves instead of six trips through the LDS permute path.  Every lane
// must be active.  FILL is the value shifted in at a row's start and kept by rows a step does not address.
template <int CTRL, int ROW_MASK> __device__ __forceinline__ float dpp_fill(float fill, float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(fill), __float_as_int(v), CTRL, ROW_MASK, 0xF, false));
}
__device__ __forceinline__ float wave_max(float v) {
  v = fmaxf(v, dpp_fill<0x111, 0xF>(-INFINITY, v));     // row_shr:1
  v = fmaxf(v, dpp_fill<0x112, 0xF>(-INFINITY, v));     // row_shr:2
  v = fmaxf(v, dpp_fill<0x114, 0xF>(-INFINITY, v));     // row_shr:4
  v = fmaxf(v, dpp_fill<0x118, 0xF>(-INFINITY, v));     // row_shr:8
  v = fmaxf(v, dpp_fill<0x142, 0xA>(-INFINITY, v));     // row_bcast:15 into rows 1 and 3
  v = fmaxf(v, dpp_fill<0x143, 0xC>(-INFINITY, v));     // row_bcast:31 into rows 2 and 3
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), kWave - 1));
}
__device__ __forceinline__ float wave_sum(float v) {
  v += dpp_fill<0x111, 0xF>(0.f, v);
  v += dpp_fill<0x112, 0xF>(0.f, v);
  v += dpp_fill<0x114, 0xF>(0.f, v);
  v += dpp_fill<0x118, 0xF>(0.f, v);
  v += dpp_fill<0x142, 0xA>(0.f, v);
  v += dpp_fill<0x143, 0xC>(0.f, v);
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), kWave - 1));
}

constexpr float kLog2E = 1.44269504088896340736f;
__device__ __forceinline__ float exp2_fast(float x) { return __builtin_amdgcn_exp2f(x); }

template <typename T, int D, int G> struct Geom {
  static constexpr int E = KvT<T>::E;           // elements per 16-byte load
  static constexpr int LPT = D / E;             // lanes per token row
  static constexpr int TPI = kWave / LPT;       // token rows per load instruction
  static constexpr int NL = kGroupTokens / TPI; // load instructions per 16-token group
  static_assert(LPT >= 8 && LPT <= 32 && G <= LPT, "unsupported geometry");
};

// Phase 1.  `block_of(jb)` gives the logical block index of list position jb (its token positions decide the
// causal mask), `phys_of(jb)` the block's place in K (the same unless a block table is in use).  s_p is [G][ld].
//
// bf16: the g x d by d x 16-token contraction runs on v_mfma_f32_16x16x32_bf16 (A = 16 K rows, B = q^T
// padded to 16 columns, fp32 accumulate); with VALU dot products plus cross-lane sums the kernel spends
// two thirds of its issue slots on arithmetic and cannot keep HBM busy.  In the operand layout lane l supplies
// token l % 16 and, the order of the contraction index being free as long as A and B agree, dims
// (l / 16) d/4 .. + d/4 - 1, eight per K-step.  D comes back as lane (head = l % 16, 4 (l / 16) + v = token), so
// lanes with head < G hold the logits.
// The K rows do not come from global memory in that layout (a row would get 64 bytes per load instruction):
// they are fetched whole - LPT adjacent lanes read one row with non-temporal loads, as V rows are - and pass
// through a wave-private LDS tile from which the operand layout is read.  A plain streaming read
// of this machine is 14 % faster with non-temporal loads, but only if an instruction covers whole 128-byte lines;
// a non-temporal load of part of a line fetches the line again for the other part.
// The tile has 8 rows, two passes per 16 tokens through an MFMA whose other eight rows repeat the tile: it fits into the
// region that holds the output partials later.
// fp32 K/V keeps the VALU form: LPT adjacent lanes share one row, 16 bytes each.
constexpr int kStageRowPad = 16;   // bytes added to a staged K row so that 16 rows spread over the LDS banks
template <int D, int ROWS = kGroupTokens, int NW = kAttnWaves> constexpr int k_stage_floats() {
  return NW * ROWS * (D * 2 + kStageRowPad) / 4;
}

template <typename T, int D, int G, int STAGE, int NW = kAttnWaves, class BlockOf, class PhysOf>
__device__ __forceinline__ void qk_logits(const T* __restrict__ q_inst, const T* __restrict__ K_inst, int b, int log2b,
                                          int t_cur, int ntok, BlockOf block_of, PhysOf phys_of, float* s_p, int ld,
                                          float* s_stage) {
  const int lane = threadIdx.x & (kWave - 1);
  const int wave = threadIdx.x / kWave;
  const float scale = rsqrtf((float)D);
  const int ngroups = (ntok + kGroupTokens - 1) / kGroupTokens;
  if constexpr (std::is_same<T, bf16_t>::value) {
    constexpr int KS = D / 32;
    const int row = lane & 15, g = lane >> 4;
    bf16x8 qb[KS];
#pragma unroll
    for (int s = 0; s < KS; ++s) {
      uint4 w = make_uint4(0, 0, 0, 0);
      if (row < G) w = *reinterpret_cast<const uint4*>(q_inst + (size_t)row * D + g * (D / 4) + s * 8);
      qb[s] = __builtin_bit_cast(bf16x8, w);
    }
    {
      static_assert(STAGE == 8, "bf16 K rows go through a staged tile of 8 rows");
      constexpr int ROWS = STAGE;                        // tokens per pass
      constexpr int NPRE = 2;                            // passes of a wave in flight (3, 4 and 6 measured the same)
      constexpr int LPT = D / 8, TPI = kWave / LPT, NLK = ROWS / TPI, RS = D * 2 + kStageRowPad;
      static_assert(NLK >= 1, "a pass is at least one load instruction");
      char* stage = reinterpret_cast<char*>(s_stage) + wave * ROWS * RS;
      const int npass = (ntok + ROWS - 1) / ROWS;
      auto load_pass = [&](int ps, uint4 (&v)[NLK]) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < NLK; ++i) {
          const int tau = ps * ROWS + i * TPI + lane / LPT;
          v[i] = make_uint4(0, 0, 0, 0);
          if (tau < ntok) {
            const int ptok = phys_of(tau >> log2b) * b + (tau & (b - 1));
            v[i] = ld_stream(K_inst + (size_t)ptok * D + (lane % LPT) * 8);
          }
        }
      };
      // One pass: stage the fetched rows, refill the registers with pass `refill` (NPRE passes of this wave ahead),
      // contract, store the logits.
      auto do_pass = [&](int ps, uint4 (&v)[NLK], int refill) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < NLK; ++i)
          *reinterpret_cast<uint4*>(stage + (i * TPI + lane / LPT) * RS + (lane % LPT) * 16) = v[i];
        asm volatile("" ::: "memory");                   // a wave's LDS accesses stay in order; so must the compiler
        if (refill < npass) load_pass(refill, v);
        float4v acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int s = 0; s < KS; ++s) {
          const uint4 kw = *reinterpret_cast<const uint4*>(stage + (row & (ROWS - 1)) * RS + (g * (D / 4) + s * 8) * 2);
          acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, kw), qb[s], acc, 0, 0, 0);
        }
        asm volatile("" ::: "memory");                   // the next pass overwrites the tile read above
        // lane (head = row, tokens 4 g .. 4 g + 3 of the pass); with 8 rows only g < 2 holds tokens
        const int tau0 = ps * ROWS + 4 * g;
        if (row < G && 4 * g < ROWS && tau0 < ntok) {
          const int gtok0 = block_of(tau0 >> log2b) * b + (tau0 & (b - 1));
          float4 o;
          o.x = gtok0 + 0 < t_cur ? acc[0] * scale : -INFINITY;
          o.y = gtok0 + 1 < t_cur ? acc[1] * scale : -INFINITY;
          o.z = gtok0 + 2 < t_cur ? acc[2] * scale : -INFINITY;
          o.w = gtok0 + 3 < t_cur ? acc[3] * scale : -INFINITY;
          *reinterpret_cast<float4*>(s_p + row * ld + tau0) = o;
        }
      };
      // Rows of this wave's next NPRE passes wait in registers.
      uint4 v[NPRE][NLK];
#pragma unroll
      for (int i = 0; i < NPRE; ++i)
        if (wave + i * NW < npass) load_pass(wave + i * NW, v[i]);
      for (int ps = wave; ps < npass; ps += NPRE * NW) {
#pragma unroll
        for (int i = 0; i < NPRE; ++i)
          if (ps + i * NW < npass) do_pass(ps + i * NW, v[i], ps + (i + NPRE) * NW);
      }
    }
  } else {
    using Ge = Geom<T, D, G>;
    constexpr int E = Ge::E, LPT = Ge::LPT, TPI = Ge::TPI, NL = Ge::NL;
    const int dpart = lane % LPT;
    const int tslot = lane / LPT;
    float qr[G][E];
#pragma unroll
    for (int h = 0; h < G; ++h) {
      static_assert(E * sizeof(T) == 16, "one 16-byte load per lane");
      uint4 w = *reinterpret_cast<const uint4*>(q_inst + (size_t)h * D + dpart * E);
      float f[E];
      unpack16(w, f, T{});
#pragma unroll
      for (int e = 0; e < E; ++e) qr[h][e] = f[e] * scale;
    }
    for (int grp = wave; grp < ngroups; grp += NW) {
      uint4 kw[NL];
      int gtok[NL];
#pragma unroll
      for (int i = 0; i < NL; ++i) {
        const int tau = grp * kGroupTokens + i * TPI + tslot;
        kw[i] = make_uint4(0, 0, 0, 0);
        gtok[i] = -1;
        if (tau < ntok) {
          gtok[i] = block_of(tau >> log2b) * b + (tau & (b - 1));
          const int ptok = phys_of(tau >> log2b) * b + (tau & (b - 1));
          kw[i] = *reinterpret_cast<const uint4*>(K_inst + (size_t)ptok * D + dpart * E);
        }
      }
#pragma unroll
      for (int i = 0; i < NL; ++i) {
        const int tau = grp * kGroupTokens + i * TPI + tslot;
        float kf[E];
        unpack16(kw[i], kf, T{});
        float mine = 0.f;
#pragma unroll
        for (int h = 0; h < G; ++h) {
          float sdot = 0.f;
#pragma unroll
          for (int e = 0; e < E; ++e) sdot = fmaf(qr[h][e], kf[e], sdot);
          sdot = lane_group_sum<LPT>(sdot);
          if (dpart == h) mine = sdot;
        }
        if (dpart < G && tau < ntok) s_p[dpart * ld + tau] = (gtok[i] < t_cur) ? mine : -INFINITY;
      }
    }
  }
}

// Phase 2.  Leaves p in s_p, (M, L) in s_m / s_l, per (head, block) max p in s_bmp[h * bmp_ld + jb].
// One wave per head; a lane handles four consecutive tokens per 16-byte LDS access (ntok and ld are multiples
// of the block size, hence of 4), so the b / 4 adjacent lanes of a block find its maximum with DPP moves.
// With s_alpha the statistics run on over several calls (pieces of one list): M is the maximum so far, p is
// relative to it, L is carried over as L * alpha + sum with alpha = exp(M_before - M), which s_alpha[h]
// receives for the caller to rescale what it has accumulated (0 on the first piece, M_before = -inf).
template <int G, int NW = kAttnWaves>
__device__ __forceinline__ void softmax_stats(float* s_p, int ld, int ntok, int b, int bmp_ld, float* s_m, float* s_l,
                                     float* s_bmp, float* s_alpha = nullptr) {
  const int lane = threadIdx.x & (kWave - 1);
  const int wave = threadIdx.x / kWave;
  const int nquad = ntok >> 2;
  const int lanes_per_blk = b >> 2;                      // 2, 4, 8 or 16
  const int blk_shift = __ffs(lanes_per_blk) - 1;
  // Heads wave, wave + NW, ... of this wave are worked on together: their loads, reductions and exponentials
  // are independent chains that hide each other's latency.
  constexpr int HPW = (G + NW - 1) / NW;
  float m[HPW], m_old[HPW], l_old[HPW], sum[HPW];
#pragma unroll
  for (int j = 0; j < HPW; ++j) { m[j] = -INFINITY; m_old[j] = -INFINITY; l_old[j] = 0.f; sum[j] = 0.f; }
  for (int qd = lane; qd < nquad; qd += kWave) {
#pragma unroll
    for (int j = 0; j < HPW; ++j) {
      const int h = wave + j * NW;
      if (h < G) {
        const float4 v = reinterpret_cast<const float4*>(s_p + (size_t)h * ld)[qd];
        m[j] = fmaxf(m[j], fmaxf(fmaxf(v.x, v.y), fmaxf(v.z, v.w)));
      }
    }
  }
#pragma unroll
  for (int j = 0; j < HPW; ++j) m[j] = wave_max(m[j]);   // (independent chains: the compiler interleaves them)
  if (s_alpha != nullptr) {
#pragma unroll
    for (int j = 0; j < HPW; ++j) {
      const int h = wave + j * NW;
      if (h < G) {
        m_old[j] = s_m[h];
        l_old[j] = s_l[h];
        m[j] = fmaxf(m[j], m_old[j]);
      }
    }
  }
  for (int q0 = 0; q0 < nquad; q0 += kWave) {            // uniform trip count: the DPP moves need every lane
    const int qd = q0 + lane;
#pragma unroll
    for (int j = 0; j < HPW; ++j) {
      const int h = wave + j * NW;
      if (h >= G) continue;                              // (wave-uniform)
      float4* prow = reinterpret_cast<float4*>(s_p + (size_t)h * ld);
      float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
      if (qd < nquad) {
        v = prow[qd];
        v.x = __expf(v.x - m[j]); v.y = __expf(v.y - m[j]); v.z = __expf(v.z - m[j]); v.w = __expf(v.w - m[j]);
        prow[qd] = v;
      }
      sum[j] += (v.x + v.y) + (v.z + v.w);
      float bm = fmaxf(fmaxf(v.x, v.y), fmaxf(v.z, v.w));
      bm = fmaxf(bm, dpp_move<0xB1>(bm));                                   // quad_perm [1,0,3,2]
      if (lanes_per_blk >= 4) bm = fmaxf(bm, dpp_move<0x4E>(bm));           // quad_perm [2,3,0,1]
      if (lanes_per_blk >= 8) bm = fmaxf(bm, dpp_move<0x141>(bm));          // row_half_mirror
      if (lanes_per_blk >= 16) bm = fmaxf(bm, dpp_move<0x140>(bm));         // row_mirror
      if (qd < nquad && (lane & (lanes_per_blk - 1)) == 0) s_bmp[h * bmp_ld + (qd >> blk_shift)] = bm;
    }
  }
#pragma unroll
  for (int j = 0; j < HPW; ++j) sum[j] = wave_sum(sum[j]);
  if (lane == 0) {
#pragma unroll
    for (int j = 0; j < HPW; ++j) {
      const int h = wave + j * NW;
      if (h < G) {
        const float alpha = (m_old[j] == -INFINITY) ? 0.f : __expf(m_old[j] - m[j]);
        s_m[h] = m[j];
        s_l[h] = l_old[j] * alpha + sum[j];
        if (s_alpha != nullptr) s_alpha[h] = alpha;
      }
    }
  }
  __syncthreads();
}

constexpr int kSparseStage = 8;
// Floats of the region shared by the staged K tile (phase 1) and the per-wave output partials (after phase 3).
template <int D, int G, int NW> constexpr int sparse_acc_floats() {
  return NW * G * D > k_stage_floats<D, kSparseStage, NW>() ? NW * G * D : k_stage_floats<D, kSparseStage, NW>();
}

struct SparseArgs {
  const void* q; const void* K; const void* V;
  const int32_t* idx; const int32_t* cnt;
  float* out; float* row; size_t row_stride;
  float* part_ml; float* part_acc; float* part_bmp;
  int t_cap, nb_cap, k, b, log2b, t_cur, nb_cur, n_split, blk_per_split, inst0;
  const int32_t* table;           // block table [n_inst][nb_cap] of a paged cache, or null
  int n_phys;                     // blocks in the pool (table entries are clamped into it)
  int piece_blocks;               // list positions whose probabilities are in LDS at a time
  float ml_unit;                  // the splits' maxima times this are exponents of 2
  const float* pred;              // scores [n_inst][nb_cap] that the decode selects by itself (kSelectInside), writing idx and cnt
  int n_sink, n_local, sel_at;    // forced blocks; where in LDS (floats) the list goes: k blocks and their number
  unsigned long long* merge_count;  // [n_inst] splits that have left their partials (take_ticket), where they are merged inside
  unsigned long long merge_nonce; // number of this launch in them (kMergeAlone; else they are zero at launch)
  int part_first;                 // instance that part_ml and part_acc begin with (0 but where whole and split lists go in one launch: streaming form, merged by a launch)
};

// What a decode launch does beside its own share: nothing; merging, by the last workgroup of an instance to finish, behind a launch that has cleared
// the counters; before that also the selection, by every workgroup for itself (whole lists too; see select_here); merging without such a launch.
constexpr int kSplitsOnly = 0, kMergeInside = 1, kSelectInside = 2, kMergeAlone = 3;
// Scores a thread holds: up to 2304 candidates.  (Steps of 8 / 32 / 128 instances, us, with 9, 12 and 15 scores a thread: 2042 candidates
// 16.6 16.8 17.2 / 18.5 18.8 19.0 / 28.6 28.6 28.8, one of fp32 with 126 candidates 16.9 and 17.4; 2442, for nine too many, 18.2 17.0 17.3 / 20.4 19.1
// 19.2 / 30.2 29.4 29.7, 2992 18.4 17.1 17.3 / 21.0 19.7 19.9 / 31.7 30.4 30.5, 3692 19.0 18.7 18.0 / 21.4 21.2 20.2 / 34.9 34.2 33.5.  More scores
// a thread win some 1.2 us where they are needed and cost 0.2 to 0.5 where they are not.)
constexpr int kSelectInsideKeys = 9;

// The instance's selection by this workgroup of 256 threads, into LDS at a.sel_at; that of the first split writes idx and cnt too.
// Returns the number of listed blocks.  smem: sel_scratch_words<256>() words that are free until it returns.
__device__ __forceinline__ int select_inside(const SparseArgs& a, int inst, int split, float* smem) {
  static_assert(kAttnThreads == kSelThreads, "one workgroup does both");
  int32_t* s_list = reinterpret_cast<int32_t*>(smem + a.sel_at);
  select_topk_body<kSelectInsideKeys, kSelThreads, 4>(a.pred + (size_t)inst * a.nb_cap, a.nb_cur, a.k, a.n_sink, a.n_local, s_list,
                                                      s_list + a.k, reinterpret_cast<uint32_t*>(smem));
  __syncthreads();
  const int cnt = __builtin_amdgcn_readfirstlane(s_list[a.k]);
  if (split == 0) {
    int32_t* idx = const_cast<int32_t*>(a.idx) + (size_t)inst * a.k;
    for (int j = threadIdx.x; j < cnt; j += kAttnThreads) idx[j] = s_list[j];
    if (threadIdx.x == 0) const_cast<int32_t*>(a.cnt)[inst] = cnt;
  }
  return cnt;
}

// Data that one workgroup leaves for another of the same launch, which may run on another XCD with an L2 of its own: stores that are
// written through to memory, loads that are answered from there (agent scope).  A release of ordinary stores would write back the
// XCD's whole L2 instead, which costs four times a decode's time.
// (SHARED = false: an ordinary store, for a launch behind this one.)
template <bool SHARED> __device__ __forceinline__ void st_shared_out(float* p, float v) {
  if constexpr (SHARED) __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); else *p = v;
}
__device__ __forceinline__ float ld_shared_out(const float* p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }

// Counting without a launch that clears the counter, in a word of the caller's workspace that may hold anything: its upper bits are a number
// that the host draws anew for every launch (new_nonce), the lower kTicketBits the count.  Whoever is going to take a ticket first sees to it that the word carries the number
// (begin_tickets, early, so that nobody waits for the answer: it is at zero where the last launch ended properly, and carries the number already where
// another was faster); the one that gets the last ticket leaves it at zero (end_tickets), so that a captured launch, whose number stands still, starts afresh
// on every replay.  What lies in a fresh workspace is taken for a count once in 2^52 words.  Called by one lane.
// A launch behind one that has cleared the words (of the predictor, of an appended row) only counts.
constexpr int kTicketBits = 12;                         // (kMergeInsideSplits and more)
__device__ __forceinline__ unsigned long long begin_tickets(unsigned long long* word, unsigned long long nonce) {
  unsigned long long seen = 0ull;
  __hip_atomic_compare_exchange_strong(word, &seen, nonce, __ATOMIC_RELAXED, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  return seen;                                           // for take_ticket
}
__device__ __forceinline__ uint32_t take_ticket(unsigned long long* word, unsigned long long nonce, unsigned long long seen) {
  // Neither zero nor this launch's: the word held something else.  It only ever changes from that to the number.
  if (seen != 0ull && ((seen ^ nonce) >> kTicketBits) != 0ull)
    __hip_atomic_compare_exchange_strong(word, &seen, nonce, __ATOMIC_RELAXED, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  return (uint32_t)(__hip_atomic_fetch_add(word, 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) & ((1ull << kTicketBits) - 1ull));
}
__device__ __forceinline__ void end_tickets(unsigned long long* word) { __hip_atomic_store(word, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }

// Called by every thread of a workgroup that has left its partials of an instance: true in the last of n_split to get here.
// TICKETS: as above; without, the word is zero at launch in any case.  s_last: an int of LDS that nothing else uses.
template <bool TICKETS>
__device__ __forceinline__ bool last_to_finish(unsigned long long* count, unsigned long long nonce, unsigned long long seen, int n_split, int* s_last) {
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");       // this wave's partials have reached memory
  __syncthreads();
  if (threadIdx.x == 0) {
    if constexpr (TICKETS) {
      const bool last = (int)take_ticket(count, nonce, seen) == n_split - 1;
      if (last) end_tickets(count);
      *s_last = last;
    } else {
      *s_last = __hip_atomic_fetch_add(reinterpret_cast<uint32_t*>(count), 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == (uint32_t)(n_split - 1);
    }
  }
  __syncthreads();
  return *s_last != 0;
}

// The pooled row of an instance in splits is zero but for the listed blocks: every split clears its share of the columns,
// before its partials are complete, and the last one fills in the values.
__device__ __forceinline__ void clear_row_share(const SparseArgs& a, int inst, int split) {
  const int per = ((a.nb_cap + a.n_split - 1) / a.n_split + 31) & ~31;
  float* row = a.row + (size_t)inst * a.row_stride;
  for (int j = split * per + threadIdx.x; j < min(a.nb_cap, (split + 1) * per); j += kAttnThreads) st_shared_out<true>(row + j, 0.f);
}

constexpr int kMergeInsideSplits = 16;                  // most splits that are merged so (merge_inside in attention.hip)
// LDS of the merge, which overlays what the decode had: factors, and a word for last_to_finish.
inline size_t merge_lds_bytes(int n_split, int g) { return n_split > 1 ? sizeof(float) * ((size_t)n_split * g + 1) : 0; }

// Merges the splits of one instance, by one workgroup of kAttnThreads that has found itself the last: global (M, L) per head, normalised
// output, pooled row.  `block_of(jb)`: block at list position jb < cnt.  smem: merge_lds_bytes(..).  The chain of loads is what it costs, so whatever does not depend on anything is asked
// for first.  (As a launch of its own: sparse_combine_kernel.)
template <int D, int G, class BlockOf>
__device__ __forceinline__ void merge_splits(const SparseArgs& a, int inst, int cnt, BlockOf block_of, float* s_scale) {
  const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
  const float* ml = a.part_ml + (size_t)inst * a.n_split * G * 2;        // [split][head] (maximum, sum relative to it)
  const float* acc = a.part_acc + (size_t)inst * a.n_split * G * D;
  const float* bmp = a.part_bmp + (size_t)inst * G * a.k;
  // This thread's first list position, with its block maxima, and its first outputs of the first splits.
  int blk = -1;
  float bm[G];
  if ((int)threadIdx.x < cnt) {
    blk = block_of(threadIdx.x);
#pragma unroll
    for (int h = 0; h < G; ++h) bm[h] = ld_shared_out(bmp + (size_t)h * a.k + threadIdx.x);
  }
  constexpr int kAhead = 8, PER = G * D > kAttnThreads ? 2 : 1;
  float x[PER][kAhead];
#pragma unroll
  for (int i = 0; i < PER; ++i)
#pragma unroll
    for (int s = 0; s < kAhead; ++s)
      x[i][s] = s < a.n_split && i * kAttnThreads + (int)threadIdx.x < G * D ? ld_shared_out(acc + (size_t)s * G * D + i * kAttnThreads + threadIdx.x) : 0.f;
  // Scales exp2((m - M) unit) / L of every split and head (0 for an empty part or an empty whole): wave h / .. of head h, a lane per
  // split.
  static_assert(kMergeInsideSplits <= kWave, "a lane per split");
  for (int h = wave; h < G; h += kAttnWaves) {
    float m0 = -INFINITY, l0 = 0.f;
    if (lane < a.n_split) {
      m0 = ld_shared_out(ml + 2 * (lane * G + h));
      l0 = ld_shared_out(ml + 2 * (lane * G + h) + 1);
    }
    const float M = wave_max(m0);
    const float L = wave_sum(m0 == -INFINITY ? 0.f : l0 * exp2_fast((m0 - M) * a.ml_unit));
    const float inv = L > 0.f ? 1.f / L : 0.f;
    if (lane < a.n_split) s_scale[lane * G + h] = m0 == -INFINITY ? 0.f : exp2_fast((m0 - M) * a.ml_unit) * inv;
  }
  __syncthreads();
  // (added up in the order of the splits)
  for (int i = 0, o = threadIdx.x; o < G * D; ++i, o += kAttnThreads) {
    const int h = o / D;
    float v = 0.f;
    for (int s0 = 0; s0 < a.n_split; s0 += kAhead) {
      if (s0 > 0 || i >= PER) {
#pragma unroll
        for (int s = 0; s < kAhead; ++s) x[0][s] = s0 + s < a.n_split ? ld_shared_out(acc + (size_t)(s0 + s) * G * D + o) : 0.f;
      }
#pragma unroll
      for (int s = 0; s < kAhead; ++s) {
        const float y = s0 > 0 || i >= PER ? x[0][s] : i == 0 ? x[0][s] : x[PER - 1][s];
        if (s0 + s < a.n_split) v = fmaf(y, s_scale[(s0 + s) * G + h], v);
      }
    }
    a.out[(size_t)inst * G * D + o] = v;
  }
  // pooled probability of list position jb: max over heads of (block max relative to its split) * split scale
  float* row = a.row + (size_t)inst * a.row_stride;
  for (int jb = threadIdx.x; jb < cnt; jb += kAttnThreads) {
    if (jb != (int)threadIdx.x) {
      blk = block_of(jb);
#pragma unroll
      for (int h = 0; h < G; ++h) bm[h] = ld_shared_out(bmp + (size_t)h * a.k + jb);
    }
    const int s = jb / a.blk_per_split;
    float mx = 0.f;
#pragma unroll
    for (int h = 0; h < G; ++h) mx = fmaxf(mx, bm[h] * s_scale[s * G + h]);
    row[blk] = mx;                                       // (a block listed twice: either of two equal values)
  }
}

// Sparse decode of instance `inst`, split `split`, by one workgroup of NW waves.
// The list is worked off in pieces of a.piece_blocks positions - logits, softmax statistics, acc += p * V per
// piece, the statistics running on and acc rescaled when the maximum moves - so that the LDS holds the
// probabilities of one piece only.  PIECED = false: a.piece_blocks covers the list, one piece, no rescaling
// (and the accumulators are not live during phase 1).
// smem: sparse_lds_floats(...) floats of LDS, 16-byte aligned.
template <typename T, int D, int G, int NW, bool PIECED, int HOW>
__device__ __forceinline__ void sparse_decode_body(const SparseArgs& a, int inst, int split, float* smem) {
  using Ge = Geom<T, D, G>;
  constexpr int E = Ge::E, LPT = Ge::LPT, NL = Ge::NL, NT = NW * kWave;
  const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
  const int dpart = lane % LPT, tslot = lane / LPT;

  constexpr bool MERGE = HOW != kSplitsOnly;
  int cnt;
  unsigned long long tickets = 0;                        // (asked for behind the first rows: answers come in order)
  if constexpr (HOW == kSelectInside) cnt = select_inside(a, inst, split, smem); else cnt = min(max(a.cnt[inst], 0), a.k);
  const int32_t* list = HOW == kSelectInside ? reinterpret_cast<const int32_t*>(smem + a.sel_at) : a.idx + (size_t)inst * a.k;
  auto listed = [&](int jb) __attribute__((always_inline)) { return min(max(list[jb], 0), a.nb_cur - 1); };
  // With one workgroup per instance the whole list is local; otherwise this split's slice.
  const int j0 = (a.n_split == 1) ? 0 : min(cnt, split * a.blk_per_split);
  const int j1 = (a.n_split == 1) ? cnt : min(cnt, j0 + a.blk_per_split);
  const int nblk = j1 - j0;
  const int nblk_cap = (a.n_split == 1) ? a.k : a.blk_per_split;
  const int pb = PIECED ? min(a.piece_blocks, nblk_cap) : nblk_cap;   // positions per piece
  const int n_pieces_cap = (nblk_cap + pb - 1) / pb;
  const int ld = pb * a.b;

  float* s_p = smem;                                   // [G][ld]
  float* s_acc = s_p + G * ld;                         // [waves][G][D]
  float* s_bmp = s_acc + sparse_acc_floats<D, G, NW>();   // [G][nblk_cap]
  float* s_m = s_bmp + G * nblk_cap;                   // [G] running maximum
  float* s_l = s_m + G;                                // [G] running sum
  float* s_alpha = s_l + G;                            // [G] rescaling factor of the piece at hand
  float* s_mpiece = s_alpha + G;                       // [n_pieces_cap][G] maximum the piece's p are relative to
  int* s_idx = reinterpret_cast<int*>(s_mpiece + n_pieces_cap * G);   // [nblk_cap] logical block of each position
  int* s_phys = s_idx + nblk_cap;                      // [nblk_cap] its place in K / V
  // For the pooled row, written whole by the workgroup that has the whole list: one bit per block (is it
  // listed) and, per 32-block word, the number of listed blocks before it, so that a column finds its list
  // position without a search.
  uint32_t* s_listed = reinterpret_cast<uint32_t*>(s_phys + nblk_cap);   // [ceil(nb_cap / 32)]
  int* s_rank = reinterpret_cast<int*>(s_listed) + (a.nb_cap + 31) / 32; // [ceil(nb_cap / 32)]
  const int nwords = (a.nb_cap + 31) / 32;
  const bool whole_row = a.n_split == 1;

  if (whole_row) {
    for (int w = threadIdx.x; w < nwords; w += NT) s_listed[w] = 0u;
  }
  if (threadIdx.x < G) { s_m[threadIdx.x] = -INFINITY; s_l[threadIdx.x] = 0.f; }
  if constexpr (MERGE) clear_row_share(a, inst, split);
  __syncthreads();
  for (int j = threadIdx.x; j < nblk; j += NT) {
    const int blk = listed(j0 + j);
    s_idx[j] = blk;
    s_phys[j] = a.table ? min(max(a.table[(size_t)inst * a.nb_cap + blk], 0), a.n_phys - 1) : blk;
    if (whole_row) atomicOr(&s_listed[blk >> 5], 1u << (blk & 31));
  }
  __syncthreads();
  if (whole_row && wave == NW - 1) {                   // exclusive prefix sum of the words' bit counts
    const int per_lane = (nwords + kWave - 1) / kWave;
    const int w0 = lane * per_lane;
    int mine = 0;
    for (int i = 0; i < per_lane; ++i)
      if (w0 + i < nwords) mine += __popc(s_listed[w0 + i]);
    int incl = mine;                                   // inclusive prefix sum over the lanes, on DPP moves
    incl += __builtin_amdgcn_update_dpp(0, incl, 0x111, 0xF, 0xF, true);   // row_shr:1
    incl += __builtin_amdgcn_update_dpp(0, incl, 0x112, 0xF, 0xF, true);   // row_shr:2
    incl += __builtin_amdgcn_update_dpp(0, incl, 0x114, 0xF, 0xF, true);   // row_shr:4
    incl += __builtin_amdgcn_update_dpp(0, incl, 0x118, 0xF, 0xF, true);   // row_shr:8
    incl += __builtin_amdgcn_update_dpp(0, incl, 0x142, 0xA, 0xF, true);   // row_bcast:15 into rows 1 and 3
    incl += __builtin_amdgcn_update_dpp(0, incl, 0x143, 0xC, 0xF, true);   // row_bcast:31 into rows 2 and 3
    int run = incl - mine;
    for (int i = 0; i < per_lane; ++i)
      if (w0 + i < nwords) { s_rank[w0 + i] = run; run += __popc(s_listed[w0 + i]); }
  }                                                    // (read after the barriers that follow)

  // Contiguous cache: [n_inst][t_cap][d].  Paged cache: one pool [n_phys][b][d] for all instances.
  const size_t kv_off = a.table ? 0 : (size_t)inst * a.t_cap * D;
  const T* q_inst = static_cast<const T*>(a.q) + (size_t)inst * G * D;
  const T* K_inst = static_cast<const T*>(a.K) + kv_off;
  const T* V_inst = static_cast<const T*>(a.V) + kv_off;

  float acc[G][E];
#pragma unroll
  for (int h = 0; h < G; ++h)
#pragma unroll
    for (int e = 0; e < E; ++e) acc[h][e] = 0.f;

  // (behind the first rows: answers come in order)
  auto begin = [&]() __attribute__((always_inline)) {
    if constexpr (HOW == kMergeAlone)
      if (threadIdx.x == 0 && !whole_row) tickets = begin_tickets(a.merge_count + (size_t)inst * kTicketStride, a.merge_nonce);
  };
  if (nblk <= 0) begin();

  int p0 = 0, piece = 0;
  if (nblk > 0) do {
    const int nb_p = min(pb, nblk - p0);
    const int ntok = nb_p * a.b;
    // (the staged K tile lives where the waves' output partials go after the last piece)
    qk_logits<T, D, G, kSparseStage, NW>(q_inst, K_inst, a.b, a.log2b, a.t_cur, ntok,
                                         [&](int jb) { return s_idx[p0 + jb]; },
                                         [&](int jb) { return s_phys[p0 + jb]; }, s_p, ld, s_acc);
    // The V rows of this wave's first 16-token group do not depend on the probabilities: they are requested before
    // the softmax pass and arrive while it runs - where the registers allow it.  The pieced forms with g = 4 are at
    // their 128 VGPRs already and would spill (0.201 vs 0.183 ms at cfg2); with g <= 2 they gain 1.5 % at cfg4, and
    // the four-wave form, which has registers to spare, 2 % at cfg3.
    constexpr bool kEarlyV = (PIECED && G <= 2) || !PIECED;
    const int ngroups = (ntok + kGroupTokens - 1) / kGroupTokens;
    uint4 vw[NL];
    auto load_v = [&](int grp) __attribute__((always_inline)) {
      const int tau0 = grp * kGroupTokens + tslot * NL;
#pragma unroll
      for (int i = 0; i < NL; ++i) vw[i] = make_uint4(0, 0, 0, 0);
      if (tau0 < ntok) {
        // Tokens at or beyond t_cur (the tail of the newest block) carry probability 0, but their V rows may hold
        // anything, NaN included, and 0 * NaN is NaN: such a token reads the block's last real row instead.
        const int jb = p0 + (tau0 >> a.log2b), off = tau0 & (a.b - 1);
        const int last = min(a.t_cur - 1 - s_idx[jb] * a.b, a.b - 1);   // >= 0: a listed block starts before t_cur
        const int prow0 = s_phys[jb] * a.b;
#pragma unroll
        for (int i = 0; i < NL; ++i) vw[i] = ld_stream(V_inst + (size_t)(prow0 + min(off + i, last)) * D + dpart * E);
      }
    };
    if (kEarlyV && wave < ngroups) load_v(wave);
    if (p0 == 0) begin();
    __syncthreads();
    softmax_stats<G, NW>(s_p, ld, ntok, a.b, nblk, s_m, s_l, s_bmp + p0, s_alpha);
    if (threadIdx.x < G) s_mpiece[piece * G + threadIdx.x] = s_m[threadIdx.x];
    if (PIECED && piece > 0) {                         // the maximum may have moved: bring acc along
#pragma unroll
      for (int h = 0; h < G; ++h) {
        const float al = s_alpha[h];
#pragma unroll
        for (int e = 0; e < E; ++e) acc[h][e] *= al;
      }
    }

    // Phase 3: acc += p * V.  A lane group takes NL consecutive tokens of a 16-token group (they lie in one
    // block, so one table lookup places them), load instruction i covers the i-th row of each of the TPI lane
    // groups - whole 256-byte rows - and the NL probabilities of a head come in one LDS access.
    static_assert(NL == 2 || NL == 4 || NL == 8, "probabilities are fetched as 8- or 16-byte vectors");
    for (int grp = wave; grp < ngroups; grp += NW) {
      const int tau0 = grp * kGroupTokens + tslot * NL;   // ntok is a multiple of 8 >= NL: all NL tokens or none
      const bool live = tau0 < ntok;
      if (!kEarlyV || grp != wave) load_v(grp);
      float pw[G][NL];
#pragma unroll
      for (int h = 0; h < G; ++h) {
        const float* src = s_p + h * ld + tau0;
        if constexpr (NL == 2) {
          const float2 t = *reinterpret_cast<const float2*>(src);
          pw[h][0] = t.x; pw[h][1] = t.y;
        } else {
#pragma unroll
          for (int c = 0; c < NL / 4; ++c) {
            const float4 t = *reinterpret_cast<const float4*>(src + 4 * c);
            pw[h][4 * c] = t.x; pw[h][4 * c + 1] = t.y; pw[h][4 * c + 2] = t.z; pw[h][4 * c + 3] = t.w;
          }
        }
      }
#pragma unroll
      for (int i = 0; i < NL; ++i) {
        float vf[E];
        unpack16(vw[i], vf, T{});
#pragma unroll
        for (int h = 0; h < G; ++h) {
          const float p = live ? pw[h][i] : 0.f;
#pragma unroll
          for (int e = 0; e < E; ++e) acc[h][e] = fmaf(p, vf[e], acc[h][e]);
        }
      }
    }
    __syncthreads();                                   // the next piece, or the partials, overwrite what was read
    p0 += pb;
    ++piece;
  } while (PIECED && p0 < nblk);

  // Block maxima of earlier pieces are relative to the maximum of their time: bring them to the final one.
  if (PIECED && nblk > pb) {
    for (int pair = threadIdx.x; pair < G * nblk; pair += NT) {
      const int h = pair / nblk, jb = pair - h * nblk;
      s_bmp[pair] *= __expf(s_mpiece[(jb / pb) * G + h] - s_m[h]);
    }
  }

  // Sum the token slots of a wave (lanes that hold the same dims), then the waves through LDS.
#pragma unroll
  for (int h = 0; h < G; ++h)
#pragma unroll
    for (int e = 0; e < E; ++e) {
      float v = acc[h][e];
#pragma unroll
      for (int o = LPT; o < kWave; o <<= 1) v += __shfl_xor(v, o, 64);
      acc[h][e] = v;
    }
  if (tslot == 0) {
#pragma unroll
    for (int h = 0; h < G; ++h)
#pragma unroll
      for (int e = 0; e < E; ++e) s_acc[(wave * G + h) * D + dpart * E + e] = acc[h][e];
  }
  __syncthreads();

  if (a.n_split == 1) {
    for (int o = threadIdx.x; o < G * D; o += NT) {
      float v = 0.f;
#pragma unroll
      for (int w = 0; w < NW; ++w) v += s_acc[w * G * D + o];
      const float L = s_l[o / D];
      a.out[(size_t)inst * G * D + o] = L > 0.f ? v / L : 0.f;      // an empty list gives a zero output
    }
    // Pooled row: column j of a listed block gets the largest block maximum over the heads, the rest zero.
    float* row = a.row + (size_t)inst * a.row_stride;
    for (int j = threadIdx.x; j < a.nb_cap; j += NT) {
      const uint32_t word = s_listed[j >> 5];
      float mx = 0.f;
      if ((word >> (j & 31)) & 1u) {
        const int pos = min(s_rank[j >> 5] + __popc(word & ((1u << (j & 31)) - 1u)), nblk - 1);
#pragma unroll
        for (int h = 0; h < G; ++h) mx = fmaxf(mx, s_bmp[h * nblk + pos] / s_l[h]);
      }
      row[j] = mx;
    }
  } else {
    const size_t ps = (size_t)inst * a.n_split + split;
    for (int o = threadIdx.x; o < G * D; o += NT) {
      float v = 0.f;
#pragma unroll
      for (int w = 0; w < NW; ++w) v += s_acc[w * G * D + o];
      st_shared_out<MERGE>(a.part_acc + ps * G * D + o, v);
    }
    if (threadIdx.x < G) {
      st_shared_out<MERGE>(a.part_ml + (ps * G + threadIdx.x) * 2 + 0, s_m[threadIdx.x]);
      st_shared_out<MERGE>(a.part_ml + (ps * G + threadIdx.x) * 2 + 1, s_l[threadIdx.x]);
    }
    for (int pair = threadIdx.x; pair < G * nblk; pair += NT) {
      const int h = pair / nblk, jb = pair - h * nblk;
      st_shared_out<MERGE>(a.part_bmp + ((size_t)inst * G + h) * a.k + j0 + jb, s_bmp[pair]);
    }
    if constexpr (MERGE)
      if (last_to_finish<HOW == kMergeAlone>(a.merge_count + (size_t)inst * kTicketStride, a.merge_nonce, tickets, a.n_split, reinterpret_cast<int*>(smem) + a.n_split * G)) merge_splits<D, G>(a, inst, cnt, listed, smem);
  }
}


// LDS floats sparse_decode_body needs for a list of up to nblk_cap blocks of b tokens out of nb_cap, worked off
// in pieces of piece_blocks.
template <int D, int G, int NW> inline size_t sparse_lds_floats(int nblk_cap, int piece_blocks, int b, int nb_cap) {
  const int pb = piece_blocks < nblk_cap ? piece_blocks : nblk_cap;
  const int n_pieces = (nblk_cap + pb - 1) / pb;
  return (size_t)G * pb * b + sparse_acc_floats<D, G, NW>() + (size_t)G * nblk_cap + 3 * G + (size_t)n_pieces * G +
         2 * nblk_cap + 2 * (size_t)((nb_cap + 31) / 32);
}

// f(integral_constant<int, 0>) .. f(integral_constant<int, G - 1>)
template <int G, int H = 0, class F> __device__ __forceinline__ void for_heads(F& f) {
  f(std::integral_constant<int, H>{});
  if constexpr (H + 1 < G) for_heads<G, H + 1>(f);
}

// Broadcast of lane LANE of every row of 16 lanes to that row.
template <int LANE> __device__ __forceinline__ float row_bcast(float v) { return dpp_move<0x150 + LANE>(v); }

// v of this lane combined with that of the lane 16 / 32 lanes away, on register swaps.
template <class Op> __device__ __forceinline__ float across_16(float v, Op op) {
  const auto s = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return op(__uint_as_float(s[0]), __uint_as_float(s[1]));
}
template <class Op> __device__ __forceinline__ float across_32(float v, Op op) {
  const auto s = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return op(__uint_as_float(s[0]), __uint_as_float(s[1]));
}

// LDS floats a wave stages 16 K rows in, later its output partial; and those of the query rows, padded like them.
template <int D, int G> constexpr int wave_tile_floats() {
  constexpr int stage = kGroupTokens * (D * 2 + kStageRowPad) / 4;
  return stage > G * D ? stage : G * D;
}
template <int D, int G> constexpr int query_floats() { return G * (D * 2 + kStageRowPad) / 4; }
// The streaming forms keep logits as they come out of the contraction and refer probabilities to whole numbers m, in units of
// log2: with c = log2(e) / sqrt(d) a probability is exp2(fma(logit, c, -m)), whose exponent is rounded once instead of three
// times, and the factors that bring sums from one reference to another are powers of two, which round nothing.
template <int D> struct LogitUnit {
  static_assert(D == 64 || D == 128, "log2(e) / sqrt(d) for the compiled head sizes");
  static constexpr float kC = D == 64 ? 1.4426950408889634 / 8.0 : 1.4426950408889634 / 11.313708498984761;
  static __device__ __forceinline__ float reference(float logit) { return ceilf(logit * kC); }
  static __device__ __forceinline__ float exp_of(float logit, float m) { return exp2_fast(fmaf(logit, kC, -m)); }
};
// How far (in units of log2) a logit may exceed the maximum that the running sums are relative to before they are rescaled:
// 2^11 leaves fp32 sums their relative precision, and after the first pass hardly any pass has to touch the accumulators.
constexpr float kRescaleAt = 11.f;
// Passes of a wave whose sums go into one set of accumulators (32 additions each at d = 128, 16 at d = 64) before these are added
// to a second set: the roundings of a long chain of additions were most of the error of long lists (128 lists of 32790 tokens in four
// splits, relative to 64 bits: 7.3e-7 with 512 in a chain, 3.9e-7 now, 4.7e-7 in 17 splits without a second set).
constexpr int kChainPasses = 8;

// Sparse decode of instance `inst`, split `split`, by one workgroup of four waves, bf16.
// Every wave works off 16-token passes of the list by itself, from K rows to acc += p * V, with running softmax
// statistics (a maximum and a sum per head and per row of 16 lanes, i.e. per token slot), so that no wave waits for
// another between the list at the start and the merge at the end: K rows of the next pass are asked for as soon as the
// present ones are staged, V rows as soon as the present ones are used, and a wave always has some 8 KiB on its way.
// sparse_decode_body goes through phases instead - all logits, softmax, all V - with barriers between them and the
// probabilities of the list in LDS.  With few instances, where nothing else fills the gaps, this form is the faster one
// (decode + merge, both in turn on one card: 1024-token lists, d = 128, g = 4, 8 instances 13.2 -> 10.5 us, 300 instances 37 -> 33 us;
// 640 x 2048 tokens, g = 8, 129 -> 121 us; over 1607 sizes of up to 1000 instances 27 % less).  With 1024 instances and more, g <= 4, the phases win (2048 instances: 177 against 190 us;
// 4096, g = 1: 337 against 373): on scattered blocks a stream that alternates between K and V reaches 5.85 TB/s,
// however many waves have loads on their way, and one that stays in one of the two for a while 6.25.
//
// The g x d by d x 16-token contraction runs on v_mfma_f32_16x16x32_bf16 (A = 16 K rows, B = q^T repeated to 16
// columns, fp32 accumulate).  In the operand layout lane l supplies token l % 16 and, the order of the contraction index
// being free as long as A and B agree, dims (l / 16) d/4 .. + d/4 - 1, eight per K-step.  The result comes back as lane
// (head = l % 16, tokens 4 (l / 16) + v), v = 0..3: a row of 16 lanes holds the logits of four tokens, which are, for
// d = 128, the tokens whose V rows the row reads, and the probability of a head is a DPP broadcast away.
// smem: sparse_stream_lds_floats(...) floats of LDS, 16-byte aligned.
template <int D, int G, int HOW>
__device__ __forceinline__ void sparse_stream_body(const SparseArgs& a, int inst, int split, float* smem) {
  using T = bf16_t;
  using Ge = Geom<T, D, G>;
  constexpr int NW = kAttnWaves;
  constexpr int E = Ge::E, LPT = Ge::LPT, TPI = Ge::TPI, NL = Ge::NL, NT = NW * kWave, KS = D / 32;
  constexpr int TILE = wave_tile_floats<D, G>();
  constexpr int RS = D * 2 + kStageRowPad;               // bytes of a staged K row
  const int lane = threadIdx.x & (kWave - 1);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int dpart = lane % LPT, tslot = lane / LPT;
  const int head = lane & 15, row16 = lane >> 4;         // what this lane's logits are of

  constexpr bool MERGE = HOW != kSplitsOnly;
  int cnt;
  unsigned long long tickets = 0;                        // (asked for behind the first rows: answers come in order)
  if constexpr (HOW == kSelectInside) cnt = select_inside(a, inst, split, smem); else cnt = min(max(a.cnt[inst], 0), a.k);
  const int32_t* list = HOW == kSelectInside ? reinterpret_cast<const int32_t*>(smem + a.sel_at) : a.idx + (size_t)inst * a.k;
  auto listed = [&](int jb) __attribute__((always_inline)) { return min(max(list[jb], 0), a.nb_cur - 1); };
  // With one workgroup per instance the whole list is local; otherwise this split's slice.
  const bool whole_row = a.n_split == 1;
  const int j0 = whole_row ? 0 : min(cnt, split * a.blk_per_split);
  const int j1 = whole_row ? cnt : min(cnt, j0 + a.blk_per_split);
  const int nblk = j1 - j0;
  const int nblk_cap = whole_row ? a.k : a.blk_per_split;
  const int qpb = a.b >> 2;                              // groups of four tokens per block

  float* s_tile = smem + wave * TILE;                    // [waves][TILE] staged K rows, then the wave's sum of p V
  char* s_q = reinterpret_cast<char*>(smem + NW * TILE); // [G] query rows, padded like the K rows
  float* s_qmax = smem + NW * TILE + query_floats<D, G>();          // [G][nblk_cap * qpb] largest logit of four tokens
  float* s_m = s_qmax + G * nblk_cap * qpb;              // [waves][G] maximum, then the factor that brings a wave's sums to the whole
  float* s_l = s_m + NW * G;                             // [waves][G] sum relative to it
  float* s_ml = s_l + NW * G;                            // [G][2] maximum and sum of the workgroup
  int* s_idx = reinterpret_cast<int*>(s_ml + 2 * G);     // [nblk_cap] logical block of each position
  int* s_phys = s_idx + nblk_cap;                        // [nblk_cap] its place in K / V
  // For the pooled row, written whole by the workgroup that has the whole list: one bit per block, is it listed.
  const int nwords = whole_row ? (a.nb_cap + 31) / 32 : 0;
  uint32_t* s_listed = reinterpret_cast<uint32_t*>(s_phys + nblk_cap);   // [nwords]

  if (whole_row) {
    for (int w = threadIdx.x; w < nwords; w += NT) s_listed[w] = 0u;
    __syncthreads();
  }
  if constexpr (MERGE)
    if (!whole_row) clear_row_share(a, inst, split);
  for (int j = threadIdx.x; j < nblk; j += NT) {
    const int blk = listed(j0 + j);
    s_idx[j] = blk;
    s_phys[j] = a.table ? min(max(a.table[(size_t)inst * a.nb_cap + blk], 0), a.n_phys - 1) : blk;
    if (whole_row) atomicOr(&s_listed[blk >> 5], 1u << (blk & 31));
  }
  // The query operand stays in LDS and is read again in every pass, which is what keeps d = 128, g = 4 within 128
  // registers.
  const T* q_inst = static_cast<const T*>(a.q) + (size_t)inst * G * D;
  for (int o = threadIdx.x; o < G * D / 8; o += NT)
    *reinterpret_cast<uint4*>(s_q + (o / (D / 8)) * RS + (o % (D / 8)) * 16) = reinterpret_cast<const uint4*>(q_inst)[o];
  __syncthreads();

  // Contiguous cache: [n_inst][t_cap][d].  Paged cache: one pool [n_phys][b][d] for all instances.
  const size_t kv_off = a.table ? 0 : (size_t)inst * a.t_cap * D;
  const T* K_inst = static_cast<const T*>(a.K) + kv_off;
  const T* V_inst = static_cast<const T*>(a.V) + kv_off;

  using Unit = LogitUnit<D>;
  const int ntok = nblk * a.b, npass = (ntok + kGroupTokens - 1) / kGroupTokens;

  // A pass's 16 tokens are two runs of eight, each inside one block (a block holds at least eight).  K rows: load i
  // brings rows i TPI .. + TPI - 1 of the pass.  V rows: lane group tslot takes tokens tslot NL .. + NL - 1, load i the
  // i-th of every group.
  struct Pass { int row[2], off[2], last[2]; };          // wave-uniform, per run: first row of its block in the cache, its
                                                         // place in the block, last row of the block inside the context
  auto pass_at = [&](int ps) __attribute__((always_inline)) {
    Pass r;
    const int tau = ps * kGroupTokens;
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      if (u == 0 || a.b == 8) {
        const int jb = min((tau + 8 * u) >> a.log2b, nblk - 1);   // (the missing run of an odd list of 8-token blocks is masked)
        const int blk = __builtin_amdgcn_readfirstlane(s_idx[jb]);
        r.row[u] = __builtin_amdgcn_readfirstlane(s_phys[jb]) * a.b;
        r.off[u] = tau & (a.b - 1);
        r.last[u] = min(a.t_cur - 1 - blk * a.b, a.b - 1);
      } else {
        r.row[1] = r.row[0];
        r.off[1] = r.off[0] + 8;
        r.last[1] = r.last[0];
      }
    }
    return r;
  };
  uint4 kw[NL], vw[NL];
  auto load_k = [&](const Pass& r) __attribute__((always_inline)) {
    constexpr int kPerRun = 8 / TPI;                     // loads per run of eight rows; a load is TPI whole rows
#pragma unroll
    for (int i = 0; i < NL; ++i) {
      const int first = r.row[i / kPerRun] + r.off[i / kPerRun] + (i % kPerRun) * TPI;
      kw[i] = ld_stream(K_inst + (size_t)first * D + (uint32_t)lane * E);
    }
  };
  auto load_v = [&](const Pass& r) __attribute__((always_inline)) {
    // Tokens at or beyond t_cur (the tail of the newest block) carry probability 0, but their V rows may hold
    // anything, NaN included, and 0 * NaN is NaN: such a token reads the block's last real row instead.
    const bool upper = tslot * NL >= 8;
    const int row = upper ? r.row[1] : r.row[0], last = upper ? r.last[1] : r.last[0];
    const int at = (upper ? r.off[1] - 8 : r.off[0]) + tslot * NL;
#pragma unroll
    for (int i = 0; i < NL; ++i) vw[i] = ld_stream(V_inst + (size_t)(row + min(at + i, last)) * D + dpart * E);
  };

  Pass next;                                             // the pass whose rows are on their way
  if (wave < npass) {                                    // (before the query: nothing else is on its way yet)
    next = pass_at(wave);
    load_k(next);
    load_v(next);
  }
  if constexpr (HOW == kMergeAlone)
    if (threadIdx.x == 0 && !whole_row) tickets = begin_tickets(a.merge_count + (size_t)inst * kTicketStride, a.merge_nonce);

  float m = -INFINITY, l = 0.f;                          // running statistics of this lane's head and row of 16 lanes
  float acc[G][E];
#pragma unroll
  for (int h = 0; h < G; ++h)
#pragma unroll
    for (int e = 0; e < E; ++e) acc[h][e] = 0.f;

  // MORE: the wave has another pass after this one, whose rows are asked for on the way.  (Two copies of the code, so that
  // the registers of a row have one source on the way round the loop and no copy has to wait for the load.)
  auto pass = [&](int ps, auto more_tag) __attribute__((always_inline)) {
    constexpr bool MORE = decltype(more_tag)::value;
    const int tau0 = ps * kGroupTokens;
    // Tokens of this pass that exist and lie inside the context: bit t of `live` (wave-uniform).
    uint32_t live;
    {
      const int n0 = min(max(next.last[0] - next.off[0] + 1, 0), 8);
      const int n1 = tau0 + 8 < ntok ? min(max(next.last[1] - next.off[1] + 1, 0), 8) : 0;
      live = ((1u << n0) - 1u) | (((1u << n1) - 1u) << 8);
    }
    if constexpr (MORE) next = pass_at(ps + NW);
    char* stage = reinterpret_cast<char*>(s_tile);
#pragma unroll
    for (int i = 0; i < NL; ++i)
      *reinterpret_cast<uint4*>(stage + (i * TPI + lane / LPT) * RS + (lane % LPT) * 16) = kw[i];
    asm volatile("" ::: "memory");                     // a wave's LDS accesses stay in order; so must the compiler
    if constexpr (MORE) load_k(next);
    float4v lg = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int s = 0; s < KS; ++s) {
      const uint4 w = *reinterpret_cast<const uint4*>(stage + head * RS + (row16 * (D / 4) + s * 8) * 2);
      // (columns of B beyond the g heads repeat them: their logits are not used)
      const uint4 wq = *reinterpret_cast<const uint4*>(s_q + (head & (G - 1)) * RS + (row16 * (D / 4) + s * 8) * 2);
      lg = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, w), __builtin_bit_cast(bf16x8, wq), lg, 0, 0, 0);
    }
    asm volatile("" ::: "memory");                     // the next pass overwrites the tile read above
    float p[4];
#pragma unroll
    for (int v = 0; v < 4; ++v) p[v] = lg[v];
    if (live != 0xffffu) {
#pragma unroll
      for (int v = 0; v < 4; ++v) p[v] = ((live >> (4 * row16 + v)) & 1u) ? p[v] : -INFINITY;
    }
    const float mx = fmaxf(fmaxf(p[0], p[1]), fmaxf(p[2], p[3]));
    if (head < G && tau0 + 4 * row16 < ntok) s_qmax[head * (nblk * qpb) + ps * 4 + row16] = mx;
    const bool above = head < G && mx * Unit::kC > m + kRescaleAt;
    if (__any(above)) {
      const float m_new = above ? Unit::reference(mx) : m;
      const float al = above ? exp2_fast(m - m_new) : 1.f;   // (0 for the first maximum)
      m = m_new;
      l *= al;
      auto rescale = [&](auto hc) __attribute__((always_inline)) {
        constexpr int h = decltype(hc)::value;
        const float f = row_bcast<h>(al);
#pragma unroll
        for (int e = 0; e < E; ++e) acc[h][e] *= f;
      };
      for_heads<G>(rescale);
    }
    const float m_ref = m == -INFINITY ? 0.f : m;          // (nothing but masked tokens so far)
#pragma unroll
    for (int v = 0; v < 4; ++v) p[v] = Unit::exp_of(p[v], m_ref);
    l += (p[0] + p[1]) + (p[2] + p[3]);
    // acc += p V: token i of this lane's group is, of the row's four tokens, i (d = 128) or 2 (tslot % 2) + i (d = 64)
#pragma unroll
    for (int i = 0; i < NL; ++i) {
      float vf[E];
      unpack16(vw[i], vf, T{});
      auto add = [&](auto hc) __attribute__((always_inline)) {
        constexpr int h = decltype(hc)::value;
        float ph = row_bcast<h>(p[i]);
        if constexpr (NL == 2) {                       // (both broadcasts by every lane: the source must be active)
          const float odd = row_bcast<h>(p[2 + i]);
          ph = (tslot & 1) ? odd : ph;
        }
#pragma unroll
        for (int e = 0; e < E; ++e) acc[h][e] = fmaf(ph, vf[e], acc[h][e]);
      };
      for_heads<G>(add);
    }
    if constexpr (MORE) load_v(next);
  };
  // Second set of accumulators: the token slots added up, relative to one maximum per head (m_sum), each lane holding its
  // share of the dims: dims dpart E + first .. + NS - 1.
  constexpr int NS = E / TPI;
  const int first = ((lane >> 5) & 1) * 4 + ((lane >> 4) & 1) * 2 + (TPI == 8 ? (lane >> 3) & 1 : 0);
  float m_sum = -INFINITY, l_sum = 0.f, sum[G][NS];
#pragma unroll
  for (int h = 0; h < G; ++h)
#pragma unroll
    for (int j = 0; j < NS; ++j) sum[h][j] = 0.f;
  const auto larger = [](float x, float y) { return fmaxf(x, y); };
  const auto plus = [](float x, float y) { return x + y; };
  auto fold = [&]() __attribute__((always_inline)) {
    const float mw = across_32(across_16(m, larger), larger);
    const float f_acc = m == -INFINITY ? 0.f : exp2_fast(m - mw), f_sum = m_sum == -INFINITY ? 0.f : exp2_fast(m_sum - mw);
    m = m_sum = mw;
    l_sum = fmaf(l_sum, f_sum, across_32(across_16(l * f_acc, plus), plus));
    l = 0.f;
    auto head_share = [&](auto hc) __attribute__((always_inline)) {
      constexpr int h = decltype(hc)::value;
      const float f = row_bcast<h>(f_acc), fs = row_bcast<h>(f_sum);
      float x[E];
#pragma unroll
      for (int e = 0; e < E; ++e) { x[e] = acc[h][e] * f; acc[h][e] = 0.f; }
      // Lanes 32 and up take elements 4..7, lanes below 0..3; odd rows of 16 the upper two of these, and so on.
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const auto s = __builtin_amdgcn_permlane32_swap(__float_as_uint(x[e]), __float_as_uint(x[e + 4]), false, false);
        x[e] = __uint_as_float(s[0]) + __uint_as_float(s[1]);
      }
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        const auto s = __builtin_amdgcn_permlane16_swap(__float_as_uint(x[e]), __float_as_uint(x[e + 2]), false, false);
        x[e] = __uint_as_float(s[0]) + __uint_as_float(s[1]);
      }
      if constexpr (TPI == 8) {
        const bool upper = (lane >> 3) & 1;
        x[0] = (upper ? x[1] : x[0]) + dpp_move<0x128>(upper ? x[0] : x[1]);     // row_ror:8
      }
#pragma unroll
      for (int j = 0; j < NS; ++j) sum[h][j] = fmaf(sum[h][j], fs, x[j]);
    };
    for_heads<G>(head_share);
  };
  int ps = wave, chain = 0;
#pragma unroll 1
  for (; ps + NW < npass; ps += NW) {
    pass(ps, std::true_type{});
    if (++chain == kChainPasses) { fold(); chain = 0; }
  }
  if (ps < npass) pass(ps, std::false_type{});
  fold();

  if (lane < G) { s_m[wave * G + lane] = m; s_l[wave * G + lane] = l_sum; }
#pragma unroll
  for (int h = 0; h < G; ++h)
#pragma unroll
    for (int j = 0; j < NS; ++j) s_tile[h * D + dpart * E + first + j] = sum[h][j];
  __syncthreads();

  // The waves: one maximum and sum per head, and the factor for each wave's share.
  if (threadIdx.x < G) {
    const int h = threadIdx.x;
    float M = -INFINITY;
#pragma unroll
    for (int w = 0; w < NW; ++w) M = fmaxf(M, s_m[w * G + h]);
    float L = 0.f;
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      const float mw = s_m[w * G + h], f = mw == -INFINITY ? 0.f : exp2_fast(mw - M);
      L += s_l[w * G + h] * f;
      s_m[w * G + h] = f;
    }
    s_ml[2 * h] = M;
    s_ml[2 * h + 1] = L;
  }
  __syncthreads();

  auto block_max = [&](int h, int jb) __attribute__((always_inline)) {
    const float* qm = s_qmax + h * (nblk * qpb) + jb * qpb;
    float mx = qm[0];
#pragma unroll 1
    for (int i = 1; i < qpb; ++i) mx = fmaxf(mx, qm[i]);
    return Unit::exp_of(mx, s_ml[2 * h]);                // (a listed block has a token inside the context: M is finite)
  };
  if (whole_row) {
    for (int o = threadIdx.x; o < G * D; o += NT) {
      const int h = o / D;
      float v = 0.f;
#pragma unroll
      for (int w = 0; w < NW; ++w) v = fmaf(smem[w * TILE + o], s_m[w * G + h], v);
      const float L = s_ml[2 * h + 1];
      a.out[(size_t)inst * G * D + o] = L > 0.f ? v / L : 0.f;      // an empty list gives a zero output
    }
    // Pooled row: a listed block's column gets the largest block maximum over the heads, the rest zero.  The values go
    // where the list says, so entries that come twice (after clamping) or out of order have theirs too, as in the merge of splits.
    float* row = a.row + (size_t)inst * a.row_stride;
    for (int j = threadIdx.x; j < a.nb_cap; j += NT)
      if (!((s_listed[j >> 5] >> (j & 31)) & 1u)) row[j] = 0.f;
    for (int jb = threadIdx.x; jb < nblk; jb += NT) {
      float mx = 0.f;
#pragma unroll
      for (int h = 0; h < G; ++h) mx = fmaxf(mx, block_max(h, jb) / s_ml[2 * h + 1]);
      row[s_idx[jb]] = mx;                               // (a block listed twice: either of two equal values)
    }
  } else {
    const size_t ps = (size_t)(MERGE ? inst : inst - a.part_first) * a.n_split + split;
    for (int o = threadIdx.x; o < G * D; o += NT) {
      const int h = o / D;
      float v = 0.f;
#pragma unroll
      for (int w = 0; w < NW; ++w) v = fmaf(smem[w * TILE + o], s_m[w * G + h], v);
      st_shared_out<MERGE>(a.part_acc + ps * G * D + o, v);
    }
    if (threadIdx.x < 2 * G) st_shared_out<MERGE>(a.part_ml + ps * G * 2 + threadIdx.x, s_ml[threadIdx.x]);
    for (int pair = threadIdx.x; pair < G * nblk; pair += NT) {
      const int h = pair / nblk, jb = pair - h * nblk;
      st_shared_out<MERGE>(a.part_bmp + ((size_t)inst * G + h) * a.k + j0 + jb, block_max(h, jb));
    }
    if constexpr (MERGE)
      if (last_to_finish<HOW == kMergeAlone>(a.merge_count + (size_t)inst * kTicketStride, a.merge_nonce, tickets, a.n_split, reinterpret_cast<int*>(smem) + a.n_split * G)) merge_splits<D, G>(a, inst, cnt, listed, smem);
  }
}

// LDS floats sparse_stream_body needs for a list of up to nblk_cap blocks of b tokens; nb_cap: blocks of the pooled row
// where the workgroup writes it, else 0.
template <int D, int G> inline size_t sparse_stream_lds_floats(int nblk_cap, int b, int nb_cap) {
  const size_t words = (size_t)((nb_cap + 31) / 32);
  return (size_t)kAttnWaves * wave_tile_floats<D, G>() + query_floats<D, G>() + (size_t)G * nblk_cap * (b / 4) +
         2 * kAttnWaves * G + 2 * G + 2 * nblk_cap + words;
}

}  // namespace
}  // namespace ap
