// Top-K block selection (Algorithm 1 step 5) with forced sink / local blocks (Sec. 4.1).
//
// One workgroup per instance.  Scores are mapped to order-preserving 32-bit keys.  With few free places (launch_select) the few keys
// that reach a lower bound of the last one are ranked against each other (select_by_bound).  With more, or where too many keys
// reach the bound (scores that all but coincide), a 4-pass
// radix select (8 bits per pass, histogram in LDS) finds the key T of the k_mid-th largest score
// and how many scores equal to T are still needed.  A final ordered sweep keeps every block with
// key > T and the first `need` blocks with key == T, compacting in index order, so the output is
// ascending and equal scores go to the lower index.  Integer work only: the result is exact.
// When the candidates fit (up to 32 per thread) their keys are fetched once into registers, so the five
// passes do not each wait on memory; longer rows are re-read from cache in every pass.
#pragma once

#include "ap_internal.h"

namespace ap {
namespace {

constexpr int kSelThreads = 256;           // workgroup size of the common variant
constexpr int kSelThreadsWide = 1024;      // few instances, long rows: more threads per instance
constexpr int kSelBins = 256;              // radix of one pass; the first kSelBins threads own one bin each
constexpr int kSelRanked = 256;            // select_by_bound: most keys it ranks against each other
constexpr int kSelMaxMid = 128;            // ... and most free places it fills
constexpr int kSelFewMid = 96;             // places up to which it wins whatever the number of candidates (launch_select)
template <int NT> constexpr int sel_scratch_words() {
  constexpr int radix = kSelBins + 3 * (NT / kWave) + 8, bound = 2 * (kSelRanked + 16) + 8 * kWave + kSelMaxMid + 18;
  return radix > bound ? radix : bound;
}

__device__ __forceinline__ uint32_t score_key(float x) {
  uint32_t u = __float_as_uint(x);
  if (u == 0x80000000u) u = 0u;                         // -0 ranks with +0
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);    // larger score <=> larger key
}

// Adds one to hist[bin] for every lane with `active`.  Predicted scores of neighbouring blocks are close,
// so most lanes of a wave share a bin and per-lane LDS atomics would serialise on it: the two most common
// leading bins are counted with a ballot and added once per wave, the rest fall back to single adds.
__device__ __forceinline__ void hist_add(uint32_t* hist, uint32_t bin, bool active) {
#pragma unroll
  for (int round = 0; round < 2; ++round) {
    if (active) {                                       // (the lanes still to be counted are the ones executing here)
      const uint32_t b0 = __builtin_amdgcn_readfirstlane(bin);          // bin of the first of them
      const bool same = bin == b0;
      const unsigned long long m = __ballot(same);
      const uint32_t before = __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
      if (same && before == 0) atomicAdd(&hist[b0], (uint32_t)__popcll(m));
      if (same) active = false;
    }
  }
  if (active) atomicAdd(&hist[bin], 1u);
}

// Inclusive prefix sum over the 64 lanes with DPP moves (shifts within the rows of 16 lanes, then the last lane of
// row 0 / 2 added to row 1 / 3 and the last lane of row 1 to rows 2 and 3): register moves, no trip through the LDS
// permute path.  Every lane must be active.
template <int CTRL, int ROW_MASK> __device__ __forceinline__ uint32_t dpp_u32(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, ROW_MASK, 0xF, true);
}
__device__ __forceinline__ uint32_t wave_incl_scan(uint32_t v) {
  v += dpp_u32<0x111, 0xF>(v);                          // row_shr:1 (zero shifted in at the start of a row)
  v += dpp_u32<0x112, 0xF>(v);                          // row_shr:2
  v += dpp_u32<0x114, 0xF>(v);                          // row_shr:4
  v += dpp_u32<0x118, 0xF>(v);                          // row_shr:8
  v += dpp_u32<0x142, 0xA>(v);                          // row_bcast:15 into rows 1 and 3
  v += dpp_u32<0x143, 0xC>(v);                          // row_bcast:31 into rows 2 and 3
  return v;
}

// The k_mid largest of the keys that the threads hold (0 where a thread has none; ties to the lower block), written to out in
// ascending order of blocks - or false, and nothing written, if more than kSelRanked keys would have to be ranked.  Then T and need say, where
// need is not 0, that all keys above T are wanted and the first `need` equal to T.
//   A lower bound of the k_mid-th largest key is the k_mid-th largest of the maxima of 64 GR groups of keys, GR of them in
//   every lane: each wave finds one for itself by trying the key's bits from the top, until hardly more than k_mid maxima reach
//   it.  With the large keys spread over the groups few more keys than that do (74 of 2041 for k_mid = 56 and 128
//   groups); these are ranked by counting, for each, how many come before it, and the same again by block.
// Where the bound lets too many keys through because they coincide with it, the radix passes are left out (2048 instances of 2041 candidates, all
// scores equal: 13.6 us by the radix select alone, 21.9 with a bound in front of it, 14.3 so; eight different scores 18.2, 23.8, 21.9).
// Three barriers and no histogram, where the radix select has three a pass and an LDS atomic per key (the scores of a decode run, us,
// radix select -> this: 2048 instances of 2041 candidates 14.9 -> 8.1, 4096 25.6 -> 13.6, 128 of 8186 12.6 -> 6.8, 8 of
// 2041 5.8 -> 4.0, one of 126 3.5 -> 2.6).  What is left is the chain: scores, 15-20 tried bits, one LDS atomic, two rounds of counting.
template <int KPT, int NT, int GR>
__device__ __forceinline__ bool select_by_bound(const uint32_t (&keys)[KPT], int first, uint32_t k_mid,
                                                int32_t* __restrict__ out, uint32_t* s_mem, uint32_t& T, uint32_t& need) {
  constexpr int kWaves = NT / kWave;
  constexpr int kHolders = GR * kWave / kWaves;         // lanes of a wave that hold the maximum of a group
  static_assert(kHolders == 64 || kHolders == 32 || kHolders == 16 || kHolders == 8, "groups are lanes, or lanes 32, 16, 8 apart");
  // (what is read in fours reads past the end of a list into zeros, which count as nothing)
  unsigned long long* s_cand = reinterpret_cast<unsigned long long*>(s_mem);   // [kSelRanked + 16] key | ~block: larger comes first
  uint32_t* s_max = s_mem + 2 * (kSelRanked + 16);      // [64 GR]
  uint32_t* s_sel = s_max + 8 * kWave;                  // [k_mid] ~block by rank
  uint32_t* s_count = s_sel + kSelMaxMid + 16;
  const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;

  uint32_t gm = keys[0];
#pragma unroll
  for (int i = 1; i < KPT; ++i) gm = max(gm, keys[i]);
  if constexpr (kHolders <= 32) {
    const auto s = __builtin_amdgcn_permlane32_swap(gm, gm, false, false);
    gm = max(s[0], s[1]);
  }
  if constexpr (kHolders <= 16) {
    const auto s = __builtin_amdgcn_permlane16_swap(gm, gm, false, false);
    gm = max(s[0], s[1]);
  }
  if constexpr (kHolders <= 8) gm = max(gm, dpp_u32<0x128, 0xF>(gm));          // row_ror:8
  if (lane < kHolders) s_max[wave * kHolders + lane] = gm;
  for (int i = tid; i < kSelRanked + 16; i += NT) s_cand[i] = 0ull;
  for (int i = tid; i < kSelMaxMid + 18; i += NT) s_sel[i] = 0u;               // (and the counts)
  __syncthreads();
  uint32_t g[GR];
#pragma unroll
  for (int r = 0; r < GR; ++r) g[r] = s_max[r * kWave + lane];
  T = 0;
  const uint32_t enough = k_mid + (k_mid >> 3);
#pragma unroll 1
  for (uint32_t bit = 0x80000000u; bit != 0u; bit >>= 1) {
    const uint32_t t = T | bit;
    uint32_t c = 0;
#pragma unroll
    for (int r = 0; r < GR; ++r) c += (uint32_t)__popcll(__ballot(g[r] >= t));
    if (c >= k_mid) {
      T = t;
      if (c <= enough) break;
    }
  }
  T = max(T, 1u);                                       // (a thread without a key holds 0)

  uint32_t mine = 0;                                    // keys of this wave that reach the bound
#pragma unroll
  for (int i = 0; i < KPT; ++i) mine += (uint32_t)__popcll(__ballot(keys[i] >= T));
  uint32_t at = 0;
  if (mine != 0u) {
    if (lane == 0) at = atomicAdd(s_count, mine);
    at = __builtin_amdgcn_readfirstlane(at);
    if (at + mine <= (uint32_t)kSelRanked) {
#pragma unroll
      for (int i = 0; i < KPT; ++i) {
        const bool take = keys[i] >= T;
        const unsigned long long m = __ballot(take);
        if (take) s_cand[__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, at))] =
            ((unsigned long long)keys[i] << 32) | (uint32_t)~(first + i * NT);
        at += (uint32_t)__popcll(m);
      }
    }
  }
  __syncthreads();
  const uint32_t n = *s_count;
  need = 0;
  if (n < k_mid) return false;                          // (the same for every thread; scores that are NaN)
  if (n > (uint32_t)kSelRanked) {
    // Scores of which many coincide - blocks without a history all have the same - make the bound the last wanted key itself: fewer than
    // k_mid keys are larger.
    uint32_t above = 0;
#pragma unroll
    for (int i = 0; i < KPT; ++i) above += (uint32_t)__popcll(__ballot(keys[i] > T));
    if (lane == 0 && above != 0u) atomicAdd(s_count + 1, above);
    __syncthreads();
    above = s_count[1];
    if (above < k_mid) need = k_mid - above;
    __syncthreads();                                    // (the caller uses this LDS)
    return false;
  }
  // Four lanes a key, each counting a quarter of the others.
  const uint32_t part = tid & 3;
#pragma unroll 1
  for (uint32_t c = tid >> 2; c < n; c += NT / 4) {
    const unsigned long long x = s_cand[c];
    uint32_t rank = 0;
#pragma unroll 1
    for (uint32_t o = 0; o < n; o += 16) {
#pragma unroll
      for (int i = 0; i < 4; ++i) rank += s_cand[o + 4 * i + part] > x ? 1u : 0u;
    }
    rank += dpp_u32<0xB1, 0xF>(rank);                   // quad_perm [1,0,3,2]
    rank += dpp_u32<0x4E, 0xF>(rank);                   // quad_perm [2,3,0,1]
    if (part == 0 && rank < k_mid) s_sel[rank] = (uint32_t)x;
  }
  __syncthreads();
#pragma unroll 1
  for (uint32_t c = tid >> 2; c < k_mid; c += NT / 4) {
    const uint32_t x = s_sel[c];
    uint32_t before = 0;
#pragma unroll 1
    for (uint32_t o = 0; o < k_mid; o += 16) {
#pragma unroll
      for (int i = 0; i < 4; ++i) before += s_sel[o + 4 * i + part] > x ? 1u : 0u;
    }
    before += dpp_u32<0xB1, 0xF>(before);
    before += dpp_u32<0x4E, 0xF>(before);
    if (part == 0) out[before] = (int32_t)~x;
  }
  return true;
}

// Selection for one instance by one workgroup of NT threads (a multiple of kSelBins).
//   p        the instance's scores (nb_cur valid entries)
//   out      the instance's k index slots, cnt_out its count
//   s_mem    sel_scratch_words<NT>() words of LDS, free for this call (the caller synchronises before)
// KPT: keys per thread held in registers; 0 = re-read the scores in every pass.  GR > 0: by a bound first, k_mid in 1 .. 32 GR.
template <int KPT, int NT, int GR>
__device__ __forceinline__ void select_topk_body(const float* __restrict__ p, int nb_cur, int k, int n_sink, int n_local,
                                        int32_t* __restrict__ out, int32_t* __restrict__ cnt_out, uint32_t* s_mem) {
  constexpr int kSelThreads = NT, kSelWaves = NT / kWave;
  uint32_t* s_hist = s_mem;                     // [kSelBins]
  uint32_t* s_wsum = s_mem + kSelBins;          // [kSelWaves]
  uint32_t* s_wgt = s_wsum + kSelWaves;         // [kSelWaves]
  uint32_t* s_weq = s_wgt + kSelWaves;          // [kSelWaves]
  uint32_t* s_found = s_mem + kSelBins + 3 * kSelWaves; // [4 passes][bin, keys above it]: a slot per pass, so no
                                                        // barrier is needed before the next pass may write
  const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;

  if (nb_cur <= k) {                                    // everything fits the budget
    for (int j = tid; j < nb_cur; j += kSelThreads) out[j] = j;
    if (tid == 0) *cnt_out = nb_cur;
    return;
  }
  const int lo = n_sink, hi = nb_cur - n_local;         // candidates [lo, hi), hi - lo > k_mid
  const int k_mid = k - n_sink - n_local;

  // Candidate i of thread tid is block lo + i * kSelThreads + tid; past the end the key is a sentinel that
  // no pass counts (valid is false).
  constexpr int NK = KPT > 0 ? KPT : 1;
  uint32_t keys[NK];
  if constexpr (KPT > 0) {
#pragma unroll
    for (int i = 0; i < KPT; ++i) {
      const int j = lo + i * kSelThreads + tid;
      keys[i] = score_key(p[min(j, hi - 1)]);
    }
  }
  auto forced = [&]() __attribute__((always_inline)) {
    for (int j = tid; j < n_sink; j += kSelThreads) out[j] = j;
    for (int j = tid; j < n_local; j += kSelThreads) out[k - n_local + j] = nb_cur - n_local + j;
    if (tid == 0) *cnt_out = k;
  };
  uint32_t prefix = 0;                                  // high bits of T found so far
  uint32_t need = 0;                                    // still to take among keys matching prefix
  if constexpr (GR > 0) {
    uint32_t own[NK];
#pragma unroll
    for (int i = 0; i < NK; ++i) own[i] = lo + i * NT + tid < hi ? keys[i] : 0u;
    if (select_by_bound<NK, NT, GR>(own, lo + tid, (uint32_t)k_mid, out + n_sink, s_mem, prefix, need)) { forced(); return; }
  }
  auto key_at = [&](int i, int j) __attribute__((always_inline)) -> uint32_t {
    if constexpr (KPT > 0) return keys[i]; else return score_key(p[min(j, hi - 1)]);
  };
  const int n_iter = KPT > 0 ? KPT : (hi - lo + kSelThreads - 1) / kSelThreads;

  if (need == 0u && k_mid > 0) {
    prefix = 0;
    need = (uint32_t)k_mid;
    if (tid < kSelBins) s_hist[tid] = 0;
    __syncthreads();
    for (int shift = 24, pass = 0; shift >= 0; shift -= 8, ++pass) {
#pragma unroll NK
      for (int i = 0; i < n_iter; ++i) {                   // uniform trip count: ballots need every lane
        const int j = lo + i * kSelThreads + tid;
        const uint32_t key = key_at(i, j);
        const bool match = j < hi && ((shift == 24) || ((key >> (shift + 8)) == prefix));
        hist_add(s_hist, (key >> shift) & 255u, match);
      }
      __syncthreads();
      // Suffix sums over bins: thread r < kSelBins handles bin 255 - r, inclusive scan in that order
      // (whole waves take or skip these branches).
      uint32_t c = 0, incl = 0;
      if (tid < kSelBins) {
        c = s_hist[kSelBins - 1 - tid];
        s_hist[kSelBins - 1 - tid] = 0;                 // for the next pass, whose adds come two barriers later
        incl = wave_incl_scan(c);
        if (lane == kWave - 1) s_wsum[wave] = incl;
      }
      __syncthreads();
      if (tid < kSelBins) {
        uint32_t base = 0;
        for (int w = 0; w < wave; ++w) base += s_wsum[w];
        incl += base;                                   // keys in bins >= 255 - tid
        const uint32_t excl = incl - c;                 // keys in bins >  255 - tid
        if (excl < need && need <= incl) { s_found[2 * pass] = kSelBins - 1 - tid; s_found[2 * pass + 1] = excl; }
      }
      __syncthreads();
      prefix = (prefix << 8) | s_found[2 * pass];
      need -= s_found[2 * pass + 1];
    }
  }
  const uint32_t T = prefix;

  // Ordered sweep in chunks of one workgroup width.
  uint32_t taken = 0;                                   // selected so far (all threads agree)
  uint32_t eq_seen = 0;                                 // keys == T seen so far
#pragma unroll NK
  for (int i = 0; i < n_iter; ++i) {
    if (k_mid <= 0) break;
    const int j = lo + i * kSelThreads + tid;
    bool gt = false, eq = false;
    if (j < hi) {
      const uint32_t key = key_at(i, j);
      gt = key > T;
      eq = key == T;
    }
    const unsigned long long bgt = __ballot(gt), beq = __ballot(eq);
    const unsigned long long below = (lane == 0) ? 0ull : (~0ull >> (kWave - lane));
    if (lane == 0) { s_wgt[wave] = __popcll(bgt); s_weq[wave] = __popcll(beq); }
    __syncthreads();
    uint32_t gt_before = __popcll(bgt & below), eq_before = __popcll(beq & below);
    uint32_t gt_total = 0, eq_total = 0;
    for (int w = 0; w < kSelWaves; ++w) {
      if (w < wave) { gt_before += s_wgt[w]; eq_before += s_weq[w]; }
      gt_total += s_wgt[w];
      eq_total += s_weq[w];
    }
    // equal keys taken before this lane within the chunk: those whose global rank < need
    const uint32_t eq_rank = eq_seen + eq_before;
    const uint32_t eq_taken_before = min(eq_rank, need) - min(eq_seen, need);
    const bool take = gt || (eq && eq_rank < need);
    if (take) out[n_sink + taken + gt_before + eq_taken_before] = j;
    taken += gt_total + (min(eq_seen + eq_total, need) - min(eq_seen, need));
    eq_seen += eq_total;
    __syncthreads();
  }
  forced();
}

}  // namespace
}  // namespace ap
