// Top-K block selection kernel: one workgroup per instance around select_topk_body (select_body.h).
#include "select_body.h"

namespace ap {
namespace {

template <int KPT, int NT, int GR>
__global__ __launch_bounds__(NT) void select_topk_kernel(const float* __restrict__ pred, int nb_cap, int nb_cur, int k,
                                                         int n_sink, int n_local, int inst0,
                                                         int32_t* __restrict__ idx, int32_t* __restrict__ cnt) {
  __shared__ __align__(16) uint32_t s_mem[sel_scratch_words<NT>()];
  const int inst = inst0 + blockIdx.x;
  select_topk_body<KPT, NT, GR>(pred + (size_t)inst * nb_cap, nb_cur, k, n_sink, n_local, idx + (size_t)inst * k,
                            cnt + inst, s_mem);
}

// A selection made for nb_prev blocks, carried over to nb_cur >= nb_prev blocks without new scores: the picks
// below the local window stay (ascending order is kept by an ordered compaction), the blocks of the old local
// window are dropped unless they are sink blocks, at most k - n_local entries survive, and the last n_local
// blocks of the current context are appended.  One workgroup per instance; smem: k ints.
__global__ __launch_bounds__(kSelThreads) void refresh_selection_kernel(int nb_prev, int nb_cur, int k, int n_sink,
                                                                        int n_local, int32_t* __restrict__ idx,
                                                                        int32_t* __restrict__ cnt) {
  extern __shared__ int s_in[];
  constexpr int kSelWaves = kSelThreads / kWave;
  __shared__ int s_wsum[kSelWaves];
  const int inst = blockIdx.x, tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
  int32_t* out = idx + (size_t)inst * k;
  if (nb_cur <= k) {
    for (int j = tid; j < nb_cur; j += kSelThreads) out[j] = j;
    if (tid == 0) cnt[inst] = nb_cur;
    return;
  }
  const int c = min(max(cnt[inst], 0), k);
  for (int p = tid; p < c; p += kSelThreads) s_in[p] = out[p];
  __syncthreads();
  const int hi = nb_cur - n_local, cap = k - n_local;
  const int old_lo = nb_prev > k ? nb_prev - n_local : nb_prev;      // old local window [old_lo, nb_prev)
  int taken = 0;
  for (int p0 = 0; p0 < c; p0 += kSelThreads) {
    const int p = p0 + tid;
    bool keep = false;
    int j = 0;
    if (p < c) {
      j = s_in[p];
      keep = j >= 0 && j < hi && (j < n_sink || j < old_lo || j >= nb_prev);
    }
    const unsigned long long m = __ballot(keep);
    const int before = __popcll(m & ((1ull << lane) - 1ull));
    if (lane == 0) s_wsum[wave] = __popcll(m);
    __syncthreads();
    int base = 0, total = 0;
    for (int w = 0; w < kSelWaves; ++w) {
      if (w < wave) base += s_wsum[w];
      total += s_wsum[w];
    }
    const int pos = taken + base + before;
    if (keep && pos < cap) out[pos] = j;
    taken += total;
    __syncthreads();
  }
  const int m = min(taken, cap);
  for (int j = tid; j < n_local; j += kSelThreads) out[m + j] = hi + j;
  if (tid == 0) cnt[inst] = m + n_local;
}

}  // namespace

hipError_t launch_refresh_selection(const Shape& s, int nb_prev, int nb_cur, int32_t* idx, int32_t* cnt,
                                    hipStream_t st) {
  refresh_selection_kernel<<<dim3(s.n_inst), kSelThreads, sizeof(int) * s.k, st>>>(nb_prev, nb_cur, s.k, s.n_sink,
                                                                                 s.n_local, idx, cnt);
  return hipGetLastError();
}

hipError_t launch_select(const Shape& s, int inst0, int ninst, const float* pred, int nb_cur, int32_t* idx,
                         int32_t* cnt, hipStream_t st) {
  const int n_mid = nb_cur - s.n_sink - s.n_local, k_mid = s.k - s.n_sink - s.n_local;
  const dim3 grid(ninst);
#define AP_SELECT(KPT, NT, GR) \
  select_topk_kernel<KPT, NT, GR><<<grid, NT, 0, st>>>(pred, s.nb_cap, nb_cur, s.k, s.n_sink, s.n_local, inst0, idx, cnt)
  // By a bound, where its groups are at least twice the free places and the keys fit the registers: 128 groups up to 64 places (2048
  // instances of 2041 candidates, 56 places: 8.1 us, 8.7 with 256 groups), 256 up to 96, and to 128 where the radix select has long rows to
  // go through: what is ranked grows with the square of the places.  (By a bound / radix select alone, us, 96 places: 8 instances x 700 candidates
  // 5.6 / 6.4, 2048 x 700 10.9 / 11.2; 126 places: 8 x 160 6.6 / 5.9, 8 x 1300 6.4 / 6.8, 640 x 2050 10.5 / 9.8, x 4000 12.7 / 16.5, 2048 x 700
  // 15.0 / 11.1, x 4000 24.1 / 29.2.)  Threads: as many as leave the launch
  // one round of workgroups and every thread some eight keys (us at 256 / 512 / 1024 threads: 8 instances x 2041 4.4 / 4.0 / 4.3,
  // 128 x 8186 10.8 / 7.3 / 6.8, 640 x 3742 6.5 / 6.4 / 11.0, 2048 x 2041 8.1 / 10.4 / 17.6).
#define AP_SELECT_BOUND(KPT, NT) \
  if (n_mid <= KPT * NT) { \
    if (k_mid <= 64) AP_SELECT(KPT, NT, 2); else AP_SELECT(KPT, NT, 4); \
    return hipGetLastError(); \
  }
  if (k_mid >= 1 && (k_mid <= kSelFewMid || (k_mid <= kSelMaxMid && n_mid > (ninst <= 512 ? 1024 : 3072)))) {
    if (ninst > 1024 || n_mid <= 1024 || (ninst > 512 && n_mid <= 4096)) {
      AP_SELECT_BOUND(4, 256) AP_SELECT_BOUND(8, 256) AP_SELECT_BOUND(9, 256) AP_SELECT_BOUND(12, 256)
      AP_SELECT_BOUND(16, 256) AP_SELECT_BOUND(24, 256) AP_SELECT_BOUND(32, 256)
    } else if (ninst > 512 || n_mid <= 4096) {
      AP_SELECT_BOUND(4, 512) AP_SELECT_BOUND(6, 512) AP_SELECT_BOUND(8, 512) AP_SELECT_BOUND(12, 512) AP_SELECT_BOUND(16, 512)
    } else {
      AP_SELECT_BOUND(8, 1024) AP_SELECT_BOUND(9, 1024) AP_SELECT_BOUND(12, 1024) AP_SELECT_BOUND(16, 1024)
    }
  }
#undef AP_SELECT_BOUND
  // The radix select alone.  Few instances with long rows: 1024 threads per instance cut the serial chain of every pass (a
  // 256-thread workgroup walks 32 keys per thread at 128K context while half of the chip has no workgroup at all).
  if (ninst <= 512 && n_mid > 4 * kSelThreads) {
    if (n_mid <= 4 * kSelThreadsWide) AP_SELECT(4, kSelThreadsWide, 0);
    else if (n_mid <= 8 * kSelThreadsWide) AP_SELECT(8, kSelThreadsWide, 0);
    else if (n_mid <= 9 * kSelThreadsWide) AP_SELECT(9, kSelThreadsWide, 0);     // (a 128K context that has grown a little)
    else if (n_mid <= 12 * kSelThreadsWide) AP_SELECT(12, kSelThreadsWide, 0);
    else if (n_mid <= 16 * kSelThreadsWide) AP_SELECT(16, kSelThreadsWide, 0);
    else AP_SELECT(0, kSelThreadsWide, 0);
  }
  else if (n_mid <= 8 * kSelThreads) AP_SELECT(8, kSelThreads, 0);       // the variants differ only in unrolled trip count (2048
  // instances, 198 places, us: 2248 candidates with 9 keys a thread 18.8, with 12 20.4; 2448 with 10 19.8, with 12 20.8)
  else if (n_mid <= 9 * kSelThreads) AP_SELECT(9, kSelThreads, 0);
  else if (n_mid <= 10 * kSelThreads) AP_SELECT(10, kSelThreads, 0);
  else if (n_mid <= 12 * kSelThreads) AP_SELECT(12, kSelThreads, 0);
  else if (n_mid <= 16 * kSelThreads) AP_SELECT(16, kSelThreads, 0);
  else if (n_mid <= 24 * kSelThreads) AP_SELECT(24, kSelThreads, 0);
  else if (n_mid <= 32 * kSelThreads) AP_SELECT(32, kSelThreads, 0);
  else AP_SELECT(0, kSelThreads, 0);
#undef AP_SELECT
  return hipGetLastError();
}

}  // namespace ap
