// Kernels around attention_body.h: block-sparse decode (+ combine of splits) and dense calibration.
#include <mutex>

#include "attention_body.h"

// Scratch for the entry point that must not allocate (ap_sparse_decode_noalloc): the split partials of one
// sparse-decode call.  Every device the library runs on holds its own copy until the process ends.  In host code
// this name is only a handle for hipGetSymbolAddress; kernels get the address that call returned.
constexpr size_t kStaticScratchBytes = AP_NOALLOC_SCRATCH_BYTES;
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

namespace ap {
namespace {

// (the narrow forms are only worth launching if many of their workgroups fit a CU: four waves per SIMD, 128 VGPRs)
template <typename T, int D, int G, int NW, bool PIECED, int HOW = kSplitsOnly>
__global__ __launch_bounds__(NW * kWave) __attribute__((amdgpu_waves_per_eu(NW < kAttnWaves ? 4 : 1)))
void sparse_decode_kernel(SparseArgs a) {
  extern __shared__ __align__(16) float smem[];
  sparse_decode_body<T, D, G, NW, PIECED, HOW>(a, a.inst0 + blockIdx.y, blockIdx.x, smem);
}

// Waves per SIMD the registers are to leave room for: g d / 16 accumulators beside 16 of K and V rows each.
template <int D, int G, int HOW>
__global__ __launch_bounds__(kAttnThreads) __attribute__((amdgpu_waves_per_eu(G <= 4 ? 4 : 3)))
void sparse_stream_kernel(SparseArgs a) {
  extern __shared__ __align__(16) float smem[];
  sparse_stream_body<D, G, HOW>(a, a.inst0 + blockIdx.y, blockIdx.x, smem);
}

// The first n_whole instances by a workgroup each, those after them in a.n_split splits, whose workgroups come behind (mixed_splits).
template <int D, int G>
__global__ __launch_bounds__(kAttnThreads) __attribute__((amdgpu_waves_per_eu(G <= 4 ? 4 : 3)))
void sparse_mixed_kernel(SparseArgs a, int n_whole) {
  extern __shared__ __align__(16) float smem[];
  int inst = blockIdx.x, split = 0;
  if (inst < n_whole) {
    a.n_split = 1;
  } else {
    const int unit = inst - n_whole;
    inst = n_whole + unit / a.n_split;
    split = unit % a.n_split;
  }
  sparse_stream_body<D, G, kSplitsOnly>(a, a.inst0 + inst, split, smem);
}

// Brings the partial softmax statistics of one instance - ml[part * G + h] = (maximum, sum relative to it), part < n_part -
// to factors scale[part * G + h] = exp2((m - M) unit) / L in LDS (0 for an empty part or an empty whole); unit is 1 where the
// maxima are in units of log2, log2(e) for natural ones.  Every value is fetched by
// a thread of its own, all at once: a thread that walks the parts of a head waits for memory once per part.  Calibration
// merge: 33 -> 10 us for 128 instances of 129 chunks, 10 -> 4 us for 8 of 33; sparse decode: 6.4 -> 3.8 us for 8 instances
// of 16 splits, 12.7 -> 8.9 us for 128 of 17.  Called by every thread of the workgroup; ends with a barrier.
template <int G>
__device__ __forceinline__ void merge_scales(const float2* __restrict__ ml, int n_part, float unit, float* scale) {
  __shared__ float s_ml[2 * G];
  const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
  float2 first = make_float2(-INFINITY, 0.f);            // (most merges have no more values than threads)
  if ((int)threadIdx.x < n_part * G) first = ml[threadIdx.x];
  // Wave h / .. of head h: lane l holds parts l, l + 64, ..  (the values are in cache by now)
  for (int h = wave; h < G; h += kAttnWaves) {
    float M = -INFINITY;
    for (int p = lane; p < n_part; p += kWave) M = fmaxf(M, ml[p * G + h].x);
    M = wave_max(M);
    float L = 0.f;
    for (int p = lane; p < n_part; p += kWave) {
      const float2 v = ml[p * G + h];
      L += v.x == -INFINITY ? 0.f : v.y * exp2_fast((v.x - M) * unit);
    }
    L = wave_sum(L);
    if (lane == 0) { s_ml[2 * h] = M; s_ml[2 * h + 1] = L > 0.f ? 1.f / L : 0.f; }
  }
  __syncthreads();
  for (int o = threadIdx.x; o < n_part * G; o += kAttnThreads) {
    const float m = o == (int)threadIdx.x ? first.x : ml[o].x;
    const int h = o % G;
    scale[o] = m == -INFINITY ? 0.f : exp2_fast((m - s_ml[2 * h]) * unit) * s_ml[2 * h + 1];
  }
  __syncthreads();
}

// Merges the splits of one instance: global (M, L) per head, normalised output, pooled row.  The row is nb_cap
// columns long (8K at a 128K context) and all but `cnt` of them are zero, so it is cut into chunks of
// kCombineCols columns, one workgroup each (blockIdx.x - 1 = chunk, blockIdx.y = instance): the chunk is put together
// in LDS - zeros, then the values of the listed blocks that fall into it - and written out whole and coalesced.
// Workgroup 0 of an instance writes the output.  Every workgroup works out the split scales for itself (n_split x G
// values).  It is a launch of a few microseconds whose length is the chain of dependent loads, so whatever does
// not depend on anything is asked for first.
constexpr int kCombineCols = 1024;

template <int D, int G>
__global__ __launch_bounds__(kAttnThreads) void sparse_combine_kernel(SparseArgs a) {
  extern __shared__ __align__(16) float smem[];
  const int inst = a.inst0 + blockIdx.y;
  float* s_scale = smem;                               // [n_split][G]  exp(m_s - M) / L
  const float2* ml = reinterpret_cast<const float2*>(a.part_ml) + (size_t)(inst - a.part_first) * a.n_split * G;
  if (blockIdx.x == 0) {
    merge_scales<G>(ml, a.n_split, a.ml_unit, s_scale);
    const float* acc = a.part_acc + (size_t)(inst - a.part_first) * a.n_split * G * D;
    for (int o = threadIdx.x; o < G * D; o += kAttnThreads) {
      const int h = o / D;
      float v = 0.f;
      int s = 0;
      for (; s + 8 <= a.n_split; s += 8) {             // (eight loads on their way; added up in the order of the splits)
        float x[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) x[i] = acc[(size_t)(s + i) * G * D + o];
#pragma unroll
        for (int i = 0; i < 8; ++i) v = fmaf(x[i], s_scale[(s + i) * G + h], v);
      }
      for (; s < a.n_split; ++s) v = fmaf(acc[(size_t)s * G * D + o], s_scale[s * G + h], v);
      a.out[(size_t)inst * G * D + o] = v;
    }
    return;
  }
  float* s_row = s_scale + a.n_split * G;              // [kCombineCols]
  const int c0 = (blockIdx.x - 1) * kCombineCols, c1 = min(a.nb_cap, c0 + kCombineCols);
  const int cnt = min(max(a.cnt[inst], 0), a.k);
  // This thread's first list position, with its block maxima (a position costs a load of its index and one per head).
  const float* bmp = a.part_bmp + (size_t)inst * G * a.k;
  auto block_of = [&](int jb) __attribute__((always_inline)) {
    return min(max(a.idx[(size_t)inst * a.k + jb], 0), a.nb_cur - 1);
  };
  int blk = -1;
  float bm[G];
  if ((int)threadIdx.x < cnt) {
    blk = block_of(threadIdx.x);
#pragma unroll
    for (int h = 0; h < G; ++h) bm[h] = bmp[(size_t)h * a.k + threadIdx.x];
  }
  for (int j = threadIdx.x; j < c1 - c0; j += kAttnThreads) s_row[j] = 0.f;
  merge_scales<G>(ml, a.n_split, a.ml_unit, s_scale);
  // pooled probability of list position jb: max over heads of (block max relative to its split) * split scale
  for (int jb = threadIdx.x; jb < cnt; jb += kAttnThreads) {
    if (jb != (int)threadIdx.x) {
      blk = block_of(jb);
#pragma unroll
      for (int h = 0; h < G; ++h) bm[h] = bmp[(size_t)h * a.k + jb];
    }
    if (blk >= c0 && blk < c1) {
      const int s = jb / a.blk_per_split;
      float mx = 0.f;
#pragma unroll
      for (int h = 0; h < G; ++h) mx = fmaxf(mx, bm[h] * s_scale[s * G + h]);
      s_row[blk - c0] = mx;                            // (a block listed twice: either of two equal values)
    }
  }
  __syncthreads();
  float* row = a.row + (size_t)inst * a.row_stride;
  for (int j = threadIdx.x; j < c1 - c0; j += kAttnThreads) row[c0 + j] = s_row[j];
}

struct CalibArgs {
  const void* q; const void* K;
  float* row; float* cal_ml; float* cal_bmp;
  int n_units;                    // n_inst * n_chunks
  int t_cap, nb_cap, b, log2b, t_cur, nb_cur, chunk_blocks, n_chunks, chunk_slots;
  const int32_t* table;
  int n_phys;
  float ml_unit;                  // the chunks' maxima times this are exponents of 2
};

// A workgroup for every unit (chunk blockIdx.x of instance blockIdx.y).  (fp32.  With units off a counter, cleared by a launch before, 100 instances at 32K took 321 us
// instead of 304; 16 55.8, 54.4.  g = 8, d = 128 alone lost by it beyond 1024 units: 100 at 32K 326 then, 329 now, 200 at 16K 371, 377; 1024 workgroups that take every 1024th unit 340,
// 376, LDS for three workgroups a CU 351, 384.)
template <int D, int G>
__global__ __launch_bounds__(kAttnThreads) void calibrate_f32_kernel(CalibArgs a) {
  using T = float;
  extern __shared__ __align__(16) float smem[];
  const int inst = blockIdx.y, chunk = blockIdx.x;
  const int c0 = chunk * a.chunk_blocks;
  const int nblk = min(a.chunk_blocks, a.nb_cur - c0);
  const int ld = a.chunk_blocks * a.b;
  const int ntok = nblk * a.b;
  float* s_p = smem;                    // [G][ld]
  float* s_bmp = s_p + G * ld;          // [G][chunk_blocks]
  float* s_m = s_bmp + G * a.chunk_blocks;
  float* s_l = s_m + G;
  int* s_phys = reinterpret_cast<int*>(s_l + G);   // [chunk_blocks] place of each block of the chunk in K

  for (int j = threadIdx.x; j < nblk; j += kAttnThreads)
    s_phys[j] = a.table ? min(max(a.table[(size_t)inst * a.nb_cap + c0 + j], 0), a.n_phys - 1) : c0 + j;
  __syncthreads();
  const T* q_inst = static_cast<const T*>(a.q) + (size_t)inst * G * D;
  const T* K_inst = static_cast<const T*>(a.K) + (a.table ? 0 : (size_t)inst * a.t_cap * D);
  qk_logits<T, D, G, 0>(q_inst, K_inst, a.b, a.log2b, a.t_cur, ntok, [&](int jb) { return c0 + jb; },
                       [&](int jb) { return s_phys[jb]; }, s_p, ld, nullptr);
  __syncthreads();
  softmax_stats<G>(s_p, ld, ntok, a.b, nblk, s_m, s_l, s_bmp);
  for (int pair = threadIdx.x; pair < G * nblk; pair += kAttnThreads) {
    const int h = pair / nblk, jb = pair - h * nblk;
    a.cal_bmp[((size_t)inst * G + h) * a.nb_cap + c0 + jb] = s_bmp[pair];
  }
  if (threadIdx.x < G) {
    float* ml = a.cal_ml + (((size_t)inst * a.chunk_slots + chunk) * G + threadIdx.x) * 2;
    ml[0] = s_m[threadIdx.x];
    ml[1] = s_l[threadIdx.x];
  }
}

// The same for bf16, streaming: the four waves of a workgroup take 16-token passes of a unit in turn (whole blocks, where a
// block is longer) - so that together they read consecutive memory, which streams better than four places at once -
// with the K rows of a wave's next pass on their way while it works on the present one
// (logits on MFMA as in sparse_stream_body; no probabilities are kept, one largest logit per four tokens goes to LDS for
// the block maxima).  The waves meet once per unit, to bring their maxima and sums together, and write the block maxima.
// A workgroup each for the units of K in device memory; over PCIe a few workgroups, each taking every gridDim.x-th, with the rows of the next unit's first pass
// on their way as well.  run_calib says how many workgroups a CU has.
// What bounds it: reads of K, and what little is written.  The block maxima are 0.4 % of the bytes, but of 510 us of 256 instances at 50K they cost 48
// by plain stores, whichever lanes write them, and of 484 they cost 22 written through to memory, though the same bytes get there in as many requests.  Measured, launch
// and merge, us, before (512 workgroups, units off a counter, plain stores) and now: 256 instances at 50K 520, 484 (6.8 TB/s); 2048 at 32K
// 2698, 2530; 4096, g = 1, 5083, 4768; 62 93, 83; 24 48, 40; 300 at 30K, d = 64, 245, 185; 8 16.5, 16.3.  No difference: two or four
// passes of rows on their way per wave, units of 63 or 65 blocks.  Merging by the last workgroup of an instance: 8 instances 17.6, 256 a wave's merge
// holds up its workgroup's stream, 558.
struct CalibUnit { int inst, chunk, nblk, c0; };

template <int D, int G>
__global__ __launch_bounds__(kAttnThreads) __attribute__((amdgpu_waves_per_eu(4)))
void calibrate_stream_kernel(CalibArgs a) {
  using T = bf16_t;
  using Ge = Geom<T, D, G>;
  constexpr int NW = kAttnWaves, E = Ge::E, LPT = Ge::LPT, TPI = Ge::TPI, NL = Ge::NL, KS = D / 32;
  constexpr int RS = D * 2 + kStageRowPad, TILE = kGroupTokens * RS, QROWS = G * RS;
  extern __shared__ __align__(16) char smem_c[];
  __shared__ float s_ml[2][NW][2 * G];                           // [unit parity][wave][maxima | sums]
  const int lane = threadIdx.x & (kWave - 1);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int head = lane & 15, row16 = lane >> 4;
  const int log2gran = max(a.log2b, 4);                          // tokens a wave takes at a time: a pass, or a whole block
  const int qpb = a.b >> 2, quads = (a.chunk_blocks * qpb + 4 * NW - 1) / NW;   // groups of four tokens: per block, per wave (at most)
  char* stage = smem_c + wave * TILE;
  char* s_q = smem_c + NW * TILE + wave * QROWS;                 // (a wave may be a unit ahead, in another instance)
  float* s_qmax = reinterpret_cast<float*>(smem_c + NW * (TILE + QROWS));       // [unit parity][wave][G][quads]

  auto unit_of = [&](int unit) __attribute__((always_inline)) {
    CalibUnit u;
    u.inst = unit / a.n_chunks;
    u.chunk = unit - u.inst * a.n_chunks;
    u.c0 = u.chunk * a.chunk_blocks;
    u.nblk = min(a.nb_cur - u.c0, a.chunk_blocks);
    return u;
  };
  // Passes of this wave in a unit, and the token of the unit that one starts at.
  auto passes = [&](const CalibUnit& u) __attribute__((always_inline)) {
    const int grains = (u.nblk * a.b + (1 << log2gran) - 1) >> log2gran;
    return grains > wave ? ((grains - wave + NW - 1) / NW) << (log2gran - 4) : 0;
  };
  auto token_of = [&](int ps) __attribute__((always_inline)) {
    const int per = log2gran - 4;
    return ((((ps >> per) * NW + wave) << per) + (ps & ((1 << per) - 1))) * kGroupTokens;
  };
  // Where the blocks of a unit lie in K: themselves, or for a paged cache block jb < 64 in lane jb.
  auto place_of = [&](const CalibUnit& u, int jb) __attribute__((always_inline)) {
    return min(max(a.table[(size_t)u.inst * a.nb_cap + min(u.c0 + jb, a.nb_cur - 1)], 0), a.n_phys - 1);
  };
  auto places = [&](const CalibUnit& u) __attribute__((always_inline)) { return a.table ? place_of(u, lane) : 0; };
  auto lookup = [&](const CalibUnit& u, int place, int jb) __attribute__((always_inline)) {
    if (!a.table) return u.c0 + jb;
    return jb < kWave ? __builtin_amdgcn_readlane(place, jb) : __builtin_amdgcn_readfirstlane(place_of(u, jb));
  };
  uint4 kw[NL];
  // Rows of a wave's pass ps: two runs of eight rows, each inside one block.  (A wave without a pass reads a valid row.)
  auto load_k = [&](const CalibUnit& u, int place, int ps) __attribute__((always_inline)) {
    const T* K_inst = static_cast<const T*>(a.K) + (a.table ? 0 : (size_t)u.inst * a.t_cap * D);
    constexpr int kPerRun = 8 / TPI;
    const int tau = token_of(ps), last = u.nblk - 1;
    const int row0 = lookup(u, place, min(tau >> a.log2b, last)) * a.b + (tau & (a.b - 1));
    const int row1 = a.b > 8 ? row0 + 8 : lookup(u, place, min((tau + 8) >> a.log2b, last)) * a.b;
#pragma unroll
    for (int i = 0; i < NL; ++i) {
      const int first = (i < kPerRun ? row0 : row1) + (i % kPerRun) * TPI;
      kw[i] = ld_stream(K_inst + (size_t)first * D + (uint32_t)lane * E);
    }
  };

  int unit = blockIdx.x;
  if (unit >= a.n_units) return;                         // (the whole workgroup)
  CalibUnit u = unit_of(unit);
  int place = places(u);
  load_k(u, place, 0);
  int q_inst = -1;
  using Unit = LogitUnit<D>;

#pragma unroll 1
  for (int round = 0;; ++round) {
    unit += gridDim.x;
    const bool more = unit < a.n_units;
    const CalibUnit v = more ? unit_of(unit) : u;
    const int place_v = more ? places(v) : place;
    if (u.inst != q_inst) {
      const T* q = static_cast<const T*>(a.q) + (size_t)u.inst * G * D;
      for (int o = lane; o < G * D / 8; o += kWave)
        *reinterpret_cast<uint4*>(s_q + (o / (D / 8)) * RS + (o % (D / 8)) * 16) = reinterpret_cast<const uint4*>(q)[o];
      q_inst = u.inst;
      asm volatile("" ::: "memory");                     // a wave's LDS accesses stay in order; so must the compiler
    }
    const int npass = passes(u), n_valid = min(a.t_cur - u.c0 * a.b, u.nblk * a.b);    // tokens of the unit inside the context
    float m = -INFINITY, l = 0.f;
    float* qmax = s_qmax + ((round & 1) * NW + wave) * G * quads;
#pragma unroll 1
    for (int ps = 0; ps < max(npass, 1); ++ps) {         // (a wave without a pass hands its loads on)
#pragma unroll
      for (int i = 0; i < NL; ++i)
        *reinterpret_cast<uint4*>(stage + (i * TPI + lane / LPT) * RS + (lane % LPT) * 16) = kw[i];
      asm volatile("" ::: "memory");
      {
        const bool inside = ps + 1 < npass;              // (one load site: the rows have one source on the way round)
        const CalibUnit w = inside ? u : v;
        if (inside || more) load_k(w, inside ? place : place_v, inside ? ps + 1 : 0);
      }
      float4v lg = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int s = 0; s < KS; ++s) {
        const uint4 wk = *reinterpret_cast<const uint4*>(stage + head * RS + (row16 * (D / 4) + s * 8) * 2);
        const uint4 wq = *reinterpret_cast<const uint4*>(s_q + (head & (G - 1)) * RS + (row16 * (D / 4) + s * 8) * 2);
        lg = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, wk), __builtin_bit_cast(bf16x8, wq), lg, 0, 0, 0);
      }
      asm volatile("" ::: "memory");                     // the next pass overwrites the tile read above
      const int n_in = ps < npass ? n_valid - token_of(ps) - 4 * row16 : 0;
      float p[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) p[i] = i < n_in ? lg[i] : -INFINITY;
      const float mx = fmaxf(fmaxf(p[0], p[1]), fmaxf(p[2], p[3]));
      if (head < G && ps < npass) qmax[head * quads + ps * 4 + row16] = mx;
      const float m_new = fmaxf(m, Unit::reference(mx)), m_ref = m_new == -INFINITY ? 0.f : m_new;      // (nothing but masked tokens so far)
      auto rel = [&](float x) __attribute__((always_inline)) { return Unit::exp_of(x, m_ref); };
      l = l * exp2_fast(m - m_ref) + ((rel(p[0]) + rel(p[1])) + (rel(p[2]) + rel(p[3])));
      m = m_new;
    }
    const auto larger = [](float x, float y) { return fmaxf(x, y); };
    const auto plus = [](float x, float y) { return x + y; };
    const float mw = across_32(across_16(m, larger), larger);
    const float lw = across_32(across_16(m == -INFINITY ? 0.f : l * exp2_fast(m - mw), plus), plus);
    float (*ml)[2 * G] = s_ml[round & 1];
    if (lane < G) { ml[wave][lane] = mw; ml[wave][G + lane] = lw; }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // (not __syncthreads(): that would wait for the K rows on their way)
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    // The unit's maximum and sum, of head lane % G; block maxima relative to that maximum, one head's columns by neighbouring lanes, written
    // through to memory.  (The next unit's maxima go to the other half of s_ml and s_qmax: a wave that gets to the one
    // after it has met the others in between.)
    {
      const int hl = lane & (G - 1);
      float M = -INFINITY, L = 0.f;
#pragma unroll
      for (int w = 0; w < NW; ++w) M = fmaxf(M, ml[w][hl]);            // (a unit has a token inside the context)
#pragma unroll
      for (int w = 0; w < NW; ++w) L += ml[w][G + hl] * exp2_fast(ml[w][hl] - M);
      if (wave == 0 && lane < G) {
        float* to = a.cal_ml + (((size_t)u.inst * a.chunk_slots + u.chunk) * G + lane) * 2;
        st_shared_out<true>(to, M);
        st_shared_out<true>(to + 1, L);
      }
      const int per = log2gran - a.log2b;                // (log2) blocks of a grain; the grains are dealt to the waves in turn
      const int log2blocks = 31 - __builtin_clz(a.chunk_blocks);
#pragma unroll 1
      for (int p = threadIdx.x; p < G << log2blocks; p += kAttnThreads) {
        const int h = p >> log2blocks, jb = p & (a.chunk_blocks - 1);
        const float Mh = fmaxf(fmaxf(ml[0][h], ml[1][h]), fmaxf(ml[2][h], ml[3][h]));
        const int grain = jb >> per, i = ((grain / NW) << per) + (jb & ((1 << per) - 1));
        const float* qm = s_qmax + (((round & 1) * NW + grain % NW) * G + h) * quads + i * qpb;
        if (jb < u.nblk) {
          float mx = qm[0];
#pragma unroll 1
          for (int k = 1; k < qpb; ++k) mx = fmaxf(mx, qm[k]);
          st_shared_out<true>(a.cal_bmp + ((size_t)u.inst * G + h) * a.nb_cap + u.c0 + jb, Unit::exp_of(mx, Mh));
        }
      }
    }
    if (!more) break;                                    // (the same for every wave)
    u = v;
    place = place_v;
  }
}
static_assert(kAttnWaves == 4, "four waves' maxima");

// Merges the chunks of one instance into the dense row, kCombineCols columns per workgroup (blockIdx.x; blockIdx.y =
// instance); the block maxima do not wait for the scales.
template <int G>
__global__ __launch_bounds__(kAttnThreads) void calibrate_finish_kernel(CalibArgs a) {
  extern __shared__ __align__(16) float smem[];
  constexpr int PER = kCombineCols / kAttnThreads;
  const int inst = blockIdx.y, c0 = blockIdx.x * kCombineCols;
  float* s_scale = smem;                // [n_chunks][G]
  const float* bmp = a.cal_bmp + (size_t)inst * G * a.nb_cap;
  float bm[PER][G];
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    const int j = c0 + i * kAttnThreads + threadIdx.x;
#pragma unroll
    for (int h = 0; h < G; ++h) bm[i][h] = j < a.nb_cur ? bmp[(size_t)h * a.nb_cap + j] : 0.f;
  }
  merge_scales<G>(reinterpret_cast<const float2*>(a.cal_ml) + (size_t)inst * a.chunk_slots * G, a.n_chunks, a.ml_unit, s_scale);
  float* row = a.row + (size_t)inst * a.nb_cap;
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    const int j = c0 + i * kAttnThreads + threadIdx.x;
    if (j >= a.nb_cap) continue;
    float mx = 0.f;
    if (j < a.nb_cur) {
      const int c = j / a.chunk_blocks;
#pragma unroll
      for (int h = 0; h < G; ++h) mx = fmaxf(mx, bm[i][h] * s_scale[c * G + h]);
    }
    row[j] = mx;
  }
}

int ilog2(int x) { int l = 0; while ((1 << l) < x) ++l; return l; }

// Workgroups of kernel `fn` (NT threads, lds bytes of LDS) the device holds at once; 0 if it cannot be asked.
template <class Fn> int resident_workgroups(Fn fn, int nt, size_t lds) {
  int per_cu = 0, dev = 0;
  int n_cu = 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, fn, nt, lds) != hipSuccess ||
      hipGetDevice(&dev) != hipSuccess || hipDeviceGetAttribute(&n_cu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
    return 0;
  return per_cu * n_cu;
}

template <int D, int G> hipError_t run_combine(int ninst, const SparseArgs& a, hipStream_t st) {
  const size_t lds = sizeof(float) * ((size_t)a.n_split * G + kCombineCols);
  sparse_combine_kernel<D, G><<<dim3(1 + (a.nb_cap + kCombineCols - 1) / kCombineCols, ninst), kAttnThreads, lds, st>>>(a);
  return hipGetLastError();
}

// Are the splits merged by the last workgroup of an instance to finish, or by a launch of their own?  By the last one where the workspace has counters, and
//   - there are no more than two workgroups a CU, which are resident at once whatever LDS they have: in further rounds every workgroup holds its
//     place until its partials have reached memory.  (513 to 1024 workgroups, steps in us, merged inside / by a launch: fp32, 1024 tokens, g = 8,
//     d = 128, 60 instances 42.0 / 35.9, g = 4, 40 instances 26.0 / 24.5; bf16, g = 8, d = 64, 510 x 8192 tokens 231 / 214, g = 4, d = 128,
//     350 x 8192 250 / 246, 510 x 16384 699 / 705.)  Single fp32 calls with d = 128 one workgroup a CU (1024 tokens, g = 4, 30 instances 13.6 / 12.1, 3
//     11.0 / 11.6; d = 64, 48 x 512, g = 8, 12.1 / 12.8, 32 x 1024, g = 4, 9.6 / 10.8; behind a predictor, d = 128, 128 x 256, 18.3 / 20.5).
//   - one workgroup has little to merge: few splits, and few sums in all.  (8 instances, fp32, g = 4, d = 128: 16 splits 19.4 / 21.9, 24 22.9 /
//     22.2, 64 36.1 / 25.8; g = 1, 64 splits 29.0 / 22.1; bf16, d = 128, g = 4: 8 splits 16.2 / 20.1, 16 20.5 / 21.3, 20 23.1 / 22.0; 4 instances,
//     g = 8, 12 splits 22.0 / 25.8, 16 24.3 / 23.5, 64 51.6 / 29.0.)
// Fewer sums behind a selection that is a launch of its own, where the merge's launch finds the host ahead (g = 4, d = 128: 16 splits, 126
// places, 16 instances 23.5 / 20.6, 8 instances 21.6 / 20.6, 4 splits, 128 instances, 35.5 / 36.5; g = 1, d = 64: 15 splits, 7 instances 22.0 / 23.2;
// without a selection 16 splits, 8 instances 15.1 / 16.5).  Single calls, us, by a launch / inside, bf16, d = 128: 8 instances x 1024 tokens, g = 4, 10.8 /
// 8.3, 16 x 2048 10.8 / 9.8, 64 x 2048, g = 8, 21.2 / 18.1, 100 x 1024 15.4 / 13.1, 32 x 4096 15.9 / 15.6, 128 x 4096 44.3 / 43.6.
static_assert(kMergeInsideSplits < 1 << kTicketBits, "a ticket each");
constexpr int kMergeInsideWorkgroups = 512, kMergeInsideSums = 12288, kMergeFewSums = 4096;
static_assert(2 * kTicketInstances >= kMergeInsideWorkgroups, "every instance in two splits or more has a word");
bool merge_inside(const Shape& s, int ninst, int n_split, int most_sums = kMergeInsideSums) {
  return !s.no_counters && n_split > 1 && n_split <= kMergeInsideSplits && n_split * s.g * s.d <= most_sums &&
         (long)ninst * n_split <= kMergeInsideWorkgroups;
}

// Does a launch without a selection of its own merge inside?  Behind a selection's launch (a.pred) with few sums.  Single calls (us, by a launch / inside) not with
//   - 16 splits of many sums: the merge's launch takes eight splits at a time and is slow only on a remainder - unless the decode is over before the
//     host has the second launch ready.  (bf16, d = 128, g = 4, 16 instances x 2048 tokens 11.5 / 9.9, 3072 11.7 / 10.9, 4096 11.4 / 11.8, 8192 15.8 /
//     17.0; d = 64, g = 8: 30 x 2048 11.5 / 12.0, 32 x 8192 18.9 / 19.7; fp32, d = 64, g = 8, 1024 tokens: 8 instances 11.0 / 11.7, 32 13.0 / 13.6; d = 128,
//     g = 4: 8 instances 11.3 / 11.1, 10.8 / 11.0.  12 splits: bf16, 20 x 8192, g = 4, 20.6 / 19.9, g = 8 26.6 / 25.3; d = 64, g = 8, 40 x 4096 17.5 / 16.0; fp32, d = 64,
//     g = 8, 768 tokens, 8 12.9 / 11.4, 32 14.8 / 13.0.)
//   - more than a workgroup a CU with d = 128, more than eight splits of many sums and long lists (g = 8, 52 x 8192 42.7 / 44.5, 40 x 16384, 12 splits, 114.6 / 116.9; g = 4, 52 x
//     8192 38.0 / 38.6, 4096 22.4 / 22.6), or a long share for each (g = 4, 200 x 16384 255.4 / 259.3, 86 x 16384 113.3 / 115.3, x 8192 60.8 / 60.1, 128 x 32768 322.1 / 323.6; g = 2,
//     200 x 32768 507.6 / 510.8; g = 8, 86 x 16384 124.4 / 123.9; g = 1, 86 x 32768 214.6 / 215.0, 100 x 32768 248.4 / 247.2).  d = 64 gains with all (128 x 32768, g = 4, 167.2 / 165.0).
//   - more than eight splits of many sums with d = 128 and up to a workgroup a CU, where lists are long for that number: the more splits the launch has beyond eight, the longer it waits for
//     the remainder.  (g = 4 and 8, 28 instances, nine splits: 4096 tokens 15.6 / 15.3, 19.3 / 19.9, 5120 17.3 / 17.7, 21.7 / 22.4, 16384 41.7 / 42.2, 47.2 / 48.4; 24, ten: 6144 17.7 / 18.5, 23.3 / 23.7,
//     8192 21.5 / 21.7, 27.6 / 27.1, 16384 37.3 / 37.8, 43.5 / 44.5; 22, eleven: 8192 21.3 / 20.8, 26.7 / 26.2, 12288 27.7 / 28.4, 34.8 / 34.4, 24576 49.5 / 50.5, 56.6 / 57.2; 20, twelve: 12288 26.3 / 26.0, 32.5 /
//     31.5, 16384 32.1 / 32.9, 39.8 / 39.3, 32768 57.6 / 58.6, 67.0 / 67.5; g = 4, 18, fourteen: 16384 31.7 / 31.0, 24576 42.8 / 42.6, 32768 54.4 / 54.9.)
constexpr int kMergeHostTokens = 3072, kMergeLongTokens = 4096, kMergeLongStep = 3072, kMergeLongShare = 2560;
bool merge_now(const Shape& s, const SparseArgs& a, int ninst) {
  int most = a.pred != nullptr ? kMergeFewSums : kMergeInsideSums;
  if (a.pred == nullptr && !s.cleared) {
    const int tokens = a.k * a.b;
    const bool crowded = s.d == 128 && (long)ninst * a.n_split > 256, host_behind = s.kv_dtype == AP_BF16 && s.d == 128 && tokens <= kMergeHostTokens;
    if (crowded && tokens > kMergeLongShare * a.n_split) return false;
    const int longest = kMergeLongTokens + (crowded ? 0 : kMergeLongStep * (a.n_split - 9));
    if ((a.n_split == kMergeInsideSplits && !host_behind) || (s.d == 128 && a.n_split > 8 && tokens > longest)) most = kMergeFewSums;
  }
  return merge_inside(s, ninst, a.n_split, most);
}

// Does the streaming decode (and the fp32 one in splits) make the selection too?  Every workgroup of an instance makes all of it, which is
// no loss where they would otherwise wait for the launch that does, and hardly any CU has two of them.  (Whole steps, 2041 candidates, us:
// 8 instances 17.6 -> 16.6, 32 19.7 -> 18.4, 128 29.3 -> 28.0, one of fp32 with 126 candidates 16.8 -> 15.3, two launches instead of three; whole
// lists, 256 of 1243 candidates, 57.5 -> 55.1.)  Many places for one workgroup to rank (97 to 128 of them) only where there are few splits: 8 instances,
// 16 splits, 126 places 20.6 with three launches or four, 16 instances 21.9 and 20.6, 128 instances of four splits 34.4 and 36.7.
constexpr int kRankedSplits = 8;
bool select_here(const Shape& s, int ninst, int n_split, int nb_cur) {
  const int n_mid = nb_cur - s.n_sink - s.n_local, k_mid = s.k - s.n_sink - s.n_local;
  return (n_split == 1 || (s.cleared && merge_inside(s, ninst, n_split))) && (long)ninst * n_split <= kMergeInsideWorkgroups &&
         n_mid <= kSelectInsideKeys * kSelThreads && k_mid >= 1 && k_mid <= (n_split <= kRankedSplits ? kSelMaxMid : kSelFewMid);
}

// LDS bytes of a launch that merges, and selects if HOW says so, on top of lds for the decode; sets a.sel_at.
size_t lds_of_form(SparseArgs& a, size_t lds, int g, int how) {
  const size_t merge = merge_lds_bytes(a.n_split, g), scratch = sizeof(uint32_t) * sel_scratch_words<kSelThreads>();
  if (lds < merge) lds = merge;
  if (how != kSelectInside) return lds;
  if (lds < scratch) lds = scratch;
  a.sel_at = (int)(lds / sizeof(float));
  return lds + sizeof(int32_t) * (a.k + 1);
}

// The selection that a decode launch leaves to one of its own.
hipError_t select_first(const Shape& s, int ninst, const SparseArgs& a, hipStream_t st) {
  if (a.pred == nullptr) return hipSuccess;
  return launch_select(s, a.inst0, ninst, a.pred, a.nb_cur, const_cast<int32_t*>(a.idx), const_cast<int32_t*>(a.cnt), st);
}

// Workgroups per instance the streaming form uses, of the a.n_split that the workspace has room for: the number with the least
// time by this reckoning.  The fullest of 256 CUs has r = ceil(workgroups / 256) of them and takes r shares of a list, at 32 KB
// a us where it has one workgroup (20 at d = 64, whose workgroups have half the bytes on their way), 29 with two and 22.5
// with more, when all of memory is busy; a merge costs 3 us, 0.03 a split and 0.006 an instance.  So few instances are split until every
// CU has work, and 280 are not left with two lists on 24 CUs and one on the others.  No split is shorter than two passes a wave (128
// tokens), 64 to merge at most unless LDS asks for more.  (Over 1 to 1000 instances, lists of 256 to 16384 tokens, g = 1 to 8,
// both head sizes, wherever it takes 14 us or more, the choice is 1.3 % from the best one.  Decode + merge in us, d = 128, bf16,
// splits: time.  128 x 8192 tokens, g = 4, 1: 120, 2: 87, 8: 90; 144 x 8192, g = 1, 1: 109, 2: 118, 3: 97, 5: 95; 280 x 4096,
// g = 2, 1: 116, 4: 98; 512 x 8192, g = 4, 1: 318, 2: 334; 8 x 1024, g = 4, 4: 13.4, 8: 10.8.)
template <int D> int stream_splits(const SparseArgs& a, int ninst, int g) {
  const long tokens = (long)a.k * a.b;
  const long least = (g * tokens + 40959) / 40960;       // (a list's largest logits, one float per head and four tokens, in 40 KiB)
  int best = least < 1 ? 1 : (int)least;
  if (best >= a.n_split) return a.n_split;
  double best_us = 0.0;
  for (int u = best, first = best; u <= a.n_split && (u == first || (u <= 64 && tokens >= 128L * u)); ++u) {
    const long r = ((long)u * ninst + 255) / 256;
    const double kb_per_us = r == 1 ? (D == 128 ? 32.0 : 20.0) : r == 2 ? 29.0 : 22.5;
    const double us = r * (4e-3 * D * tokens / u) / kb_per_us + (u > 1 ? 3.0 + 0.03 * u + 0.006 * ninst : 0.0);
    if (u == first || us < best_us) { best = u; best_us = us; }
  }
  return best;
}

// Instances a little beyond a multiple of the CUs: that multiple goes a workgroup each, as many a CU, and only what is beyond it in splits, in one launch
// with the long workgroups first.  Splitting every list alike leaves some CUs a share more than others, however short the shares, and merges all
// instances.  Returns the splits of those beyond, 0 or 1 if all are to be treated alike.  They get one more workgroup a CU, two where they are a quarter of the CUs
// or fewer, not more (600 instances x 2048 tokens, g = 8, 88 beyond: 109 us with two splits, 114 with three, 113 with five; 300 x 1024, g = 4, 44 beyond: with
// eight, all that 1024 tokens allow, 31.2, with five 32.2, eleven 32.8, two 32.3) - so no more than half of the CUs' number beyond, or one more workgroup would take a whole
// list.  Beyond one list a CU no more than a quarter: up to half it depends on the length (all alike / mixed, g = 8, 330 instances x 4096 tokens 127 / 120, 384 x 1024 39.1 / 42.3; g = 4, 350 x
// 4096 129 / 122, 384 x 2048 70.4 / 73.0).  Not where half of the CUs would still be without one, or short lists make a merge of them cost more than the balance gives.
// bf16, us, all alike / mixed: g = 8, d = 128, 2048 tokens, 264 instances 60.7 / 52.5, 320 67.9 / 62.3, 576 118.5 / 109.3, 640 127.1 / 113.9, 896 174 / 159; g = 4, 1024 tokens, 264 31.2 / 28.2,
// 576 56.8 / 54.3, 640 61.2 / 58.0, 896 83.5 / 80.2; g = 1, 4096 tokens, 264 94.7 / 87.3, 640 208.7 / 207.4, 896 293 / 299; d = 64, g = 4, 4096 tokens, 576 115 / 104, 896 161 / 153.  Not taken:
// 512 tokens, d = 128, g = 4, 320 17.7 / 20.3, 640 30.0 / 31.6; d = 64, 264 x 4096, g = 4, 58.0 / 57.2, g = 8, 280 x 4096 64.4 / 71.2, 1024 tokens, g = 4, 640 30.7 / 31.8.
template <int D> int mixed_splits(const SparseArgs& a, int ninst, int g) {
  constexpr int kCUs = 256;
  const int n_whole = ninst / kCUs * kCUs, beyond = ninst - n_whole;
  const long tokens = (long)a.k * a.b;
  if (a.n_split < 2 || n_whole == 0 || beyond == 0 || beyond > (n_whole == kCUs ? kCUs / 4 : kCUs / 2) || (D == 64 && n_whole == kCUs)) return 0;
  if (4 * D * tokens < 512 * 1024 || g * tokens > 40960) return 0;         // (the latter: a whole list's logits, as in stream_splits)
  // Contiguous instances 4 KB less or more than 512 KB apart: whole lists, which stay in step, then read from few channels at a time, shares of lists less so.  (All alike /
  // mixed, d = 128, g = 4: 516 KB, 640 x 1024 tokens 60.8 / 67.5, x 2016 114 / 130, 896 x 1024 83 / 90; d = 64, 640 x 2048 65.2 / 69.7; 508 KB, 640 x 1024 61.5 / 67.4, 264 30.3 /
  // 33.6.  Not so at 506 or 510, 514 or 518: 60 / 57.)  Twice that: d = 128, 1032 KB, lists of half the context or more lose, 640 x 2016 118 / 126, 300 x 1024, g = 2, 29.5 / 33.9,
  // shorter ones are as fast, 640 x 1024 of 4128 62.7 / 62.3; d = 64 gains, 640 x 2048 of 8256 74 / 64, and 1016 KB does, 640 x 1024 of 4064 62.7 / 60.8, 264 31.3 / 28.4.
  const size_t apart = sizeof(bf16_t) * D * (size_t)a.t_cap;
  if (a.table == nullptr && (apart == 508 * 1024 || apart == 516 * 1024 || (D == 128 && apart == 1032 * 1024))) return 0;
  long splits = (beyond > kCUs / 4 ? kCUs : 2 * kCUs) / beyond;
  if (splits > tokens / 128) splits = tokens / 128;                        // (two passes a wave)
  if (splits > 64) splits = 64;
  const long room = (long)a.n_split * ninst / beyond;                      // partials the workspace is laid out for
  return (int)(splits < room ? splits : room);
}

template <int D, int G>
hipError_t run_stream(const Shape& s, int ninst, SparseArgs a, hipStream_t st) {
  a.ml_unit = 1.f;
  int want = a.n_split > 1 ? stream_splits<D>(a, ninst, G) : 1;
  // (Lists of so many blocks, or rows with so many, that their entries beside the logits exceed 64 KiB take more splits; with
  // those the workspace is laid out for they fit.)
  auto lds_of = [&](int splits) {
    return sizeof(float) * sparse_stream_lds_floats<D, G>((a.k + splits - 1) / splits, a.b, splits == 1 ? a.nb_cap : 0);
  };
  while (want < a.n_split && lds_of(want) > 65536) ++want;
  if (const int splits = mixed_splits<D>(a, ninst, G); splits > 1) {
    SparseArgs m = a;
    m.blk_per_split = (a.k + splits - 1) / splits;
    m.n_split = (a.k + m.blk_per_split - 1) / m.blk_per_split;
    const size_t lds_whole = lds_of(1), lds_split = lds_of(m.n_split), lds = lds_whole > lds_split ? lds_whole : lds_split;
    if (m.n_split > 1 && lds <= 65536) {
      const int beyond = ninst % 256, n_whole = ninst - beyond;
      hipError_t e = select_first(s, ninst, m, st);
      if (e != hipSuccess) return e;
      m.part_first = m.inst0 + n_whole;
      sparse_mixed_kernel<D, G><<<dim3(n_whole + beyond * m.n_split), kAttnThreads, lds, st>>>(m, n_whole);
      e = hipGetLastError();
      if (e != hipSuccess) return e;
      m.inst0 = m.part_first;
      return run_combine<D, G>(beyond, m, st);
    }
  }
  a.blk_per_split = (a.k + want - 1) / want;
  a.n_split = (a.k + a.blk_per_split - 1) / a.blk_per_split;
  const dim3 grid(a.n_split, ninst);
  if (a.pred != nullptr && select_here(s, ninst, a.n_split, a.nb_cur)) {
    const size_t lds = lds_of_form(a, lds_of(want), G, kSelectInside);
    if (lds <= 65536) {
      sparse_stream_kernel<D, G, kSelectInside><<<grid, kAttnThreads, lds, st>>>(a);
      return hipGetLastError();
    }
  }
  hipError_t e = select_first(s, ninst, a, st);
  if (e != hipSuccess) return e;
  if (merge_now(s, a, ninst)) {
    const size_t lds = lds_of_form(a, lds_of(want), G, kMergeInside);
    if (s.cleared) sparse_stream_kernel<D, G, kMergeInside><<<grid, kAttnThreads, lds, st>>>(a);
    else sparse_stream_kernel<D, G, kMergeAlone><<<grid, kAttnThreads, lds, st>>>(a);
    return hipGetLastError();
  }
  sparse_stream_kernel<D, G, kSplitsOnly><<<grid, kAttnThreads, lds_of(want), st>>>(a);
  e = hipGetLastError();
  if (e != hipSuccess || a.n_split == 1) return e;
  return run_combine<D, G>(ninst, a, st);
}

template <typename T, int D, int G>
hipError_t run_sparse(const Shape& s, int ninst, SparseArgs a, hipStream_t st) {
  // The streaming form: bf16 lists cut into splits, and whole lists with g = 8 (1024 instances 120 -> 99 us, 1700
  // 172 -> 162; the phased form has no narrow variants for it).
  if constexpr (std::is_same<T, bf16_t>::value && G == 8) return run_stream<D, G>(s, ninst, a, st);
  else {
  if constexpr (std::is_same<T, bf16_t>::value)
    if (a.n_split > 1) return run_stream<D, G>(s, ninst, a, st);
  const int nblk_cap = (a.n_split == 1) ? a.k : a.blk_per_split;
  a.piece_blocks = nblk_cap;
  const size_t lds = sizeof(float) * sparse_lds_floats<D, G, kAttnWaves>(nblk_cap, nblk_cap, a.b, a.nb_cap);
  size_t lds_inside = 0;
  if (std::is_same<T, float>::value && a.n_split > 1 && a.pred != nullptr && select_here(s, ninst, a.n_split, a.nb_cur)) lds_inside = lds_of_form(a, lds, G, kSelectInside);
  const bool inside = lds_inside != 0 && lds_inside <= 65536;
  hipError_t e = inside ? hipSuccess : select_first(s, ninst, a, st);
  if (e != hipSuccess) return e;
  // More instances than the chip holds four-wave workgroups: the launch runs in rounds, the last one part
  // empty, and every round pays its start-up and drain.  Workgroups of two waves or one that keep the
  // probabilities of kNarrowPieceTokens tokens at a time are small enough for more of them to be resident; the
  // widest form with the fewest rounds is used.
  if constexpr (G <= 4) if (a.n_split == 1 && nblk_cap * a.b > kNarrowPieceTokens) {   // (g = 8 would spill in those forms)
    const int pb_n = kNarrowPieceTokens / a.b;
    const size_t lds_2 = sizeof(float) * sparse_lds_floats<D, G, 2>(nblk_cap, pb_n, a.b, a.nb_cap);
    const size_t lds_1 = sizeof(float) * sparse_lds_floats<D, G, 1>(nblk_cap, pb_n, a.b, a.nb_cap);
    if (s.occ->sparse_slots[0] < 0) {
      s.occ->sparse_slots[0] = resident_workgroups(sparse_decode_kernel<T, D, G, kAttnWaves, false>, kAttnThreads, lds);
      s.occ->sparse_slots[1] = resident_workgroups(sparse_decode_kernel<T, D, G, 2, true>, 2 * kWave, lds_2);
      s.occ->sparse_slots[2] = resident_workgroups(sparse_decode_kernel<T, D, G, 1, true>, kWave, lds_1);
    }
    int form = 0, best_rounds = 0;
    for (int f = 0; f < 3; ++f) {
      if (s.occ->sparse_slots[f] <= 0) { form = 0; break; }     // occupancy unknown: stay with the four-wave form
      const int rounds = (ninst + s.occ->sparse_slots[f] - 1) / s.occ->sparse_slots[f];
      if (f == 0 || rounds < best_rounds) { form = f; best_rounds = rounds; }
    }
    if (form != 0) {
      a.piece_blocks = pb_n;
      if (form == 1) sparse_decode_kernel<T, D, G, 2, true><<<dim3(1, ninst), 2 * kWave, lds_2, st>>>(a);
      else sparse_decode_kernel<T, D, G, 1, true><<<dim3(1, ninst), kWave, lds_1, st>>>(a);
      return hipGetLastError();
    }
  }
  if constexpr (std::is_same<T, float>::value)
    if (inside || (merge_now(s, a, ninst) && (s.cleared || D == 64 || ninst * a.n_split <= 256))) {
      const dim3 grid(a.n_split, ninst);
      const size_t lds_merge = lds_of_form(a, lds, G, kMergeInside);
      if (inside) sparse_decode_kernel<T, D, G, kAttnWaves, false, kSelectInside><<<grid, kAttnThreads, lds_inside, st>>>(a);
      else if (s.cleared) sparse_decode_kernel<T, D, G, kAttnWaves, false, kMergeInside><<<grid, kAttnThreads, lds_merge, st>>>(a);
      else sparse_decode_kernel<T, D, G, kAttnWaves, false, kMergeAlone><<<grid, kAttnThreads, lds_merge, st>>>(a);
      return hipGetLastError();
    }
  sparse_decode_kernel<T, D, G, kAttnWaves, false><<<dim3(a.n_split, ninst), kAttnThreads, lds, st>>>(a);
  e = hipGetLastError();
  if (e != hipSuccess || a.n_split == 1) return e;
  return run_combine<D, G>(ninst, a, st);
  }
}

// Tokens of a calibration unit (and of the chunks the merge sees): 1024, or 512 or 256 where that leaves the chip
// without a workgroup for every place it has (8 instances at 32K: 1032 units of 256 tokens instead of 264 of 1024; 8 at 8K with
// room for 128K 13.2 -> 9.5 us), unless the merge would have more than 60000 bytes of factors.  fp32 at d = 128 has half as many places, and a
// last round of few units costs more than long units (us with 256 / 512 / 1024 tokens: 32 instances x 8000 tokens 26.7 / 29.8 / 42.2, 50 x 8000
// 58.3 / 42.0 / 46.3, 8 x 131000 116 / 117 / 98, 400 x 2000 95 / 95 / 90; d = 64, 200 x 2000 23.6 / 24.0 / 25.7).
int calib_chunk_tokens(const Shape& s, int t_cur) {
  int tokens = kCalibChunkTokens;
  if (s.kv_dtype != AP_BF16 && s.k_on_host) return tokens;   // (the fp32 form has no small grid for the link)
  const size_t places = s.kv_dtype != AP_BF16 && s.d == 128 ? 512 : 1024;
  while (tokens > kCalibMinChunkTokens && (size_t)s.n_inst * t_cur / tokens < places &&
         (2 * (size_t)t_cur / tokens + 2) * s.g * sizeof(float) <= 60000 && (2 * t_cur + tokens - 1) / tokens <= s.calib_chunks)
    tokens /= 2;
  return tokens;
}

// LDS that leaves room for two workgroups a CU.  With d = 128 these keep memory busy, and more only spread the reads over more places - in calls of many units (us with two
// / as many as fit: 256 instances at 50K 482 / 501, 2048 at 32K 2488 / 2606, 300 at 8K 100 / 104, 64 at 32K 86.2 / 90.0).  Where all units fit at once none has to wait (8 instances at 32K
// 18.6 / 16.5, 45 at 8K 21.7 / 18.9, 33 at 32K 54.6 / 51.3, though 32 at 32K 45.9 / 50.5).  A little beyond what fits it is the length of the last round that tells, either way: 62 at 8K 28.0 / 24.4, 62 at 32K 82.5 /
// 87.9, 50 at 16K 41.2 / 37.1, 128 at 16K 90.5 / 91.0, 64 at 32K with g = 8 91.1 / 87.6.  d = 64, with half the bytes on their way per workgroup: as many as fit (300 at 30K, two 261, three 201, five 188).
constexpr size_t kCalibPairLds = 65536;

// A launch has fewer than 2^32 threads in x: workgroups take several units each beyond this (65535 instances of 131073 tokens, in a pool that they share).
constexpr int kCalibMostWorkgroups = 1 << 23;

template <typename T, int D, int G>
hipError_t run_calib(const Shape& s, CalibArgs a, hipStream_t st) {
  if constexpr (std::is_same<T, bf16_t>::value) {
    a.ml_unit = 1.f;
    auto lds_of = [&](int tokens, bool several) {          // (largest logits of two units, where a workgroup takes several)
      const size_t quads = (tokens / 4 + 4 * kAttnWaves - 1) / kAttnWaves;
      return (size_t)kAttnWaves * ((kGroupTokens + G) * (D * 2 + kStageRowPad) + (several ? 2 : 1) * sizeof(float) * G * quads);
    };
    // Over PCIe 16 workgroups fill the link, and a thousand places at once cost it 15 % (8 instances at 32K, 67 MB, us: 16
    // workgroups 1178, 64 1190, 256 1272, 512 1358).
    const int most = s.k_on_host ? 16 : kCalibMostWorkgroups, grid = a.n_units < most ? a.n_units : most;
    const int tokens = a.chunk_blocks * a.b;
    size_t lds = lds_of(tokens, grid < a.n_units);
    if (D == 128 && !s.k_on_host) {
      const int kind = tokens == kCalibChunkTokens ? 0 : tokens == kCalibChunkTokens / 2 ? 1 : 2;
      if (s.occ->calib_slots[kind] < 0) s.occ->calib_slots[kind] = resident_workgroups(calibrate_stream_kernel<D, G>, kAttnThreads, lds);
      if (a.n_units > s.occ->calib_slots[kind] && lds < kCalibPairLds) lds = kCalibPairLds;
    }
    calibrate_stream_kernel<D, G><<<dim3(grid), kAttnThreads, lds, st>>>(a);
  } else {
    const size_t lds = sizeof(float) * ((size_t)G * a.chunk_blocks * a.b + G * a.chunk_blocks + 2 * G + a.chunk_blocks);
    calibrate_f32_kernel<D, G><<<dim3(a.n_chunks, s.n_inst), kAttnThreads, lds, st>>>(a);
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  calibrate_finish_kernel<G><<<dim3((a.nb_cap + kCombineCols - 1) / kCombineCols, s.n_inst), kAttnThreads,
                               sizeof(float) * a.n_chunks * G, st>>>(a);
  return hipGetLastError();
}

#define AP_DISPATCH_G(FN, T, D, ...)                              \
  switch (s.g) {                                                  \
    case 1: return FN<T, D, 1>(__VA_ARGS__);                      \
    case 2: return FN<T, D, 2>(__VA_ARGS__);                      \
    case 4: return FN<T, D, 4>(__VA_ARGS__);                      \
    case 8: return FN<T, D, 8>(__VA_ARGS__);                      \
    default: return hipErrorInvalidValue;                         \
  }
#define AP_DISPATCH(FN, ...)                                                      \
  if (s.kv_dtype == AP_BF16) {                                                    \
    if (s.d == 128) { AP_DISPATCH_G(FN, bf16_t, 128, __VA_ARGS__) }               \
    if (s.d == 64) { AP_DISPATCH_G(FN, bf16_t, 64, __VA_ARGS__) }                 \
  } else {                                                                        \
    if (s.d == 128) { AP_DISPATCH_G(FN, float, 128, __VA_ARGS__) }                \
    if (s.d == 64) { AP_DISPATCH_G(FN, float, 64, __VA_ARGS__) }                  \
  }                                                                               \
  return hipErrorInvalidValue;

}  // namespace

hipError_t launch_sparse_decode(const Shape& s, int inst0, int ninst, const void* q, const void* K, const void* V,
                                int t_cur, const int32_t* idx, const int32_t* cnt, float* out, float* row,
                                size_t row_stride, float* ws, hipStream_t st) {
  const WsLayout wl = ws_layout(s);
  SparseArgs a;
  a.q = q; a.K = K; a.V = V; a.idx = idx; a.cnt = cnt; a.out = out; a.row = row; a.row_stride = row_stride;
  a.merge_count = reinterpret_cast<unsigned long long*>(ws + wl.merge_count);
  a.merge_nonce = new_nonce(kTicketBits);
  a.part_ml = ws + wl.part_ml; a.part_acc = ws + wl.part_acc; a.part_bmp = ws + wl.part_bmp;
  a.t_cap = s.t_cap; a.nb_cap = s.nb_cap; a.k = s.k; a.b = s.b; a.log2b = ilog2(s.b); a.t_cur = t_cur;
  a.nb_cur = (t_cur + s.b - 1) / s.b;
  a.n_split = s.n_split;
  a.blk_per_split = (s.k + s.n_split - 1) / s.n_split;
  a.inst0 = inst0;
  a.part_first = 0;
  a.piece_blocks = s.k;
  a.ml_unit = kLog2E;
  a.table = s.table; a.n_phys = s.n_phys;
  a.pred = s.select_by; a.n_sink = s.n_sink; a.n_local = s.n_local; a.sel_at = 0;
  AP_DISPATCH(run_sparse, s, ninst, a, st)
}

hipError_t static_scratch(float** ptr, size_t* bytes) {
  constexpr int kMaxDevices = 64;
  static std::mutex mu;
  static void* addr[kMaxDevices] = {};
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(mu);
  if (addr[dev] == nullptr) {                            // once per device, with that device current
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    if (p == nullptr) return hipErrorInvalidSymbol;
    addr[dev] = p;
  }
  *ptr = static_cast<float*>(addr[dev]);
  *bytes = kStaticScratchBytes;
  return hipSuccess;
}

hipError_t launch_calibrate(const Shape& s, const void* q, const void* K, int t_cur, float* row, float* ws,
                            hipStream_t st) {
  const WsLayout wl = ws_layout(s);
  CalibArgs a;
  a.q = q; a.K = K; a.row = row; a.cal_ml = ws + wl.cal_ml; a.cal_bmp = ws + wl.cal_bmp;
  a.t_cap = s.t_cap; a.nb_cap = s.nb_cap; a.b = s.b; a.log2b = ilog2(s.b); a.t_cur = t_cur;
  a.nb_cur = (t_cur + s.b - 1) / s.b;
  a.chunk_blocks = calib_chunk_tokens(s, t_cur) / s.b;
  a.ml_unit = kLog2E;
  a.n_chunks = (a.nb_cur + a.chunk_blocks - 1) / a.chunk_blocks;
  a.n_units = a.n_chunks * s.n_inst;
  a.chunk_slots = s.calib_chunks;
  a.table = s.table; a.n_phys = s.n_phys;
  AP_DISPATCH(run_calib, s, a, st)
}

}  // namespace ap
