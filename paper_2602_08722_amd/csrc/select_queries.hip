// Query sub-selection and group pre-aggregation (Alg. 1, first block and the normalise / group-mean steps;
// Sec. 3.1, 3.3).
// Memory reads are spread over the whole chip (one compute unit alone cannot pull a head's queries at more
// than a few tens of GB/s), and every kernel requests all the rows it needs before it uses the first.
//   sq_partial_sums : per (b, q-head, token tile) column sums of Q                     -> ws.part
//   sq_cosine       : per (b, q-head, token tile) mean query from the partials (fixed order, so the
//                     result is bit-reproducible), then CosSim(q_i, M_Q) for the tile   -> ws.cos
//   sq_select       : per (b, q-head) the N' lowest cosines in rank order (histogram of register-held
//                     keys + rank by counting)                                          -> q_idx
//   sq_head_select  : the three steps above in one block per (b, q-head), for short chunks (the rows of a head fit the
//                     block's registers)
//   sq_qbar         : per (b, KV head, r) unit-normalise the r-th retained query of each head of the
//                     group and average                                                 -> qbar
#include "common.hip.h"
#include "kernels.h"
#include "qbar_row.hip.h"
#include "score_tile.hip.h"

namespace quoka {

constexpr int kSqTile = 64;     // tokens per tile
constexpr int kSqThreads = 256;

template <typename T>
struct Raw8;   // eight consecutive elements as loaded
template <>
struct Raw8<uint16_t> {
  u32x4 r;
  // What was formed from the row before is formed again, not kept beside it (sq_head_select, d 128, 8 rows a thread: 94 -> 62 registers,
  // 16 rows: 97 instead of 128 and spills).
  __device__ __forceinline__ void pin() { asm volatile("" : "+v"(r)); }
  __device__ __forceinline__ void load(const uint16_t* p) { r = *reinterpret_cast<const u32x4*>(p); }
  __device__ __forceinline__ void widen(float (&v)[8]) const {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      v[2 * i] = __uint_as_float(r[i] << 16);
      v[2 * i + 1] = __uint_as_float(r[i] & 0xFFFF0000u);
    }
  }
};
template <>
struct Raw8<float> {
  float4 a, b;
  __device__ __forceinline__ void load(const float* p) {
    a = *reinterpret_cast<const float4*>(p);
    b = *reinterpret_cast<const float4*>(p + 4);
  }
  __device__ __forceinline__ void widen(float (&v)[8]) const {
    v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w;
    v[4] = b.x; v[5] = b.y; v[6] = b.z; v[7] = b.w;
  }
};

// ---------------------------------------------------------------------------------------------
template <typename T, int D>
__global__ __launch_bounds__(kSqThreads) void sq_partial_sums(Dims dm, const T* __restrict__ q, float* __restrict__ part,
                                                             int n_tiles) {
  constexpr int CG = D / 8;              // lanes per row (8 elements each)
  constexpr int RPB = kSqThreads / CG;   // rows handled concurrently
  const int tile = blockIdx.x, h = blockIdx.y, b = blockIdx.z;
  const int C = dm.chunk(b);
  const int cg = threadIdx.x % CG, rr = threadIdx.x / CG;
  const T* base = q + b * dm.qs[0] + h * dm.qs[1];
  float acc[8] = {0, 0, 0, 0, 0, 0, 0, 0};
  const int t0 = tile * kSqTile;
  Raw8<T> rows[kSqTile / RPB];   // all requested before the first is used
#pragma unroll
  for (int u = 0; u < kSqTile / RPB; ++u) rows[u].load(base + (size_t)min(t0 + u * RPB + rr, C - 1) * dm.qs[2] + cg * 8);
#pragma unroll
  for (int u = 0; u < kSqTile / RPB; ++u) {
    float v[8];
    rows[u].widen(v);
    if (t0 + u * RPB + rr < C) {
#pragma unroll
      for (int e = 0; e < 8; ++e) acc[e] += v[e];
    }
  }
  __shared__ float red[RPB][D];
#pragma unroll
  for (int e = 0; e < 8; ++e) red[rr][cg * 8 + e] = acc[e];
  __syncthreads();
  if (threadIdx.x < D) {
    float s = 0.f;
    for (int i = 0; i < RPB; ++i) s += red[i][threadIdx.x];
    part[((size_t)(b * dm.n_q + h) * n_tiles + tile) * D + threadIdx.x] = s;
  }
}

// Norm of the mean by one thread, summed in order.
template <int D>
__device__ __forceinline__ float norm_in_order(const float* mean) {   // 16-byte aligned
  float ss = 0.f;
#pragma unroll
  for (int i = 0; i < D; i += 4) {
    const float4 v = *reinterpret_cast<const float4*>(mean + i);
    ss += v.x * v.x;
    ss += v.y * v.y;
    ss += v.z * v.z;
    ss += v.w * v.w;
  }
  return fmaxf(sqrtf(ss), kNormEps);
}

// ---------------------------------------------------------------------------------------------
template <typename T, int D>
__global__ __launch_bounds__(kSqThreads) void sq_cosine(Dims dm, const T* __restrict__ q, const float* __restrict__ part,
                                                       float* __restrict__ cosv, int n_tiles) {
  constexpr int CG = D / 8;
  constexpr int RPB = kSqThreads / CG;
  const int tile = blockIdx.x, h = blockIdx.y, b = blockIdx.z;
  const int C = dm.chunk(b);
  __shared__ __align__(16) float mean[D];
  __shared__ float mnorm;
  const int cg = threadIdx.x % CG, rr = threadIdx.x / CG;
  const T* base = q + b * dm.qs[0] + h * dm.qs[1];
  const int t0 = tile * kSqTile;
  if (threadIdx.x < D) {
    const float* p = part + (size_t)(b * dm.n_q + h) * n_tiles * D + threadIdx.x;
    float s = 0.f;
    for (int i0 = 0; i0 < n_tiles; i0 += 8) {   // 8 partials requested at a time, summed in tile order
      float t[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) t[u] = p[(size_t)min(i0 + u, n_tiles - 1) * D];
#pragma unroll
      for (int u = 0; u < 8; ++u)
        if (i0 + u < n_tiles) s += t[u];
    }
    mean[threadIdx.x] = s / (float)C;
  }
  Raw8<T> rows[kSqTile / RPB];   // travel while the mean's norm is formed
#pragma unroll
  for (int u = 0; u < kSqTile / RPB; ++u) rows[u].load(base + (size_t)min(t0 + u * RPB + rr, C - 1) * dm.qs[2] + cg * 8);
  __syncthreads();
  if (threadIdx.x == kSqThreads - kWave) mnorm = norm_in_order<D>(mean);
  float m[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) m[e] = mean[cg * 8 + e];
  float dots[kSqTile / RPB], qn[kSqTile / RPB];   // (the norm of the mean is needed last)
#pragma unroll
  for (int u = 0; u < kSqTile / RPB; ++u) {
    float v[8];
    rows[u].widen(v);
    float dot = 0.f, qq = 0.f;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      dot += v[e] * m[e];
      qq += v[e] * v[e];
    }
    if constexpr (CG == 16) {   // a query row is exactly one 16-lane DPP row
      dot = row16_sum(dot);
      qq = row16_sum(qq);
    } else {
      dot = group_sum<CG>(dot);
      qq = group_sum<CG>(qq);
    }
    dots[u] = dot;
    qn[u] = fmaxf(sqrtf(qq), kNormEps);
  }
  __syncthreads();
  const float mn = mnorm;
#pragma unroll
  for (int u = 0; u < kSqTile / RPB; ++u) {
    const int tok = t0 + u * RPB + rr;
    if (cg == 0 && tok < C) cosv[(size_t)(b * dm.n_q + h) * dm.C + tok] = dots[u] / (qn[u] * mn) + 0.0f;
  }
}

// ---------------------------------------------------------------------------------------------
constexpr int kSelThreads = 1024;

// The N' lowest keys of a block's register-held order-preserving keys, in rank order, to out[0..n_keep).  Thread t holds
// positions lo .. lo+IPT-1.  A histogram over 1024 equal bins of the cosines' range finds the bin that holds the N'-th lowest;
// the keys up to that bin, a few more than N', are listed in any order, and the rank of each among them is counted: one
// barrier for the range, one for the histogram, one for the list.  Where they do not fit the list (many equal cosines,
// or nearly so) or a cosine is not finite, the exact cut is found by radix select first.
// (Radix select and an ordered compaction for every head, three to four passes: sq_select 5.5 -> 4.0 us at 8 to 32 heads of 64 to
// 1024 cosines, 9.3 -> 6.8 at 4096.)
constexpr int kSqBins = 1024, kSqRowPitch = 20;   // 16 bins a lane; the pitch spreads 16-byte reads over the banks
constexpr int kMaxCands = 256;
struct __align__(16) RankLds {
  uint32_t hist[kWave * kSqRowPitch];
  unsigned long long cand[kMaxCands];   // key in the high half, position in the low one
  uint32_t wmin[kSelThreads / kWave], wmax[kSelThreads / kWave];
  uint32_t n_listed;
  RadixSelectLds rs;
  uint32_t wsum[kSelThreads / kWave + 1];
};
static_assert(alignof(RankLds) >= sizeof(u32x4), "the histogram is read 16 bytes at a time");

__device__ __forceinline__ float okey_value(uint32_t k) { return __uint_as_float(k & 0x80000000u ? k ^ 0x80000000u : ~k); }

// (before the first barrier of the caller, or with one between this and the selection)
__device__ __forceinline__ void clear_rank_lds(RankLds& L) {
  for (int i = threadIdx.x; i < kWave * kSqRowPitch; i += kSelThreads) L.hist[i] = 0u;
  if (threadIdx.x == 0) L.n_listed = 0u;
}

template <int IPT>
__device__ __forceinline__ void select_lowest_ranked(const uint32_t (&key)[IPT], uint32_t valid, int lo, int n_keep,
                                                     RankLds& L, int32_t* __restrict__ out) {
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  uint32_t kmin = 0xFFFFFFFFu, kmax = 0u;
#pragma unroll
  for (int j = 0; j < IPT; ++j) {
    if ((valid >> j) & 1u) {
      kmin = min(kmin, key[j]);
      kmax = max(kmax, key[j]);
    }
  }
  kmin = wave_min_u32(kmin);
  kmax = wave_max_u32(kmax);
  if (lane == 0) {
    L.wmin[w] = kmin;
    L.wmax[w] = kmax;
  }
  __syncthreads();
  constexpr int NW = kSelThreads / kWave;
  kmin = wave_min_u32(L.wmin[lane % NW]);
  kmax = wave_max_u32(L.wmax[lane % NW]);
  if (kmin == kmax) {   // all cosines are equal: the lowest positions, in order (block-uniform)
#pragma unroll
    for (int j = 0; j < IPT; ++j)
      if (lo + j < n_keep) out[lo + j] = lo + j;
    return;
  }
  const float fmin_ = okey_value(kmin), range = okey_value(kmax) - fmin_;
  // (infinities and NaN have the outermost keys, so a finite range means that every cosine is finite)
  bool listed = range < INFINITY;   // wave-uniform, and the same in every wave
  int bin[IPT];
  int cut_bin = 0;
  uint32_t n_c = 0;
  if (listed) {
    const float per = fminf((float)(kSqBins - 1) / range, 3.0e38f);   // monotone in the cosine, whatever it rounds to
#pragma unroll
    for (int j = 0; j < IPT; ++j) {
      bin[j] = min(max((int)((okey_value(key[j]) - fmin_) * per), 0), kSqBins - 1);
      if ((valid >> j) & 1u) atomicAdd(&L.hist[bin[j] + (bin[j] >> 4) * (kSqRowPitch - 16)], 1u);
    }
    __syncthreads();
    // every wave finds the cut's bin for itself; lane l has bins 16 l .. 16 l + 15
    uint32_t c[16];
    uint32_t sum = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const u32x4 v = *reinterpret_cast<const u32x4*>(&L.hist[lane * kSqRowPitch + 4 * i]);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        c[4 * i + e] = v[e];
        sum += v[e];
      }
    }
    const uint32_t upto = wave_incl_scan_u32(sum), need = (uint32_t)n_keep;
    uint32_t run = upto - sum;
    int found = 0;
    uint32_t at = upto;
#pragma unroll
    for (int i = 0; i < 16; ++i) {   // the lane's first bin with which the running count reaches n_keep
      run += c[i];
      const bool before = run < need;
      found += before ? 1 : 0;
      at = !before && at > run ? run : at;
    }
    const unsigned long long hit = __builtin_amdgcn_ballot_w64(upto - sum < need && need <= upto);   // exactly one lane
    const int src = hit ? (int)__builtin_ctzll(hit) : 63;
    cut_bin = __builtin_amdgcn_readlane(16 * lane + min(found, 15), src);
    n_c = (uint32_t)__builtin_amdgcn_readlane((int)at, src);
    listed = n_c <= (uint32_t)kMaxCands;
  }
  if (listed) {
#pragma unroll
    for (int j = 0; j < IPT; ++j) {
      const bool in = ((valid >> j) & 1u) && bin[j] <= cut_bin;
      const unsigned long long m = __builtin_amdgcn_ballot_w64(in);
      if (m != 0) {   // wave-uniform; any order will do
        uint32_t slot = 0;
        if (lane == 0) slot = atomicAdd(&L.n_listed, (uint32_t)__popcll(m));
        slot = (uint32_t)__builtin_amdgcn_readfirstlane((int)slot) + (uint32_t)__popcll(m & ((1ull << lane) - 1ull));
        if (in && slot < (uint32_t)kMaxCands) L.cand[slot] = ((unsigned long long)key[j] << 32) | (uint32_t)(lo + j);
      }
    }
  } else {
    // key of the n_keep-th smallest cosine; need_eq: how many elements equal to it are kept (lowest positions first)
    uint32_t tau, need_eq;
    block_radix_select<IPT, false>(key, valid, (uint32_t)n_keep, L.rs, &tau, &need_eq);
    uint32_t eq = 0, tot;
#pragma unroll
    for (int j = 0; j < IPT; ++j) eq += ((valid >> j) & 1u) && key[j] == tau ? 1u : 0u;
    uint32_t eq_rank = block_excl_scan<kSelThreads>(eq, L.wsum, &tot);
#pragma unroll
    for (int j = 0; j < IPT; ++j) {
      const bool is_eq = ((valid >> j) & 1u) && key[j] == tau;
      if (((valid >> j) & 1u) && (key[j] < tau || (is_eq && eq_rank < need_eq))) {
        const uint32_t slot = atomicAdd(&L.n_listed, 1u);
        if (slot < (uint32_t)kMaxCands) L.cand[slot] = ((unsigned long long)key[j] << 32) | (uint32_t)(lo + j);
      }
      eq_rank += is_eq ? 1u : 0u;
    }
    n_c = (uint32_t)n_keep;
  }
  __syncthreads();
  // rank by counting: P consecutive lanes share one listed query and split the comparisons (equal cosines: the lower
  // position first, as the low halves say)
  int e_cap = 16;
  while (e_cap < (int)n_c) e_cap <<= 1;
  const int P = kSelThreads / e_cap;         // 4 .. 64
  const int e = tid / P, part = tid % P;
  int rank = 0;
  const unsigned long long mine = L.cand[min(e, (int)n_c - 1)];
  if (e < (int)n_c)
    for (int jj = part; jj < (int)n_c; jj += P) rank += L.cand[jj] < mine ? 1 : 0;
  for (int o = 1; o < P; o <<= 1) rank += __shfl_xor(rank, o, kWave);
  if (e < (int)n_c && part == 0 && rank < n_keep) out[rank] = (int32_t)(uint32_t)mine;
}

template <int IPT>
__global__ __launch_bounds__(kSelThreads) void sq_select(Dims dm, const float* __restrict__ cosv,
                                                        int32_t* __restrict__ q_idx, int n_keep) {
  __shared__ RankLds L;
  const int h = blockIdx.x, b = blockIdx.y;
  const int C = dm.chunk(b);
  const float* cv = cosv + (size_t)(b * dm.n_q + h) * dm.C;
  const int lo = threadIdx.x * IPT;
  uint32_t key[IPT];
  uint32_t valid = 0u;
#pragma unroll
  for (int j = 0; j < IPT; ++j) {
    const bool in = lo + j < C;
    key[j] = in ? okey(cv[lo + j]) : 0xFFFFFFFFu;
    valid |= (in ? 1u : 0u) << j;
  }
  clear_rank_lds(L);   // (the selection's first barrier comes before it counts)
  select_lowest_ranked<IPT>(key, valid, lo, n_keep, L, q_idx + (size_t)(b * dm.n_q + h) * n_keep);
}

// ---------------------------------------------------------------------------------------------
// Mean, cosines and selection of one (b, q-head) in one block, for chunks short enough that the block can hold the
// head's queries in registers: every row is requested at once (one memory latency; a compute unit that fetches a
// few rows per thread at a time pulls only a few tens of GB/s) and read only once.
// Column sums, two orders.  TILED: the very sums of the tiled kernels -- the rows of a 64-token tile by the same groups, the
// groups of a tile in order, the tiles in order, the norm in order -- so a call may take either route, bit for bit.
// Otherwise (batches, see select_queries_one_block): per group of concurrently handled rows over the whole chunk, the groups in
// order; its rounding differs from the tiled one's in the last bits, and the two are never mixed within one call.
template <typename T, int D, int NR, bool TILED>   // NR: rows per thread (all held in registers)
__global__ __launch_bounds__(kSelThreads) void sq_head_select(Dims dm, const T* __restrict__ q,
                                                             int32_t* __restrict__ q_idx, int n_keep) {
  constexpr int CG = D / 8;                  // lanes per row (8 elements each)
  constexpr int RPB = kSelThreads / CG;      // rows handled concurrently
  constexpr int IPT = (RPB * NR + kSelThreads - 1) / kSelThreads;   // cosines per thread in the selection
  constexpr int RT = kSqThreads / CG;        // TILED: rows of a tile handled concurrently, as in sq_partial_sums ...
  constexpr int UT = kSqTile / RT;           // ... and rows of a tile per thread
  constexpr int TB = kSelThreads / kSqThreads;   // TILED: tiles handled concurrently
  static_assert(!TILED || NR % UT == 0, "whole tiles");
  constexpr int NT = TILED ? NR / UT * TB : 1;
  __shared__ RankLds L;
  __shared__ __align__(16) float mean[D];
  __shared__ float mnorm;
  __shared__ float buf[RPB * D];             // column partials, then products and squared norms (2 RPB NR <= RPB D)
  __shared__ float tsum[NT * D];
  const int h = blockIdx.x, b = blockIdx.y;
  const int C = dm.chunk(b);
  const int tid = threadIdx.x;
  const int cg = tid % CG, rr = TILED ? (tid / CG) % RT : tid / CG;
  // token of a thread's register u
  auto token = [&](int u) __attribute__((always_inline)) {
    if constexpr (TILED) return (tid / kSqThreads + TB * (u / UT)) * kSqTile + (u % UT) * RT + rr;
    return u * RPB + rr;
  };
  const T* base = q + b * dm.qs[0] + h * dm.qs[1];
  Raw8<T> rows[NR];
#pragma unroll
  for (int u = 0; u < NR; ++u) rows[u].load(base + (size_t)min(token(u), C - 1) * dm.qs[2] + cg * 8);
  clear_rank_lds(L);
  // ---- column sums, mean ----
  float acc[8];
#pragma unroll
  for (int u = 0; u < NR; ++u) {
    if (u == 0 || (TILED && u % UT == 0)) {
#pragma unroll
      for (int e = 0; e < 8; ++e) acc[e] = 0.f;
    }
    float v[8];
    rows[u].widen(v);
    if (token(u) < C) {
#pragma unroll
      for (int e = 0; e < 8; ++e) acc[e] += v[e];
    }
    if (TILED && u % UT == UT - 1) {   // four tiles at a time through the buffer
      if (u >= UT) __syncthreads();    // (the sums of the four before have been read)
#pragma unroll
      for (int e = 0; e < 8; ++e) buf[(tid / CG) * D + cg * 8 + e] = acc[e];
      __syncthreads();
      if (tid < TB * D) {
        const float* p = buf + (tid / D) * RT * D + tid % D;
        float s = 0.f;
#pragma unroll
        for (int i = 0; i < RT; ++i) s += p[i * D];
        tsum[(u / UT * TB) * D + tid] = s;
      }
    }
  }
  if constexpr (!TILED) {
#pragma unroll
    for (int e = 0; e < 8; ++e) buf[rr * D + cg * 8 + e] = acc[e];
  }
  __syncthreads();
  if (tid < D) {
    float s = 0.f;
    if constexpr (TILED) {
#pragma unroll
      for (int i = 0; i < NT; ++i) s += tsum[i * D + tid];
    } else {
      for (int i = 0; i < RPB; ++i) s += buf[i * D + tid];
    }
    mean[tid] = s / (float)C;
  }
  __syncthreads();   // (also: the partials in buf are dead from here on)
  if constexpr (TILED) {
    if (tid == kSelThreads - kWave) mnorm = norm_in_order<D>(mean);
  } else if (tid >= kSelThreads - kWave) {   // one wave: squared norm of the mean
    const int lane = tid & 63;
    float ss = 0.f;
    for (int i = lane; i < D; i += 64) ss += mean[i] * mean[i];
    ss = wave64_sum(ss);
    if (lane == 0) mnorm = fmaxf(sqrtf(ss), kNormEps);
  }
  float m[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) m[e] = mean[cg * 8 + e];
  // ---- cosines of the rows held in registers.  The norm of the mean is needed last: products and squared norms wait for it in LDS, and
  // the root and the division are then taken once a token, not by every lane of its row.  (With the registers that this and pin()
  // free: 32 heads of 423 tokens 12.0 -> 10.9 us, 256 of 512 17.1 -> 15.7, float32 32 of 512 13.8 -> 11.7.) ----
#pragma unroll
  for (int u = 0; u < NR; ++u) {
    if constexpr (sizeof(T) == 2) rows[u].pin();
    float v[8];
    rows[u].widen(v);
    float dot = 0.f, qq = 0.f;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      dot += v[e] * m[e];
      qq += v[e] * v[e];
    }
    if constexpr (CG == 16) {
      dot = row16_sum(dot);
      qq = row16_sum(qq);
    } else {
      dot = group_sum<CG>(dot);
      qq = group_sum<CG>(qq);
    }
    if (cg == 0 && token(u) < C) {
      buf[token(u)] = dot;
      buf[RPB * NR + token(u)] = qq;
    }
  }
  __syncthreads();
  const int lo = tid * IPT;
  const float mn = mnorm;
  uint32_t key[IPT];
  uint32_t valid = 0u;
#pragma unroll
  for (int j = 0; j < IPT; ++j) {
    const bool in = lo + j < C;
    const int t = in ? lo + j : 0;
    const float qn = fmaxf(sqrtf(buf[RPB * NR + t]), kNormEps);
    key[j] = in ? okey(buf[t] / (qn * mn) + 0.0f) : 0xFFFFFFFFu;
    valid |= (in ? 1u : 0u) << j;
  }
  select_lowest_ranked<IPT>(key, valid, lo, n_keep, L, q_idx + (size_t)(b * dm.n_q + h) * n_keep);
}

// ---------------------------------------------------------------------------------------------
// One wave per (r, kv, b); GU: heads of the group whose rows travel, and whose norms form, side by side (all of them: with the
// positions in one vector load and no branch per head, the query stage of one KV head of 16, d 128, 600 tokens takes 15.8 us
// instead of 18.6, of 8 KV heads of 4 14.2 instead of 14.9).
template <typename T, int D, int RULE, int GU>
__global__ __launch_bounds__(64) void sq_qbar(Dims dm, const T* __restrict__ q, int32_t* __restrict__ q_idx,
                                             float* __restrict__ qbar, int n_keep, uint32_t* __restrict__ zero,
                                             uint32_t zero_words, uint16_t* __restrict__ terms) {
  constexpr int EPL = D / 64;
  clear_words(zero, zero_words);   // side job of the fused call: histograms and counters of the key-selection stage
  const int r = blockIdx.x, kv = blockIdx.y, b = blockIdx.z;
  const int lane = threadIdx.x;
  if (r >= n_keep) return;   // (such a block only clears)
  float row[EPL];
  qbar_row<T, D, RULE, GU, true>(dm, q, q_idx, n_keep, r, kv, b, lane, true, row);
  float* out = qbar + ((size_t)(b * dm.n_kv + kv) * n_keep + r) * D;
#pragma unroll
  for (int e = 0; e < EPL; ++e) out[lane * EPL + e] = row[e];
  if (terms != nullptr) {   // (kernel-uniform)
    uint16_t* th = terms + (size_t)(b * dm.n_kv + kv) * TermsLayout<D>::head_elems(n_keep);
    uint16_t t[3][EPL];
#pragma unroll
    for (int e = 0; e < EPL; ++e) {
      const __bf16 hi = (__bf16)row[e];
      const float r1 = row[e] - (float)hi;
      const __bf16 mid = (__bf16)r1;
      t[0][e] = __builtin_bit_cast(uint16_t, hi);
      t[1][e] = __builtin_bit_cast(uint16_t, mid);
      t[2][e] = __builtin_bit_cast(uint16_t, (__bf16)(r1 - (float)mid));
    }
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      uint16_t* p = th + TermsLayout<D>::at(r, lane * EPL, k);
      if constexpr (EPL == 2) {
        *reinterpret_cast<uint32_t*>(p) = t[k][0] | ((uint32_t)t[k][1] << 16);
      } else {
        *p = t[k][0];
      }
    }
  }
}

// ---------------------------------------------------------------------------------------------
// One block per head for everything where that is the faster, one launch instead of three.  Short chunks, whatever the heads, in
// the sums of the tiled kernels: up to kHeadTokens tokens (query stage, bf16, d 128: 12 heads of 128 tokens 15.2 -> 10.2 us, 32 of
// 423 15.8 -> 10.9; float32 32 of 512 11.7).  From there on one compute unit per head pulls too little (32 heads of 1024 tokens
// 15.5 against 14.7 us), so calls of few heads spread the two reads of Q over the whole chip.
// Batches, where the heads alone give half the compute units a block and the block can hold the head (8 rows of 8 elements per
// thread): 256 heads of 512 tokens 14.8 us against 24 us.  Their sums differ in the last bits, and cosines that differ in theirs
// only can change ranks, so that line stays where it is.  (It goes by the batch of the whole call and the chunk's own length; how
// many chunks of a prompt share a launch does not count.)
constexpr int kHeadTokens = 512;
constexpr int kRowsPerThread = 8;
bool select_queries_one_block(const Dims& dm) {
  const int rows_at_once = kSelThreads / (dm.d / 8);
  const int sequences = dm.prompt_chunks ? dm.ls : dm.b;   // (ls: the batch of the whole call)
  return dm.C <= rows_at_once * kRowsPerThread && sequences * dm.n_q >= 128;
}

// bf16 calls of 64 heads or more (sequences, and chunks of a prompt that share a launch, count alike: the sums are the tiled kernels')
// up to kManyTokens tokens: Q is read once instead of twice, and that pays as soon as a good part of the compute units has a head.
// Query stage, d 128: 64 heads of 1024 tokens 16.9 -> 16.0 us, 128 23.0 -> 18.3, 256 36.1 -> 24.3, 512 63.4 -> 47.8; d 64 0.97 - 0.99 of the
// time for 64 heads, 0.90 - 0.96 for 112 to 256, 0.63 - 0.82 beyond, wherever it was measured (513 - 1024 tokens, up to 4096 heads).
// At d 128 a head takes its compute unit long enough that the last round of blocks counts: 260 heads of 513 tokens 24.9 -> 28.3, 520 of
// 513 43.9 -> 46.2, and 64 of 513 14.5 -> 14.6.  The line there is a fit of both times, in us, to 2810 calls of up to 768 heads (with it they
// take 0.01 % more than the better route on the mean, 2.6 % at most; one block throughout 1 and 14 %); beyond that, rounds are many and one
// block is the faster, 0.66 - 0.98.
// Whole calls over 8192 keys, 1024 tokens: 8 x 32 heads 263 -> 251 us, 4 x 32 145 -> 140, 64 84.9 -> 84.1; with 48 heads even, with 32, 16
// and 8 1 to 3 % slower.  (Float32 heads of d 64 gain 2 to 3 % of the stage, of d 128 do not fit; 2048 tokens of d 64 gain where the heads
// nearly fill the last round, 256 40 -> 31 us, and lose elsewhere: neither is built.)
constexpr int kManyTokens = 1024, kComputeUnits = 256;
static bool select_queries_many_heads(const Dims& dm) {
  const int heads = dm.n_q * dm.b, rounds = (heads + kComputeUnits - 1) / kComputeUnits;
  if (dm.C > kManyTokens || heads < 64) return false;
  const float c = (float)dm.C / 1024.f;
  return dm.d == 64 || rounds > 3 || (float)rounds * (7.8f + 2.0f * c) < 6.5f + (float)heads * c * (4.0f / 64.f);
}

template <typename T, int D, int RULE>
static void launch_qbar(const Dims& dm, const T* q, int32_t* q_idx, float* qbar, int n_keep, hipStream_t st, uint32_t* zero,
                        uint32_t zero_words, uint16_t* terms) {
  // (what is cleared, 128 to 260 KiB for up to 16 heads, wants more than the blocks of a few queries)
  const int heads = dm.n_kv * dm.b, least = zero != nullptr ? (64 + heads - 1) / heads : 0;
  const dim3 grid(n_keep > least ? n_keep : least, dm.n_kv, dm.b);
  if (dm.g <= 4) {
    hipLaunchKernelGGL((sq_qbar<T, D, RULE, 4>), grid, dim3(64), 0, st, dm, q, q_idx, qbar, n_keep, zero, zero_words, terms);
  } else if (dm.g <= 8) {
    hipLaunchKernelGGL((sq_qbar<T, D, RULE, 8>), grid, dim3(64), 0, st, dm, q, q_idx, qbar, n_keep, zero, zero_words, terms);
  } else {
    hipLaunchKernelGGL((sq_qbar<T, D, RULE, 16>), grid, dim3(64), 0, st, dm, q, q_idx, qbar, n_keep, zero, zero_words, terms);
  }
}

template <typename T, int D>
static hipError_t launch_typed(const Dims& dm, const void* q, int32_t* q_idx, float* qbar, float* ws_part,
                               float* ws_cos, hipStream_t st, uint32_t* zero, uint32_t zero_words,
                               uint16_t* terms) {
  const int n_keep = dm.n_ret < dm.C ? dm.n_ret : dm.C;
  const T* qp = static_cast<const T*>(q);
  if (dm.C <= dm.n_ret) {
    launch_qbar<T, D, kIdentity>(dm, qp, q_idx, qbar, n_keep, st, zero, zero_words, terms);
  } else if (dm.flags & QUOKA_SELECT_UNIFORM) {
    launch_qbar<T, D, kUniform>(dm, qp, q_idx, qbar, n_keep, st, zero, zero_words, terms);
  } else {
    const dim3 sgrid(dm.n_q, dm.b), sblock(kSelThreads);
    const int ipt = (dm.C + kSelThreads - 1) / kSelThreads;
    if (select_queries_one_block(dm)) {
      hipLaunchKernelGGL((sq_head_select<T, D, kRowsPerThread, false>), sgrid, sblock, 0, st, dm, qp, q_idx, n_keep);
    } else if (dm.C <= kHeadTokens / 2) {
      hipLaunchKernelGGL((sq_head_select<T, D, kHeadTokens / 2 * D / 8 / kSelThreads, true>), sgrid, sblock, 0, st, dm, qp, q_idx,
                         n_keep);
    } else if (dm.C <= kHeadTokens) {
      hipLaunchKernelGGL((sq_head_select<T, D, kHeadTokens * D / 8 / kSelThreads, true>), sgrid, sblock, 0, st, dm, qp, q_idx,
                         n_keep);
    } else if (sizeof(T) == 2 && select_queries_many_heads(dm)) {
      hipLaunchKernelGGL((sq_head_select<uint16_t, D, kManyTokens * D / 8 / kSelThreads, true>), sgrid, sblock, 0, st, dm,
                         static_cast<const uint16_t*>(q), q_idx, n_keep);
    } else {
      const int n_tiles = (dm.C + kSqTile - 1) / kSqTile;
      dim3 grid(n_tiles, dm.n_q, dm.b);
      hipLaunchKernelGGL((sq_partial_sums<T, D>), grid, dim3(kSqThreads), 0, st, dm, qp, ws_part, n_tiles);
      hipLaunchKernelGGL((sq_cosine<T, D>), grid, dim3(kSqThreads), 0, st, dm, qp, ws_part, ws_cos, n_tiles);
      if (ipt <= 1) {
        hipLaunchKernelGGL((sq_select<1>), sgrid, sblock, 0, st, dm, ws_cos, q_idx, n_keep);
      } else if (ipt <= 2) {
        hipLaunchKernelGGL((sq_select<2>), sgrid, sblock, 0, st, dm, ws_cos, q_idx, n_keep);
      } else if (ipt <= 4) {
        hipLaunchKernelGGL((sq_select<4>), sgrid, sblock, 0, st, dm, ws_cos, q_idx, n_keep);
      } else {
        hipLaunchKernelGGL((sq_select<8>), sgrid, sblock, 0, st, dm, ws_cos, q_idx, n_keep);
      }
    }
    launch_qbar<T, D, kFromIndex>(dm, qp, q_idx, qbar, n_keep, st, zero, zero_words, terms);
  }
  return hipGetLastError();
}

size_t query_terms_bytes(const Dims& dm) {
  const int n_keep = dm.n_ret < dm.C ? dm.n_ret : dm.C;
  return (size_t)dm.b * dm.n_kv * (dm.d == 64 ? TermsLayout<64>::head_elems(n_keep) : TermsLayout<128>::head_elems(n_keep)) * 2;
}

size_t select_queries_ws_floats(const Dims& dm) {
  const size_t n_tiles = (dm.C + kSqTile - 1) / kSqTile;
  return (size_t)dm.b * dm.n_q * (n_tiles * dm.d + dm.C);
}

hipError_t launch_select_queries(const Dims& dm, int dtype, const void* q, int32_t* q_idx, float* qbar, float* ws,
                                 hipStream_t st, uint32_t* zero, size_t zero_words_sz, uint16_t* terms) {
  const uint32_t zero_words = (uint32_t)zero_words_sz;
  const size_t n_tiles = (dm.C + kSqTile - 1) / kSqTile;
  float* ws_part = ws;
  float* ws_cos = ws + (size_t)dm.b * dm.n_q * n_tiles * dm.d;
  if (dtype == QUOKA_F32) {
    return dm.d == 64 ? launch_typed<float, 64>(dm, q, q_idx, qbar, ws_part, ws_cos, st, zero, zero_words, terms)
                      : launch_typed<float, 128>(dm, q, q_idx, qbar, ws_part, ws_cos, st, zero, zero_words, terms);
  }
  return dm.d == 64 ? launch_typed<uint16_t, 64>(dm, q, q_idx, qbar, ws_part, ws_cos, st, zero, zero_words, terms)
                    : launch_typed<uint16_t, 128>(dm, q, q_idx, qbar, ws_part, ws_cos, st, zero, zero_words, terms);
}

}  // namespace quoka
