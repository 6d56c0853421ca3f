// Key scoring and top-B selection as one stage for long caches (Alg. 1: S = Qbar K^T, S-hat = max, I = topk(S-hat,
// B_SA); the paper's conclusion names a cheaper Qbar K^T as the thing to improve).
//
// The exact product costs three bf16 MFMA terms per key (Qbar is float32).  Only the keys near the cut need it:
//   1. provisional scores p from ONE term (Qbar rounded to bf16).  For every key |p - s| <= eps, where s is the exact
//      score and eps = max_r ||qbar_r - bf16(qbar_r)||_2 (Cauchy-Schwarz with the unit key; the max over queries moves
//      by at most the largest per-query error), plus the float32 accumulation slack of both;
//   2. a histogram of p over 4096 equal bins of [-1, 1] locates the bin of the provisional cut (the B-th largest p);
//   3. keys whose bin lies more than m bins above the cut bin are certainly selected, keys more than m bins below it
//      certainly not (m bins cover 2 eps and the width of the cut bin); the keys in between -- the band, a few per
//      cent -- are scored again with the exact three-term product, by the same tile arithmetic as the streaming
//      kernel, so their scores carry the same float32 bits;
//   4. the best (B - certain) band keys by exact score complete the set; equal scores go to the lower position;
//      indices come out in ascending position.
// The selected set is therefore exactly the top-B of the exact scores, as the separate scoring and top-B calls
// produce it; the `scores` array ends up holding exact values inside the band and provisional values elsewhere.
//
// Up to a size the fused call takes a shorter way to the same lists: exact scores of every key with their histogram
// (score_bf16; for large caches and up to 64 queries score_stream with all three terms), then sel_classify and sel_finish, see
// select_keys_exact_pays and select_keys_streams_exact.
//
// Launch chain (no block ever waits for another block of its launch): provisional scoring with the histogram
// (score_stream.hip), band classification + exact re-scoring per 2048-key tile, one block per head that selects
// among the band candidates and lays out the tiles' output offsets, ordered emission per tile.
#include "common.hip.h"
#include "kernels.h"
#include "score_tile.hip.h"
#include "select_ws.hip.h"

namespace quoka {

struct SelCtx {
  int T, B, head;
  float* sc;
  SelWs w;
};
__device__ __forceinline__ SelCtx sel_ctx(const Dims& dm, float* scores, const int32_t* kv_lens,
                                          const int32_t* budgets, uint32_t* ws, int kv, int b) {
  SelCtx c;
  c.T = max(0, min(kv_lens[b * dm.ls], dm.T_cap));
  c.B = max(0, min(min(budgets[b * dm.ls], c.T), dm.B_max));
  c.head = b * dm.n_kv + kv;
  opaque(scores);
  opaque(ws);
  c.sc = scores + (size_t)c.head * dm.T_max;
  c.w = sel_ws(ws, dm.b * dm.n_kv, c.head, dm.T_max);
  return c;
}
// What a kernel has requested so far leaves before it looks at the head's length and budget.  (Otherwise the compiler moves the fetches
// behind the branches that follow: three or four fetches of 0.4 us in a row ahead of them, see opaque.)
__device__ __forceinline__ void requests_leave(const SelCtx& c) { asm volatile("" ::"s"(c.T), "s"(c.B) : "memory"); }

__global__ void sel_zero(uint32_t* __restrict__ p, size_t n) {
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) p[i] = 0u;
}

// Whole block of kSelThreads: thread t's run of the head's histogram (thread 0 has the highest bins) ...
constexpr int kBandCap = 2 * kSelTile;   // band keys a block lists before it scores them
template <uint32_t PER>
__device__ __forceinline__ void load_hist_run(const uint32_t* __restrict__ hist, uint32_t (&hv)[PER]) {
  const uint32_t top = PER * (kSelThreads - threadIdx.x);   // exclusive upper bin of the run
#pragma unroll
  for (uint32_t i = 0; i < PER; i += 4) {
    const u32x4 v = *reinterpret_cast<const u32x4*>(hist + top - PER + i);
    hv[i] = v[0]; hv[i + 1] = v[1]; hv[i + 2] = v[2]; hv[i + 3] = v[3];
  }
}
// ... and the bin of the cut: scanning from the top, where the running count reaches B (the histogram holds T > B keys).
template <uint32_t PER>
__device__ __forceinline__ int find_cut_bin(const uint32_t (&hv)[PER], uint32_t B, uint32_t* sh, uint32_t* bin) {
  const uint32_t top = PER * (kSelThreads - threadIdx.x);
  uint32_t mine = 0;
#pragma unroll
  for (uint32_t i = 0; i < PER; ++i) mine += hv[i];
  uint32_t tot;
  const uint32_t above = block_excl_scan<kSelThreads>(mine, sh, &tot);
  if (above < B && B <= above + mine) {   // exactly one thread
    uint32_t rem = B - above;
    int found = -1;
#pragma unroll
    for (int j = (int)PER - 1; j >= 0; --j) {   // from this thread's highest bin down
      if (found < 0) {
        if (rem <= hv[j]) {
          found = j;
        } else {
          rem -= hv[j];
        }
      }
    }
    *bin = top - PER + (uint32_t)max(found, 0);
  }
  __syncthreads();
  return (int)*bin;
}

// ---------------------------------------------------------------------------------------------
// Band classification and exact re-scoring.  A block takes `tpb` consecutive 2048-key tiles of one head: it locates
// the band once from the finished histogram, classifies the keys tile after tile and scores the listed band keys exactly.
// (Listing a whole block first and fetching the next rows during the products: 8 x 8 ragged heads 34.5 -> 32.9 us; an
// operand load placed beside the first rows instead of up front costs the second wave per SIMD, 48 us.)
template <int D, int QB>
__global__ __launch_bounds__(kSelThreads) void sel_band_rescore(Dims dm, const float* __restrict__ qbar,
                                                               const uint16_t* __restrict__ kc,
                                                               const int32_t* __restrict__ kv_lens,
                                                               const int32_t* __restrict__ budgets,
                                                               float* __restrict__ scores, uint32_t* __restrict__ ws,
                                                               int n_keep, int tpb) {
  using Cfg = ScoreCfg<D, QB>;
  constexpr int LD = Cfg::LD, CG = Cfg::CG, RPI = Cfg::RPI, NLD = Cfg::NLD;
  __shared__ __align__(16) uint16_t tile[kScTile * LD];
  __shared__ float ssq[2][kScTile];
  __shared__ float smax[2][QB * kScTile];
  __shared__ uint32_t band_loc[kBandCap];        // positions (relative to the block's first key) of the band keys, any order
  __shared__ uint32_t sh[kSelThreads + 2];
  __shared__ uint32_t bc[2];                     // cut bin, candidate slot base
  __shared__ uint32_t n_band;                    // keys in band_loc
  __shared__ uint32_t n_sure[2];                 // per tile parity: keys that are certainly selected

  const int kv = blockIdx.y, b = blockIdx.z;
  const SelCtx c = sel_ctx(dm, scores, kv_lens, budgets, ws, kv, b);
  const int tile_first = blockIdx.x * tpb;
  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int qb = w % QB, kg = w / QB;
  const int li = lane & 31, hf = lane >> 5;

  // What the block needs from memory before it can classify is requested up front, before the cache length is known: the
  // first tile's provisional scores, the histogram and the error bound.
  float p[kSelIPT];
  auto load_p = [&](int t0) __attribute__((always_inline)) {   // positions are clamped to the array
#pragma unroll
    for (int i = 0; i < kSelIPT; ++i) p[i] = c.sc[min(t0 + tid + kSelThreads * i, dm.T_max - 1)];   // coalesced rows
  };
  load_p(tile_first * kSelTile);
  uint32_t hv[kSelBins / kSelThreads];
  load_hist_run(c.w.hist, hv);
  const float d2 = __uint_as_float(c.w.meta[kMetaEps2]);
  requests_leave(c);
  if (c.B == 0 || c.B >= c.T || tile_first * kSelTile >= c.T) return;   // block-uniform
  const int tile_end = min(tile_first + tpb, (c.T + kSelTile - 1) / kSelTile);
  if (tid == 0) n_band = n_sure[0] = n_sure[1] = 0u;
  QueryTerms<D, true> qt;
  qt.load(qbar + (size_t)c.head * n_keep * D, n_keep, qb, li, hf, false);

  const int cut_bin = find_cut_bin(hv, (uint32_t)c.B, sh, &bc[0]);   // of the provisional cut
  // |p - s| <= ||delta|| (exact arithmetic; the scoring launch left the largest squared ||delta|| of the head) plus
  // the float32 accumulation and bin-edge slack of the two computed values
  const float eps = sqrtf(d2) * 1.001f + 4e-6f;
  const int m = (int)ceilf(2.0f * eps * (float)(kSelBins / 2)) + 1;
  const int bin_lo = max(cut_bin - m, 0), bin_hi = min(cut_bin + m, kSelBins - 1);
  if (blockIdx.x == 0 && tid == 0) c.w.meta[kMetaBinHi] = (uint32_t)bin_hi;
  const char* kbase = reinterpret_cast<const char*>(kc + b * dm.kvs[0] + kv * dm.kvs[1]);
  const uint32_t row_bytes = (uint32_t)dm.kvs[2] * 2u;
  const int cg = tid % CG, r0 = tid / CG;

  // ---- exact scores of the listed keys, 128 at a time, by the tile arithmetic of the streaming kernel; the rows of the
  // next 128 travel during the products ----
  const int first_key = tile_first * kSelTile;
  auto rescore = [&](int n) __attribute__((always_inline)) {
    uint32_t slot = 0;
    if (tid == 0) slot = atomicAdd(&c.w.meta[kMetaCand], (uint32_t)n);   // slots in the head's candidate list
    u32x4 R[NLD];
    auto load_rows = [&](int j0) __attribute__((always_inline)) {
#pragma unroll
      for (int i = 0; i < NLD; ++i) {
        const int j = min(j0 + r0 + RPI * i, n - 1);   // tail slots repeat a real row; their scores are not used
        const uint32_t row = (uint32_t)first_key + band_loc[j];
        R[i] = *reinterpret_cast<const u32x4*>(kbase + (row * row_bytes + (uint32_t)cg * 16u));
      }
    };
    load_rows(0);
    for (int j0 = 0; j0 < n; j0 += kScTile) {
      float* ssq_g = ssq[(j0 / kScTile) & 1];     // (a batch's norms and maxima are read while the next one is staged)
      float* smax_g = smax[(j0 / kScTile) & 1];
#pragma unroll
      for (int i = 0; i < NLD; ++i) {
        const int rl = r0 + RPI * i;
        *reinterpret_cast<u32x4*>(tile + rl * LD + cg * 8) = R[i];
        const float ss = row_sumsq<CG>(R[i]);
        if (cg == 0) ssq_g[rl] = ss;
      }
      __syncthreads();
      if (j0 + kScTile < n) load_rows(j0 + kScTile);
      tile_products<D, QB, true>(tile, qt, qb, kg, li, hf, false, smax_g);
      if (j0 == 0 && tid == 0) bc[1] = slot;
      __syncthreads();
      if (tid < kScTile && j0 + tid < n) {
        const float s = tile_score<QB>(smax_g, ssq_g, tid, false, false, n_keep);
        const uint32_t pos = (uint32_t)first_key + band_loc[j0 + tid], at = bc[1] + j0 + tid;
        c.sc[pos] = s;
        c.w.cand_key[at] = max(okey(s), 1u);
        c.w.cand_pos[at] = pos;
      }
    }
  };

  for (int tile_i = tile_first; tile_i < tile_end; ++tile_i) {
    const int t0 = tile_i * kSelTile;
    // ---- classify: certainly selected (counted), band (listed, flagged in the mask), certainly not ----
    uint32_t n_in = 0;
#pragma unroll
    for (int i = 0; i < kSelIPT; ++i) {
      const int tl = tid + kSelThreads * i;
      const bool valid = t0 + tl < c.T;
      const int bin = score_bin(p[i]);
      const bool inb = valid && bin >= bin_lo && bin <= bin_hi;
      n_in += (valid && bin > bin_hi) ? 1u : 0u;
      const unsigned long long bal = __builtin_amdgcn_ballot_w64(inb);
      // positions tl of one wave in one round are 64 consecutive keys: its ballot is two words of the tile's mask
      if (lane == 0) {
        uint32_t* mw = c.w.mask + (size_t)tile_i * (kSelTile / 32) + (kSelThreads * i + 64 * w) / 32;
        mw[0] = (uint32_t)bal;
        mw[1] = (uint32_t)(bal >> 32);
      }
      uint32_t base = 0;
      if (lane == 0 && bal != 0) base = atomicAdd(&n_band, (uint32_t)__popcll(bal));
      base = (uint32_t)__builtin_amdgcn_readfirstlane((int)base);
      if (inb) band_loc[base + __popcll(bal & ((1ull << lane) - 1ull))] = (uint32_t)(t0 - first_key + tl);
    }
    if (tile_i + 1 < tile_end) load_p(t0 + kSelTile);   // the next tile's scores travel
    n_in = wave_incl_scan_u32(n_in);
    if (lane == 63 && n_in) atomicAdd(&n_sure[tile_i & 1], n_in);
    __syncthreads();
    const int n = (int)n_band;
    if (tid == 0) {
      c.w.tile_in[tile_i] = n_sure[tile_i & 1];
      n_sure[tile_i & 1] = 0u;   // (serves the tile after the next, a barrier away)
    }
    if (n > kBandCap - kSelTile || (tile_i + 1 == tile_end && n > 0)) {   // block-uniform: the list may overflow, or it is complete
      rescore(n);
      __syncthreads();
      if (tid == 0) n_band = 0u;
    }
    __syncthreads();   // (n_band has been read, or cleared)
  }
}

// ---------------------------------------------------------------------------------------------
// The cut among n candidates held in registers (thread t's k[i] is number t + NT*i): the `need`-th largest key, and how many
// candidates equal to it are among the `need` largest.  A histogram over 256 equal parts of the keys' range, then the ranks of the
// few keys in the cut's part: three barriers whatever n is, where radix passes need one each for every 8 bits.  False (block-
// uniform) where more than 64 keys share that part.  L.hist and L.n are zero, with a barrier since.
struct __align__(16) CutListLds {
  uint32_t hist[256];
  uint32_t list[kWave];
  uint32_t wmin[16], wmax[16];
  uint32_t n;
};
static_assert(alignof(CutListLds) >= sizeof(u32x4), "the histogram is read 16 bytes at a time");

template <int NT, int R>
__device__ __forceinline__ bool cut_among(const uint32_t (&k)[R], uint32_t n, uint32_t need, CutListLds& L, uint32_t* tau,
                                          uint32_t* need_eq) {
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  uint32_t n_list = n;
  if (n > (uint32_t)kWave) {   // block-uniform
    uint32_t kmin = 0xFFFFFFFFu, kmax = 0u;
#pragma unroll
    for (int i = 0; i < R; ++i) {
      const bool in = (uint32_t)(tid + NT * i) < n;
      kmin = in ? min(kmin, k[i]) : kmin;
      kmax = in ? max(kmax, k[i]) : kmax;
    }
    kmin = wave_min_u32(kmin);
    kmax = wave_max_u32(kmax);
    if (lane == 0) {
      L.wmin[w] = kmin;
      L.wmax[w] = kmax;
    }
    __syncthreads();
    kmin = row16_min_u32(L.wmin[lane % (NT / 64)]);
    kmax = row16_max_u32(L.wmax[lane % (NT / 64)]);
    const uint32_t range = kmax - kmin;
    const int shift = range < 256u ? 0 : 24 - __clz(range);   // range >> shift is 255 at most
#pragma unroll
    for (int i = 0; i < R; ++i)
      if ((uint32_t)(tid + NT * i) < n) atomicAdd(&L.hist[(k[i] - kmin) >> shift], 1u);
    __syncthreads();
    // every wave locates the cut's part for itself; scan position o = 4 * lane + i is part 255 - o
    const u32x4 raw = *reinterpret_cast<const u32x4*>(L.hist + 4 * (63 - lane));
    const uint32_t cc[4] = {raw[3], raw[2], raw[1], raw[0]};
    const uint32_t sum = cc[0] + cc[1] + cc[2] + cc[3];
    const uint32_t inc = wave_incl_scan_u32(sum);
    uint32_t rem = need - (inc - sum);
    const bool hit = inc - sum < need && need <= inc;   // exactly one lane (need <= n)
    int i0 = 0;
#pragma unroll
    for (; i0 < 3; ++i0) {
      if (rem <= cc[i0]) break;
      rem -= cc[i0];
    }
    const unsigned long long bal = __builtin_amdgcn_ballot_w64(hit);
    const int src = bal ? (int)__builtin_ctzll(bal) : 0;
    const uint32_t part = (uint32_t)__builtin_amdgcn_readlane(255 - (4 * lane + i0), src);
    need = (uint32_t)__builtin_amdgcn_readlane((int)rem, src);
#pragma unroll
    for (int i = 0; i < R; ++i) {
      if ((uint32_t)(tid + NT * i) < n && (k[i] - kmin) >> shift == part) {
        const uint32_t slot = atomicAdd(&L.n, 1u);
        if (slot < (uint32_t)kWave) L.list[slot] = k[i];
      }
    }
    __syncthreads();
    n_list = L.n;
    if (n_list > (uint32_t)kWave) return false;
  } else {
    if (tid < (int)n) L.list[tid] = k[0];
    __syncthreads();
  }
  const uint32_t mine = L.list[min(lane, (int)n_list - 1)];
  uint32_t gt = 0, ge = 0;
  for (uint32_t j = 0; j < n_list; ++j) {
    const uint32_t o = L.list[j];
    gt += o > mine ? 1u : 0u;
    ge += o >= mine ? 1u : 0u;
  }
  const unsigned long long bal = __builtin_amdgcn_ballot_w64(gt < need && need <= ge);   // (equal keys all say the same)
  const int src = bal ? (int)__builtin_ctzll(bal) : 0;
  *tau = (uint32_t)__builtin_amdgcn_readlane((int)mine, src);
  *need_eq = need - (uint32_t)__builtin_amdgcn_readlane((int)gt, src);
  return true;
}

struct HeadSelectLds {
  RadixSelectLds rs;
  CutListLds cut;
  uint32_t wsum[kSelHeadThreads / 64 + 1];
};
constexpr int kHeadCands = 4;   // candidates a thread of the head's block holds in registers

// use(value...) for each of n entries of one or two arrays in memory, by a block of NT threads.  Eight loads of a thread are in flight:
// one by one, the list of a head whose scores all share a bin is 512 fetches in a row, in every emitting block (8 heads of
// 131072 equal keys, whole calls, 64 queries 403 -> 187 us, 2 queries 381 -> 164; eight different keys 138 -> 116).  The rest
// goes one by one: with runs that reach past the end, clamped, sel_finish took 88 registers instead of 62, and 8 x 8 ragged heads
// of one query, whole calls, 189 us instead of 180.
constexpr int kListRun = 8;
template <int NT, typename F>
__device__ __forceinline__ void for_each_listed(const uint32_t* __restrict__ a, uint32_t n, F use) {
  uint32_t i = threadIdx.x;
  for (; i + (kListRun - 1) * NT < n; i += kListRun * NT) {
    uint32_t v[kListRun];
#pragma unroll
    for (int j = 0; j < kListRun; ++j) v[j] = a[i + NT * j];
#pragma unroll
    for (int j = 0; j < kListRun; ++j) use(v[j]);
  }
  for (; i < n; i += NT) use(a[i]);
}
template <int NT, typename F>
__device__ __forceinline__ void for_each_listed(const uint32_t* __restrict__ a, const uint32_t* __restrict__ b, uint32_t n, F use) {
  uint32_t i = threadIdx.x;
  for (; i + (kListRun / 2 - 1) * NT < n; i += kListRun / 2 * NT) {
    uint32_t v[kListRun / 2], u[kListRun / 2];
#pragma unroll
    for (int j = 0; j < kListRun / 2; ++j) {
      v[j] = a[i + NT * j];
      u[j] = b[i + NT * j];
    }
#pragma unroll
    for (int j = 0; j < kListRun / 2; ++j) use(v[j], u[j]);
  }
  for (; i < n; i += NT) use(a[i], b[i]);
}

// Radix select (descending) over keys that are read again from memory in every pass: for lists that registers do not hold, of any length,
// and for parts that cut_among does not rank.
template <int NT>
__device__ __forceinline__ void stream_radix_select_desc(const uint32_t* __restrict__ keys, uint32_t n, uint32_t need,
                                                         RadixSelectLds& L, uint32_t* cut_key, uint32_t* need_eq) {
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  for (int i = tid; i < 768; i += NT) (&L.hist[0][0])[i] = 0u;
  uint32_t kmin = 0xFFFFFFFFu, kmax = 0u;
  for_each_listed<NT>(keys, n, [&](uint32_t k) {
    kmin = min(kmin, k);
    kmax = max(kmax, k);
  });
  kmin = wave_min_u32(kmin);
  kmax = wave_max_u32(kmax);
  if (lane == 0) {
    L.wmin[w] = kmin;
    L.wmax[w] = kmax;
  }
  __syncthreads();
  kmin = wave_min_u32(lane < NT / 64 ? L.wmin[lane] : 0xFFFFFFFFu);
  kmax = wave_max_u32(lane < NT / 64 ? L.wmax[lane] : 0u);
  const uint32_t diff = kmin ^ kmax;
  int hi = diff ? 32 - __clz(diff) : 0;                                    // the keys agree on all bits >= hi
  uint32_t mask = hi >= 32 ? 0u : ~((hi == 0) ? 0u : ((1u << hi) - 1u));   // decided bits
  uint32_t prefix = kmax & mask;
  uint32_t* h_use = L.hist[0];
  uint32_t* h_next = L.hist[1];
  uint32_t* h_clear = L.hist[2];
  bool first = true;
  while (hi > 0) {
    const int lo_bit = max(hi - 8, 0);
    const uint32_t dmask = (1u << (hi - lo_bit)) - 1u;
    for_each_listed<NT>(keys, n, [&](uint32_t k) {
      if ((k & mask) == prefix) atomicAdd(&h_use[(k >> lo_bit) & dmask], 1u);
    });
    __syncthreads();
    // h_clear was last read before this barrier (during the previous pass) and is next written after the next one
    if (!first && tid < 256) h_clear[tid] = 0u;
    first = false;
    // every wave locates the cut bin for itself; scan position o = 4 * lane + i is bin 255 - o
    const u32x4 raw = *reinterpret_cast<const u32x4*>(h_use + 4 * (63 - lane));
    const uint32_t cc[4] = {raw[3], raw[2], raw[1], raw[0]};
    const uint32_t sum = cc[0] + cc[1] + cc[2] + cc[3];
    const uint32_t inc = wave_incl_scan_u32(sum);
    const uint32_t excl = inc - sum;
    const bool hit = excl < need && need <= inc;   // exactly one lane
    uint32_t rem = need - excl;
    int i = 0;
#pragma unroll
    for (; i < 3; ++i) {
      if (rem <= cc[i]) break;
      rem -= cc[i];
    }
    const int o = 4 * lane + i;
    const unsigned long long bal = __builtin_amdgcn_ballot_w64(hit);
    if (bal == 0) break;   // cannot happen while need <= n
    const int src = __builtin_ctzll(bal);
    const uint32_t bin = (uint32_t)__builtin_amdgcn_readlane(255 - o, src);
    need = (uint32_t)__builtin_amdgcn_readlane((int)rem, src);
    prefix |= bin << lo_bit;
    mask |= dmask << lo_bit;
    hi = lo_bit;
    uint32_t* t = h_use;
    h_use = h_next;
    h_next = h_clear;
    h_clear = t;
  }
  *cut_key = prefix;
  *need_eq = need;
}

// ---------------------------------------------------------------------------------------------
// One block per head: the exact cut among the band candidates, then the output offset of every tile.
__global__ __launch_bounds__(kSelHeadThreads) void sel_band_select(Dims dm, float* __restrict__ scores,
                                                                   const int32_t* __restrict__ kv_lens,
                                                                   const int32_t* __restrict__ budgets,
                                                                   uint32_t* __restrict__ ws) {
  __shared__ HeadSelectLds L;
  __shared__ uint32_t cnt[kSelMaxTiles];   // per tile: band keys above the exact cut (high half), equal to it (low half)
  const SelCtx c = sel_ctx(dm, scores, kv_lens, budgets, ws, blockIdx.x, blockIdx.y);
  const int tid = threadIdx.x;
  // requested together: the histogram, the number of candidates, and the first of these (the arrays hold T_max > 32768 entries)
  const u32x4 hv = *reinterpret_cast<const u32x4*>(c.w.hist + 4 * tid);
  const uint32_t bin_hi = c.w.meta[kMetaBinHi];
  const uint32_t n_c = c.w.meta[kMetaCand];
  uint32_t ck[kHeadCands], cp[kHeadCands];
#pragma unroll
  for (int i = 0; i < kHeadCands; ++i) {
    ck[i] = c.w.cand_key[tid + kSelHeadThreads * i];
    cp[i] = c.w.cand_pos[tid + kSelHeadThreads * i];
  }
  requests_leave(c);
  if (c.B == 0 || c.B >= c.T) return;   // block-uniform
  const int nt = (c.T + kSelTile - 1) / kSelTile;   // tiles of this head that the per-tile kernels worked on
  for (int i = tid; i < nt; i += kSelHeadThreads) cnt[i] = 0u;
  if (tid < 256) L.cut.hist[tid] = 0u;
  if (tid == 0) L.cut.n = 0u;
  // keys that are certainly selected: everything in the bins above the band
  uint32_t n_in = 0;
#pragma unroll
  for (int i = 0; i < 4; ++i) n_in += (uint32_t)(4 * tid + i) > bin_hi ? hv[i] : 0u;
  n_in = wave_incl_scan_u32(n_in);
  if ((tid & 63) == 63) L.wsum[tid >> 6] = n_in;
  __syncthreads();
  const uint32_t tot_in = row16_sum_u32(L.wsum[tid & 15]);
  const uint32_t need = (uint32_t)c.B - tot_in;   // >= 1: fewer than B keys lie above the cut bin, let alone the band
  uint32_t tau, need_eq;
  const bool held = n_c <= (uint32_t)(kSelHeadThreads * kHeadCands);   // block-uniform
  // (radix select over memory, four passes of the candidates: 8 sequences x 8 heads of 4096 to 65536 positions 12.8 us, 8.5 so; 4 heads
  // of 39853 7.8, 6.4 so)
  if (!held || !cut_among<kSelHeadThreads, kHeadCands>(ck, n_c, need, L.cut, &tau, &need_eq))
    stream_radix_select_desc<kSelHeadThreads>(c.w.cand_key, n_c, need, L.rs, &tau, &need_eq);
  if (held) {
#pragma unroll
    for (int i = 0; i < kHeadCands; ++i)
      if ((uint32_t)(tid + kSelHeadThreads * i) < n_c && ck[i] >= tau)
        atomicAdd(&cnt[cp[i] / kSelTile], ck[i] > tau ? 0x10000u : 1u);
  } else {
    for_each_listed<kSelHeadThreads>(c.w.cand_key, c.w.cand_pos, n_c, [&](uint32_t k, uint32_t pos) {
      if (k >= tau) atomicAdd(&cnt[pos / kSelTile], k > tau ? 0x10000u : 1u);
    });
  }
  __syncthreads();
  // Output offsets.  Thread t owns tiles t*tpt .. +tpt; first the number of cut-equal band keys before every tile
  // (equal scores go to the lower positions, so a tile takes what is left of need_eq when its turn comes), then the
  // number of selected keys before it.
  const int tpt = (nt + kSelHeadThreads - 1) / kSelHeadThreads;
  const int i0 = tid * tpt, i1 = min(i0 + tpt, nt);
  uint32_t e_sum = 0;
  for (int i = i0; i < i1; ++i) e_sum += cnt[i] & 0xFFFFu;
  uint32_t tot;
  uint32_t eqb = block_excl_scan<kSelHeadThreads>(e_sum, L.wsum, &tot);
  uint32_t s_sum = 0;
  for (int i = i0; i < i1; ++i) {
    const uint32_t eq = cnt[i] & 0xFFFFu, gt = cnt[i] >> 16;
    const uint32_t take_eq = min(eq, need_eq > eqb ? need_eq - eqb : 0u);
    c.w.tile_eqb[i] = eqb;
    eqb += eq;
    const uint32_t sel = c.w.tile_in[i] + gt + take_eq;
    cnt[i] = sel;   // (own tiles only: nobody else reads them again)
    s_sum += sel;
  }
  uint32_t off = block_excl_scan<kSelHeadThreads>(s_sum, L.wsum, &tot);
  for (int i = i0; i < i1; ++i) {
    c.w.tile_off[i] = off;
    off += cnt[i];
  }
  if (tid == 0) {
    c.w.meta[kMetaTau] = tau;
    c.w.meta[kMetaNeedEq] = need_eq;
  }
}

// ---------------------------------------------------------------------------------------------
// Ordered emission of one tile.  Wave w owns 512 consecutive positions; register j of its lane l is position 64*j + l of
// them, so scores and indices travel as coalesced rows and wave ballots give the order
// (8 x 8 ragged heads: 11.7 us with eight consecutive positions a thread, 9.0 so).  `take`: keys selected whatever the
// ties; `eq`: keys equal to the cut, of which the `need_eq` lowest positions are selected (`eq_tile0` of them lie in
// earlier tiles); `off`: selected keys in earlier tiles.
constexpr int kSelWaves = kSelThreads / 64;
// (`take` and `eq`: bit j is the lane's register j)
__device__ __forceinline__ void emit_tile(uint32_t take, uint32_t eq, uint32_t eq_tile0, uint32_t need_eq, uint32_t off,
                                          int lo, int B, uint32_t* wcnt, int32_t* __restrict__ out) {
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint32_t cnt = wave_incl_scan_u32(((uint32_t)__popc(take) << 16) | (uint32_t)__popc(eq));
  if (lane == 63) wcnt[w] = cnt;   // (a tile has 2048 keys: both counts fit 16 bits)
  __syncthreads();
  uint32_t p_take = 0, p_eq = eq_tile0;
#pragma unroll
  for (int i = 0; i < kSelWaves; ++i) {
    const uint32_t c = wcnt[i];
    p_take += i < w ? c >> 16 : 0u;
    p_eq += i < w ? c & 0xFFFFu : 0u;
  }
  const unsigned long long below = (1ull << lane) - 1ull;
  const uint32_t eq_off = off - min(eq_tile0, need_eq);   // (ties taken in earlier tiles are part of `off`)
#pragma unroll
  for (int j = 0; j < kSelIPT; ++j) {
    const bool is_take = (take >> j) & 1u, is_eq = (eq >> j) & 1u;
    const unsigned long long m_take = __builtin_amdgcn_ballot_w64(is_take), m_eq = __builtin_amdgcn_ballot_w64(is_eq);
    const uint32_t eq_before = p_eq + __popcll(m_eq & below);
    if (is_take || (is_eq && eq_before < need_eq)) {
      const uint32_t pos = eq_off + p_take + __popcll(m_take & below) + min(eq_before, need_eq);
      if (pos < (uint32_t)B) out[pos] = lo + 64 * j;   // guard: inconsistent inputs cannot push writes past the budget
    }
    p_take += (uint32_t)__popcll(m_take);
    p_eq += (uint32_t)__popcll(m_eq);
  }
}

__global__ __launch_bounds__(kSelThreads) void sel_emit(Dims dm, float* __restrict__ scores,
                                                       const int32_t* __restrict__ kv_lens,
                                                       const int32_t* __restrict__ budgets, uint32_t* __restrict__ ws,
                                                       int32_t* __restrict__ k_idx, int32_t* __restrict__ k_cnt) {
  __shared__ uint32_t wcnt[kSelWaves];
  const int kv = blockIdx.y, b = blockIdx.z;
  const SelCtx c = sel_ctx(dm, scores, kv_lens, budgets, ws, kv, b);
  const int t0 = blockIdx.x * kSelTile;
  // Everything is requested before the cache length is known (a fetch of what another launch has just written takes
  // about 2 us, and they would queue up behind each other): positions are clamped to the array.
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lo = t0 + w * 64 * kSelIPT + lane;
  float v[kSelIPT];
#pragma unroll
  for (int j = 0; j < kSelIPT; ++j) v[j] = c.sc[min(lo + 64 * j, dm.T_max - 1)];
  // this wave's band mask: two words a register, lane i holds word i
  const uint32_t mword = c.w.mask[(size_t)blockIdx.x * (kSelTile / 32) + w * (2 * kSelIPT) + min(lane, 2 * kSelIPT - 1)];
  const int bin_hi = (int)c.w.meta[kMetaBinHi];
  const uint32_t tau = c.w.meta[kMetaTau], need_eq = c.w.meta[kMetaNeedEq];
  const uint32_t eq_tile0 = c.w.tile_eqb[blockIdx.x], off = c.w.tile_off[blockIdx.x];
  requests_leave(c);
  int32_t* out = k_idx + (size_t)c.head * dm.B_max;
  if (blockIdx.x == 0 && threadIdx.x == 0) k_cnt[c.head] = c.B;
  if (c.B == 0 || t0 >= c.T) return;
  const int t1 = min(t0 + kSelTile, c.T);
  if (c.B >= c.T) {
    for (int i = t0 + threadIdx.x; i < t1; i += kSelThreads) out[i] = i;
    return;
  }
  uint32_t take = 0, eq = 0;
#pragma unroll
  for (int j = 0; j < kSelIPT; ++j) {
    const bool in = lo + 64 * j < t1;
    const uint32_t m_lo = (uint32_t)__builtin_amdgcn_readlane((int)mword, 2 * j),
                   m_hi = (uint32_t)__builtin_amdgcn_readlane((int)mword, 2 * j + 1);
    const bool band = ((lane < 32 ? m_lo : m_hi) >> (lane & 31)) & 1u;
    const uint32_t k = max(okey(v[j]), 1u);
    take |= (in && (band ? k > tau : score_bin(v[j]) > bin_hi) ? 1u : 0u) << j;
    eq |= (in && band && k == tau ? 1u : 0u) << j;
  }
  emit_tile(take, eq, eq_tile0, need_eq, off, lo, c.B, wcnt, out);
}

// ---------------------------------------------------------------------------------------------
// Exact scores (score_packs, select_keys_exact_pays, select_keys_streams_exact): nothing is scored again, the candidates are the keys of the cut's own bin.  A few
// dozen of ordinary scores in 4096 bins; in the exact scorer's 2048, of one KV head of 16 whose best scores lie close together,
// beyond 1024, which are then selected from memory (131072 independent keys, 64 queries, budget 12 % 61 us a call, two-pass 109).
// Launch chain: scoring with the histogram, one count per tile, emission; every emitting block finds the cut among the
// candidates for itself, which is cheaper than a launch for it while the heads are short.  Measured (re-score, select, emit before -> these two; the scoring
// launch takes the same): 8 sequences x 8 heads of 4096 to 65536 positions 48 -> 24 us (call 216 -> 196 us), 8 heads of
// 100003 23 -> 14 us (call 88 -> 80 us).
static_assert(kPackMaxKeys / kSelTile <= 64, "one lane a tile");

template <int BINS>
__global__ __launch_bounds__(kSelThreads) void sel_classify(Dims dm, float* __restrict__ scores,
                                                           const int32_t* __restrict__ kv_lens,
                                                           const int32_t* __restrict__ budgets, uint32_t* __restrict__ ws) {
  constexpr int PER = BINS / kSelThreads;
  __shared__ uint32_t sh[kSelThreads / 64 + 1];
  __shared__ uint32_t bin, n_in, n_cand, slot0;
  const SelCtx c = sel_ctx(dm, scores, kv_lens, budgets, ws, blockIdx.y, blockIdx.z);
  const int t0 = blockIdx.x * kSelTile;
  const int tid = threadIdx.x, lane = tid & 63;
  float v[kSelIPT];   // (requested before the cache length is known)
#pragma unroll
  for (int i = 0; i < kSelIPT; ++i) v[i] = c.sc[min(t0 + tid + kSelThreads * i, dm.T_max - 1)];
  uint32_t hv[PER];
  if constexpr (BINS == kSelBins) {
    load_hist_run(c.w.hist, hv);
  } else {   // the copies of the exact scorer's histogram, four at a time
    const int heads = dm.b * dm.n_kv, copies = exact_hist_copies(heads);
#pragma unroll
    for (int i = 0; i < PER; ++i) hv[i] = 0u;
    for (int j0 = 0; j0 < copies; j0 += 4) {
      uint32_t h[4][PER];
#pragma unroll
      for (int j = 0; j < 4; ++j) load_hist_run(exact_hist(ws, heads, c.head, min(j0 + j, copies - 1)), h[j]);
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int i = 0; i < PER; ++i) hv[i] += j0 + j < copies ? h[j][i] : 0u;
    }
  }
  requests_leave(c);
  if (c.B == 0 || c.B >= c.T || t0 >= c.T) return;   // block-uniform
  if (tid == 0) n_in = n_cand = 0u;
  const int cut_bin = find_cut_bin(hv, (uint32_t)c.B, sh, &bin);
  // The candidates get slots inside the block first, and the block one piece of the head's list: waves that each asked for
  // theirs queued up at the head's counter (one head of 130664 positions: 14.7 us, 6.6 so; 4 heads of 39853 7.0, 4.8 so).
  uint32_t above = 0, mine = 0, cand = 0;
#pragma unroll
  for (int i = 0; i < kSelIPT; ++i) {
    const int t = t0 + tid + kSelThreads * i;
    const int k = coarse_bin<BINS>(v[i]);
    above += t < c.T && k > cut_bin ? 1u : 0u;
    const bool is_cand = t < c.T && k == cut_bin;
    cand |= is_cand ? 1u << i : 0u;
    mine += is_cand ? 1u : 0u;
  }
  // (one scan for both counts: a tile has 2048 keys)
  const uint32_t upto = wave_incl_scan_u32((above << 16) | mine);
  uint32_t at = 0;
  if (lane == 63) {
    if (upto >> 16) atomicAdd(&n_in, upto >> 16);
    if (upto & 0xFFFFu) at = atomicAdd(&n_cand, upto & 0xFFFFu);
  }
  at = (uint32_t)__builtin_amdgcn_readlane((int)at, 63) + (upto & 0xFFFFu) - mine;   // any order of the waves will do
  __syncthreads();
  if (tid == 0) {
    if (n_cand) slot0 = atomicAdd(&c.w.meta[kMetaCand], n_cand);
    c.w.tile_in[blockIdx.x] = n_in;
    if (blockIdx.x == 0) c.w.meta[kMetaBinHi] = (uint32_t)cut_bin;
  }
  __syncthreads();
  if (n_cand == 0) return;
  at += slot0;
#pragma unroll
  for (int i = 0; i < kSelIPT; ++i) {
    if ((cand >> i) & 1u) {
      c.w.cand_key[at] = max(okey(v[i]), 1u);
      c.w.cand_pos[at] = (uint32_t)(t0 + tid + kSelThreads * i);
      ++at;
    }
  }
}

constexpr int kFinCands = 4;   // candidates a thread holds in registers; more are radix-selected from memory
template <int BINS>
__global__ __launch_bounds__(kSelThreads) void sel_finish(Dims dm, float* __restrict__ scores,
                                                         const int32_t* __restrict__ kv_lens,
                                                         const int32_t* __restrict__ budgets, uint32_t* __restrict__ ws,
                                                         int32_t* __restrict__ k_idx, int32_t* __restrict__ k_cnt) {
  __shared__ RadixSelectLds rs;
  __shared__ CutListLds cl;
  __shared__ uint32_t sums[4], wcnt[kSelWaves];
  const SelCtx c = sel_ctx(dm, scores, kv_lens, budgets, ws, blockIdx.y, blockIdx.z);
  const int t0 = blockIdx.x * kSelTile;
  // requested before the cache length and the number of candidates are known (the arrays hold T_max > 32768 entries)
  const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lo = t0 + w * 64 * kSelIPT + lane;
  float v[kSelIPT];
#pragma unroll
  for (int j = 0; j < kSelIPT; ++j) v[j] = c.sc[min(lo + 64 * j, dm.T_max - 1)];
  const uint32_t n_c = c.w.meta[kMetaCand];
  const int cut_bin = (int)c.w.meta[kMetaBinHi];
  uint32_t ck[kFinCands], cp[kFinCands];
#pragma unroll
  for (int i = 0; i < kFinCands; ++i) {
    ck[i] = c.w.cand_key[tid + kSelThreads * i];
    cp[i] = c.w.cand_pos[tid + kSelThreads * i];
  }
  uint32_t certain = c.w.tile_in[min(tid, sel_tiles(dm.T_max) - 1)];
  requests_leave(c);
  int32_t* out = k_idx + (size_t)c.head * dm.B_max;
  if (blockIdx.x == 0 && threadIdx.x == 0) k_cnt[c.head] = c.B;
  if (c.B == 0 || t0 >= c.T) return;   // block-uniform
  const int t1 = min(t0 + kSelTile, c.T);
  if (c.B >= c.T) {
    for (int i = t0 + threadIdx.x; i < t1; i += kSelThreads) out[i] = i;
    return;
  }
  cl.hist[tid] = 0u;
  if (tid == 0) cl.n = sums[2] = sums[3] = 0u;
  // certainly selected keys, in all tiles and in the earlier ones (the first wave has a lane for every tile)
  if (w == 0) {
    if (lane >= (c.T + kSelTile - 1) / kSelTile) certain = 0u;
    const uint32_t upto = wave_incl_scan_u32(certain);
    if (lane == 63) sums[0] = upto;
    if (lane == (int)blockIdx.x) sums[1] = upto - certain;
  }
  __syncthreads();
  const uint32_t need = (uint32_t)c.B - sums[0];   // >= 1: fewer than B keys lie above the cut bin
  uint32_t tau, need_eq;
  // (every candidate against every other in 256 threads: 4 heads of 124502, 2 queries, budget 17 % 18.0 us, 6.5 so; 64 heads of 4096 to
  // 65536 14.3, 11.2 so)
  const bool held = n_c <= (uint32_t)(kSelThreads * kFinCands);   // block-uniform
  if (!held || !cut_among<kSelThreads, kFinCands>(ck, n_c, need, cl, &tau, &need_eq))
    stream_radix_select_desc<kSelThreads>(c.w.cand_key, n_c, need, rs, &tau, &need_eq);
  // candidates above the cut, and equal to it, in earlier tiles
  uint32_t gt = 0, eq0 = 0;
  if (held) {
#pragma unroll
    for (int i = 0; i < kFinCands; ++i) {
      const bool earlier = (uint32_t)(tid + kSelThreads * i) < n_c && cp[i] < (uint32_t)t0;
      gt += earlier && ck[i] > tau ? 1u : 0u;
      eq0 += earlier && ck[i] == tau ? 1u : 0u;
    }
  } else {
    for_each_listed<kSelThreads>(c.w.cand_key, c.w.cand_pos, n_c, [&](uint32_t k, uint32_t pos) {
      const bool earlier = pos < (uint32_t)t0;
      gt += earlier && k > tau ? 1u : 0u;
      eq0 += earlier && k == tau ? 1u : 0u;
    });
  }
  if (gt) atomicAdd(&sums[2], gt);
  if (eq0) atomicAdd(&sums[3], eq0);
  uint32_t take = 0, eq = 0;
#pragma unroll
  for (int j = 0; j < kSelIPT; ++j) {
    const bool in = lo + 64 * j < t1;
    const uint32_t k = max(okey(v[j]), 1u);
    const int bin = coarse_bin<BINS>(v[j]);
    take |= (in && (bin > cut_bin || (bin == cut_bin && k > tau)) ? 1u : 0u) << j;
    eq |= (in && bin == cut_bin && k == tau ? 1u : 0u) << j;
  }
  __syncthreads();
  const uint32_t eq_tile0 = sums[3];
  emit_tile(take, eq, eq_tile0, need_eq, sums[1] + sums[2] + min(eq_tile0, need_eq), lo, c.B, wcnt, out);
}

// ---------------------------------------------------------------------------------------------
bool select_keys_two_pass_applies(const Dims& dm, int dtype) {
  // the error bound of the provisional pass is uniform only for cosine scores reduced by max; short caches take one
  // single-block top-k launch after the exact scores, which the longer chain of this stage cannot beat
  return dtype == QUOKA_BF16 && dm.T_cap > 32768 &&
         (dm.flags & (QUOKA_SCORE_DOT | QUOKA_SCORE_MEAN | QUOKA_SCORE_QBAR_BF16)) == 0;
}

// Exact scores of every key (three terms, score_bf16) with their histogram, and no key scored twice: two short launches follow
// instead of three, for up to three times the matrix work.  Whole calls with a small attention part, caches not in any cache
// memory (us, two-pass -> exact): up to 64 queries 1 head of 72294 61.0 -> 41.7, 2 of 99086 75.7 -> 66.2, 8 of 55226 79.1 -> 72.3,
// 8 of 92109 90.8 -> 84.7, 3 x 8 of 53300 120.0 -> 116.8 (246 MB of keys), 8 x 8 of 49927 230.7 -> 233.4 (820 MB); up to 128
// queries 2 of 88869 76.5 -> 63.6, 4 of 58639 74.3 -> 69.0, 8 of 83522, d 64 76.8 -> 74.7 (86 MB), 8 of 47311 82.3 -> 83.0 (97 MB),
// 8 x 8 of 36611, d 64 138 -> 156.  260 sizes measured; the lines lie where the two sides meet.  Packed calls score exactly either way and the
// streaming launch is the faster for them; a prompt's chunks share one cache, 12 prompts 0.96 - 1.15 of the time, no line to draw.
// (At these sizes a scoring block has far fewer than the 65536 keys that its 16-bit counters hold.)
constexpr long long kExactBytesFew = 300'000'000, kExactBytes = 250'000'000, kExactBytesWide = 80'000'000;
static long long exact_bytes(int n_keep) { return n_keep <= 32 ? kExactBytesFew : n_keep <= 64 ? kExactBytes : kExactBytesWide; }
bool select_keys_exact_pays(const Dims& dm, int dtype) {
  if (!select_keys_two_pass_applies(dm, dtype) || dm.T_max > kPackMaxKeys || score_packs(dm)) return false;
  const int n_keep = dm.n_ret < dm.C ? dm.n_ret : dm.C;
  return (long long)dm.b * dm.n_kv * dm.T_cap * dm.d * 2 <= exact_bytes(n_keep);
}

// Beyond those sizes exact scores come from the streaming launch, as long as its products hide behind the keys' way from memory: up
// to 64 queries.  Whole calls with a small attention part, us: against the two-pass form 8 x 8 heads of 4096 to 64077 positions, 64
// queries 321 -> 310, 3 x 8 of 53300 144 -> 133, 13 x 4 of 7500 to 60000 187 -> 177, d 64 13 x 8 of 5000 to 40000 146 -> 131; against the
// exact scores of the tiled launch 8 of 131072, 268 MB 115.6 -> 111.8, 2 x 8 of 130000, d 64, 266 MB 132.5 -> 127.0 (33 to 64 queries over 250
// to 300 MB 0.95 of the time at d 64, 0.98 at d 128), but 8 of 92109, 189 MB 97.7 -> 98.3, 8 of 130000, d 64, 133 MB 83.2 -> 86.2, 1 of 72294
// 48.7 -> 53.1.  With up to 32 queries the tiled launch has little to compute, and from 250 to 300 MB the streaming one is 1 % slower (333
// calls; d 64, 4 x 8 heads of 67939 94 and 98 us); two-pass, which it replaces beyond, takes 1.10 to 1.17 of its time.
bool select_keys_streams_exact(const Dims& dm, int dtype) {
  if (!select_keys_two_pass_applies(dm, dtype) || dm.T_max > kPackMaxKeys || score_packs(dm)) return false;
  const int n_keep = dm.n_ret < dm.C ? dm.n_ret : dm.C;
  return n_keep <= 64 && (long long)dm.b * dm.n_kv * dm.T_cap * dm.d * 2 > exact_bytes(n_keep);
}

hipError_t launch_select_keys_exact(const Dims& dm, const float* qbar, const void* k_cache, const int32_t* kv_lens,
                                    const int32_t* budgets, float* scores, int32_t* k_idx, int32_t* k_cnt, uint32_t* ws,
                                    const uint16_t* terms, hipStream_t st) {
  const hipError_t e = launch_score_hist(dm, qbar, k_cache, kv_lens, scores, st, terms, ws);
  if (e != hipSuccess) return e;
  const dim3 grid(sel_tiles(dm.T_cap), dm.n_kv, dm.b);
  hipLaunchKernelGGL((sel_classify<kScoreBins>), grid, dim3(kSelThreads), 0, st, dm, scores, kv_lens, budgets, ws);
  hipLaunchKernelGGL((sel_finish<kScoreBins>), grid, dim3(kSelThreads), 0, st, dm, scores, kv_lens, budgets, ws, k_idx, k_cnt);
  return hipGetLastError();
}

size_t select_keys_ws_words(const Dims& dm) {
  if (dm.T_max <= 32768) return 0;
  const int heads = dm.b * dm.n_kv;
  return sel_zero_words(heads) + exact_hist_words(heads) + (size_t)heads * sel_head_words(dm.T_max);
}

size_t select_keys_zero_words(const Dims& dm, bool exact) {
  const int heads = dm.b * dm.n_kv;
  return sel_zero_words(heads) + (exact ? exact_hist_words(heads) : 0);
}

template <int D>
static void launch_rescore(const Dims& dm, const float* qbar, const void* kc, const int32_t* kv_lens,
                           const int32_t* budgets, float* scores, uint32_t* ws, int n_keep, hipStream_t st) {
  // one round of two blocks per compute unit: fewer, fatter blocks amortise the histogram scan and the query operands
  // (mixed-length batch of 8 x 8 heads: 37 us with 512 blocks, 41 with 1024, 49 with 2048)
  const int heads = dm.b * dm.n_kv, nt = sel_tiles(dm.T_cap);
  const int per_head = (512 + heads - 1) / heads;
  const int tpb = (nt + per_head - 1) / per_head;
  const dim3 grid((nt + tpb - 1) / tpb, dm.n_kv, dm.b);
  const int qblocks = (n_keep + 31) / 32;
  const uint16_t* k = static_cast<const uint16_t*>(kc);
  if (qblocks <= 1) {
    hipLaunchKernelGGL((sel_band_rescore<D, 1>), grid, dim3(kSelThreads), 0, st, dm, qbar, k, kv_lens, budgets, scores,
                       ws, n_keep, tpb);
  } else if (qblocks == 2) {
    hipLaunchKernelGGL((sel_band_rescore<D, 2>), grid, dim3(kSelThreads), 0, st, dm, qbar, k, kv_lens, budgets, scores,
                       ws, n_keep, tpb);
  } else {
    hipLaunchKernelGGL((sel_band_rescore<D, 4>), grid, dim3(kSelThreads), 0, st, dm, qbar, k, kv_lens, budgets, scores,
                       ws, n_keep, tpb);
  }
}

hipError_t launch_select_keys(const Dims& dm, const float* qbar, const void* k_cache, const int32_t* kv_lens,
                              const int32_t* budgets, float* scores, int32_t* k_idx, int32_t* k_cnt, uint32_t* ws,
                              hipStream_t st, bool ws_is_zero, const uint16_t* terms) {
  const int n_keep = dm.n_ret < dm.C ? dm.n_ret : dm.C;
  if (!ws_is_zero) hipLaunchKernelGGL(sel_zero, dim3(64), dim3(256), 0, st, ws, select_keys_zero_words(dm, false));
  // provisional scores and their histogram in one streaming launch
  hipError_t e = launch_score_stream(dm, qbar, terms, k_cache, kv_lens, scores, ws, st);
  if (e != hipSuccess) return e;
  const dim3 grid(sel_tiles(dm.T_cap), dm.n_kv, dm.b);
  if (score_packs(dm) || terms != nullptr) {
    hipLaunchKernelGGL((sel_classify<kSelBins>), grid, dim3(kSelThreads), 0, st, dm, scores, kv_lens, budgets, ws);
    hipLaunchKernelGGL((sel_finish<kSelBins>), grid, dim3(kSelThreads), 0, st, dm, scores, kv_lens, budgets, ws, k_idx, k_cnt);
    return hipGetLastError();
  }
  if (dm.d == 64) {
    launch_rescore<64>(dm, qbar, k_cache, kv_lens, budgets, scores, ws, n_keep, st);
  } else {
    launch_rescore<128>(dm, qbar, k_cache, kv_lens, budgets, scores, ws, n_keep, st);
  }
  hipLaunchKernelGGL(sel_band_select, dim3(dm.n_kv, dm.b), dim3(kSelHeadThreads), 0, st, dm, scores, kv_lens, budgets,
                     ws);
  hipLaunchKernelGGL(sel_emit, grid, dim3(kSelThreads), 0, st, dm, scores, kv_lens, budgets, ws, k_idx, k_cnt);
  return hipGetLastError();
}

}  // namespace quoka
