// Top-B key selection per (sequence, KV head) (Alg. 1: I = topk(S-hat, B_SA); Eq. 3).
//
// The cut (the B-th largest score) is found exactly, and an ordered compaction emits the positions of the scores above it
// and of the first ones equal to it: ascending, equal scores to the lower position.  Scores are compared as floats (-0
// equals +0, a NaN ranks as the infinity of its sign), or as order-preserving images that compare alike, so the result is
// deterministic and does not depend on the launch shape.
//
//   T_max <= kSmallMax : one to four 1024-thread blocks per head, scores held in registers, one launch; the cut from a
//                        histogram over equal score bins and a count of ranks in the cut's bin.
//   larger             : several blocks per head.  Three histogram passes (11 + 11 + 10 bits, global
//                        integer atomics) find the cut key; a count pass and an emit pass produce
//                        the ordered index list.  Each launch derives the newest step of the cut
//                        from the histogram the previous launch completed (and leaves it in the
//                        workspace for the later ones), so no kernel waits on another block.
#include "common.hip.h"
#include "kernels.h"

namespace quoka {

constexpr int kSmallMax = 32768;   // beyond this one compute unit is slower than the multi-block path
constexpr int kSmallThreads = 1024;
constexpr int kLgThreads = 256;
constexpr int kLgTile = 2048;          // scores per block in the multi-block path
constexpr int kBins = 2048;            // bins per histogram pass (11 bits; last pass uses 1024)

__device__ __forceinline__ int radix_shift(int pass) { return pass == 0 ? 21 : (pass == 1 ? 10 : 0); }
__device__ __forceinline__ uint32_t radix_bins(int pass) { return pass == 2 ? 1024u : 2048u; }

// ---------------------------------------------------------------------------------------------
// Register path.  Wave w owns scores [w*64*IPT, (w+1)*64*IPT); its register j of lane l is score
// w*64*IPT + 64*j + l, so every load is a coalesced 256-byte row and position order inside a wave is (j, lane).
// The cut: one LDS histogram over 2048 equal bins between the smallest and the largest score, a scan for the bin that
// holds the B-th largest, and a count of ranks among that bin's few keys.  (Equal bins and not key bits: the scores of a
// head lie close together, and a lane's atomic on an occupied bin waits for the others.)  Where more keys share the
// bin than LDS has room for, or the scores admit no such bins, the block-wide radix select decides.
// The ordered compaction needs no scan over threads: per register, one wave ballot (two where only some of the keys
// equal to the cut are taken) gives every lane the number of earlier taken positions of its wave, and the 16 wave totals
// are combined through LDS.
//
// What bounds it: one compute unit's instruction rate (five passes over the keys) and a chain of six barriers.  So
// from 16 keys per thread on, several blocks take a head: all of them find the cut, each emits its share of the waves'
// ranges (two blocks: 16, four: 32 keys per thread).
// Measured (us, radix select on key bits and one block a head -> now): 8 heads of 8192 scores 7.9 -> 6.0, 8 of 32768
// 20.4 -> 13.5, 12 of up to 19999 19.0 -> 12.1.
constexpr int kCutBins = 2048;
constexpr int kCutKeys = 1024;
struct CutLds {
  uint32_t hist[kCutBins];
  float key[kCutKeys];
  uint32_t wsum[kSmallThreads / 64 + 1];
  float wmin[kSmallThreads / 64], wmax[kSmallThreads / 64];
  uint32_t n, bin, need, need_eq;
  float tau;
};

template <int IPT, int NB>
__global__ __launch_bounds__(kSmallThreads) void topk_small(Dims dm, const float* __restrict__ scores,
                                                           const int32_t* __restrict__ kv_lens,
                                                           const int32_t* __restrict__ budgets,
                                                           int32_t* __restrict__ k_idx, int32_t* __restrict__ k_cnt) {
  constexpr int NW = kSmallThreads / 64;
  constexpr int BPT = kCutBins / kSmallThreads;   // bins per thread
  __shared__ RadixSelectLds rs;
  __shared__ __align__(16) CutLds cl;
  __shared__ uint32_t wgt[NW], weq[NW];
  const int kv = blockIdx.x, b = blockIdx.y;
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const float* sc = scores + (size_t)(b * dm.n_kv + kv) * dm.T_max;
  const int lo = w * 64 * IPT + lane;   // position of register 0; register j is 64*j further
  // The scores are requested before the cache length is known (the row has T_max entries; those past the length
  // are discarded below), so the two fetches overlap instead of queueing behind each other.
  uint32_t rb[IPT];   // the scores' bits (the radix select borrows the registers for key images)
  auto val = [&](int j) __attribute__((always_inline)) { return __uint_as_float(rb[j]); };
#pragma unroll
  for (int j = 0; j < IPT; ++j) rb[j] = lo + 64 * j < dm.T_cap ? __float_as_uint(sc[lo + 64 * j]) : 0u;
  const int T = max(0, min(kv_lens[b * dm.ls], dm.T_cap));
  const int B = max(0, min(min(budgets[b * dm.ls], T), dm.B_max));
  int32_t* out = k_idx + (size_t)(b * dm.n_kv + kv) * dm.B_max;
  if (tid == 0 && blockIdx.z == 0) k_cnt[b * dm.n_kv + kv] = B;
  if (B == 0) return;
  if (B >= T) {
    for (int i = blockIdx.z * kSmallThreads + tid; i < T; i += NB * kSmallThreads) out[i] = i;
    return;
  }
#pragma unroll
  for (int i = 0; i < BPT; ++i) cl.hist[i * kSmallThreads + tid] = 0u;
  if (tid == 0) cl.n = 0u;
  // positions past the length become NaN: minima and maxima pass over them and no comparison holds for them
  float vmin = INFINITY, vmax = -INFINITY;
  unsigned long long nan = 0;   // lanes with a NaN among their scores proper
#pragma unroll
  for (int j = 0; j < IPT; ++j) {
    const bool past = lo + 64 * j >= T;
    nan |= __builtin_amdgcn_ballot_w64(!past && val(j) != val(j));
    if (past) rb[j] = 0x7FC00000u;
    vmin = fminf(vmin, val(j));
    vmax = fmaxf(vmax, val(j));
  }
  vmin = -wave64_max(-vmin);
  vmax = nan == 0 ? wave64_max(vmax) : INFINITY;   // (no bins then)
  if (lane == 0) {
    cl.wmin[w] = vmin;
    cl.wmax[w] = vmax;
  }
  __syncthreads();
  vmin = -wave64_max(lane < NW ? -cl.wmin[lane] : -INFINITY);
  vmax = wave64_max(lane < NW ? cl.wmax[lane] : -INFINITY);
  // monotone in v (a rounded product and a truncation of non-negative values), the largest score lands in the last bin
  const float per = ((float)kCutBins - 0.5f) / (vmax - vmin);
  const bool binned = per > 0.f && per < 1e30f;   // false for equal or infinite extremes, and where a score is NaN
  auto bin_of = [&](float v) __attribute__((always_inline)) { return min((int)((v - vmin) * per), kCutBins - 1); };
  const bool full = (w + 1) * 64 * IPT <= T;   // (wave-uniform) no position of this wave is past the length
  float tau = 0.f;
  uint32_t need_eq = 0u, n_in = kCutKeys + 1, need = (uint32_t)B;
  int cut_bin = 0;
  if (binned) {   // block-uniform
    if (full) {
#pragma unroll
      for (int j = 0; j < IPT; ++j) atomicAdd(&cl.hist[bin_of(val(j))], 1u);
    } else {
#pragma unroll
      for (int j = 0; j < IPT; ++j)
        if (val(j) >= vmin) atomicAdd(&cl.hist[bin_of(val(j))], 1u);   // (not for a NaN)
    }
    __syncthreads();
    uint32_t hv[BPT], mine = 0, tot;   // thread 0 has the highest bins
#pragma unroll
    for (int i = 0; i < BPT; ++i) {
      hv[i] = cl.hist[kCutBins - 1 - (tid * BPT + i)];
      mine += hv[i];
    }
    uint32_t above = block_excl_scan<kSmallThreads>(mine, cl.wsum, &tot);
    if (above < need && need <= above + mine) {   // exactly one thread (the histogram holds T > B keys)
#pragma unroll
      for (int i = 0; i < BPT; ++i) {
        if (above < need && need <= above + hv[i]) {
          cl.bin = kCutBins - 1 - (tid * BPT + i);
          cl.need = need - above;
        }
        above += hv[i];
      }
    }
    __syncthreads();
    cut_bin = (int)cl.bin;
    need = cl.need;
    asm volatile("" : "+v"(vmin));   // (the bins are worked out again: kept, they would need IPT more registers)
#pragma unroll
    for (int j = 0; j < IPT; ++j) {
      if (bin_of(val(j)) == cut_bin && val(j) >= vmin) {   // (false for a NaN)
        const uint32_t slot = atomicAdd(&cl.n, 1u);
        if (slot < (uint32_t)kCutKeys) cl.key[slot] = val(j);
      }
    }
    __syncthreads();
    n_in = cl.n;
  }
  if (n_in <= (uint32_t)kCutKeys) {   // block-uniform
    if (tid < (int)n_in) {
      const float k = cl.key[tid];
      uint32_t gt = 0, ge = 0;
      for (uint32_t j = 0; j < n_in; ++j) {
        gt += cl.key[j] > k ? 1u : 0u;
        ge += cl.key[j] >= k ? 1u : 0u;
      }
      if (gt < need && need <= ge) {   // (equal keys all write the same)
        cl.tau = k;
        cl.need_eq = need - gt;
      }
    }
    __syncthreads();
    tau = cl.tau;
    need_eq = cl.need_eq;
  } else {   // descending: the `need` largest of the bin's (or all) keys
    uint32_t in_bin = 0u, tau_key;
#pragma unroll
    for (int j = 0; j < IPT; ++j) {
      if (!binned) {   // every score proper; a NaN ranks as the infinity of its sign
        const bool in = lo + 64 * j < T;
        if (in && val(j) != val(j)) rb[j] = (rb[j] & 0x80000000u) | 0x7F800000u;
        in_bin |= (in ? 1u : 0u) << j;
      } else {
        in_bin |= (val(j) >= vmin && bin_of(val(j)) == cut_bin ? 1u : 0u) << j;
      }
      rb[j] = okey(val(j) + 0.0f);   // (one zero)
    }
    block_radix_select<IPT, true>(rb, in_bin, need, rs, &tau_key, &need_eq);
    auto back = [](uint32_t k) { return (k & 0x80000000u) ? k & 0x7FFFFFFFu : ~k; };   // inverse of okey
    tau = __uint_as_float(back(tau_key));
#pragma unroll
    for (int j = 0; j < IPT; ++j) rb[j] = back(rb[j]);
  }
  // wave totals of scores above the cut and equal to it
  {
    uint32_t c_gt = 0, c_eq = 0;
#pragma unroll
    for (int j = 0; j < IPT; ++j) {
      c_gt += (uint32_t)__popcll(__builtin_amdgcn_ballot_w64(val(j) > tau));
      c_eq += (uint32_t)__popcll(__builtin_amdgcn_ballot_w64(val(j) == tau));
      __builtin_amdgcn_sched_barrier(0);   // (see below)
    }
    if (lane == 0) {
      wgt[w] = c_gt;
      weq[w] = c_eq;
    }
  }
  __syncthreads();
  if (NB > 1 && w / (NW / NB) != (int)blockIdx.z) return;   // (no barrier follows) another block emits this wave's range
  // taken candidates at earlier positions (earlier waves): greater than the cut / equal to it
  const uint32_t all_eq = wave_incl_scan_u32(lane < NW ? weq[lane] : 0u);
  uint32_t n_gt = wave_incl_scan_u32(lane < w ? wgt[lane] : 0u);
  uint32_t n_eq = wave_incl_scan_u32(lane < w ? weq[lane] : 0u);
  n_gt = (uint32_t)__builtin_amdgcn_readlane((int)n_gt, 63);
  n_eq = (uint32_t)__builtin_amdgcn_readlane((int)n_eq, 63);
  const bool take_all_eq = (uint32_t)__builtin_amdgcn_readlane((int)all_eq, 63) == need_eq;
  const unsigned long long below = (1ull << lane) - 1ull;
  // (an opaque copy of the cut: otherwise the comparison masks of the counting loop above are kept alive for this
  // loop, 2 x IPT scalar register pairs that spill)
  float tau_e = tau;
  asm volatile("" : "+v"(tau_e));
  if (take_all_eq) {   // every key equal to the cut is taken (nearly always there is just one)
    uint32_t n_before = n_gt + n_eq;
#pragma unroll
    for (int j = 0; j < IPT; ++j) {
      const bool take = val(j) >= tau_e;
      const unsigned long long m = __builtin_amdgcn_ballot_w64(take);
      const uint32_t pos = n_before + __popcll(m & below);
      if (take && pos < (uint32_t)B) out[pos] = lo + 64 * j;   // guard: a malformed score array cannot push writes past the budget
      n_before += __popcll(m);
      __builtin_amdgcn_sched_barrier(0);   // keep one register's ballot live at a time (32 of them would spill SGPRs)
    }
    return;
  }
#pragma unroll
  for (int j = 0; j < IPT; ++j) {
    const int t = lo + 64 * j;
    const bool gt = val(j) > tau_e, eq = val(j) == tau_e;
    const unsigned long long m_gt = __builtin_amdgcn_ballot_w64(gt), m_eq = __builtin_amdgcn_ballot_w64(eq);
    const uint32_t gt_before = n_gt + __popcll(m_gt & below), eq_before = n_eq + __popcll(m_eq & below);
    if (gt || (eq && eq_before < need_eq)) {   // equal scores go to the lower positions
      const uint32_t pos = gt_before + min(eq_before, need_eq);
      if (pos < (uint32_t)B) out[pos] = t;     // guard: a malformed score array cannot push writes past the budget
    }
    n_gt += __popcll(m_gt);
    n_eq += __popcll(m_eq);
    __builtin_amdgcn_sched_barrier(0);   // keep one register's ballots live at a time (32 pairs would spill SGPRs)
  }
}

// ---------------------------------------------------------------------------------------------
// Multi-block path.  Workspace per head: hist[3][kBins] then tile counts [n_tiles][2].
struct Cut {
  uint32_t prefix;  // decided high bits of the cut key
  uint32_t mask;    // which bits are decided
  uint32_t need;    // rank of the cut inside the remaining candidates (1-based, descending)
};

// Whole block: locate the bin (scanning from the top) where the running count reaches `need`.
// Returns (bin, need reduced by the counts above that bin).  `sh` is LDS scratch [kLgThreads + 2].
__device__ __forceinline__ void find_bin(const uint32_t* __restrict__ hist, uint32_t nbins, uint32_t need,
                                         uint32_t* sh, uint32_t* bin_out, uint32_t* need_out) {
  // thread t owns bins [nbins - (t+1)*per, nbins - t*per): thread 0 has the highest bins.
  const uint32_t per = nbins / kLgThreads;
  const uint32_t top = nbins - threadIdx.x * per;   // exclusive upper bin
  uint32_t mine = 0;
  for (uint32_t i = 1; i <= per; ++i) mine += hist[top - i];
  uint32_t tot;
  const uint32_t above = block_excl_scan<kLgThreads>(mine, sh, &tot);   // count in all higher-bin threads
  __syncthreads();
  if (above < need && need <= above + mine) {   // exactly one thread (need <= total is guaranteed)
    uint32_t rem = need - above;
    uint32_t i = 1;
    for (; i <= per; ++i) {
      const uint32_t c = hist[top - i];
      if (rem <= c) break;
      rem -= c;
    }
    sh[kLgThreads] = top - i;
    sh[kLgThreads + 1] = rem;
  }
  __syncthreads();
  *bin_out = sh[kLgThreads];
  *need_out = sh[kLgThreads + 1];
  __syncthreads();
}

// The cut after `npass` finished histogram passes.  Every pass adds one step (a bin and the rank left inside it).  A
// kernel works out only the newest step, from the histogram the previous launch completed; the steps before it are
// read back from `cuts` (two words per step), where block 0 of the launch that first derived them has left them
// (`newest_stored`: a previous launch has already derived the newest step too).
__device__ __forceinline__ Cut derive_cut(const uint32_t* __restrict__ hist, uint32_t* __restrict__ cuts, int npass,
                                          bool newest_stored, uint32_t B, uint32_t* sh) {
  Cut c{0u, 0u, B};
  for (int p = 0; p < npass; ++p) {
    uint32_t bin, need;
    if (p + 1 < npass || newest_stored) {
      bin = cuts[2 * p];
      need = cuts[2 * p + 1];
    } else {
      find_bin(hist + p * kBins, radix_bins(p), c.need, sh, &bin, &need);
      if (blockIdx.x == 0 && threadIdx.x == 0) {
        cuts[2 * p] = bin;
        cuts[2 * p + 1] = need;
      }
    }
    const int sft = radix_shift(p);
    c.prefix |= bin << sft;
    c.mask |= (radix_bins(p) - 1u) << sft;
    c.need = need;
  }
  return c;
}

// A score's key image in the multi-block path: one zero, and a NaN as the infinity of its sign, as in the register path
// (NaN images lie beyond those of the infinities, and the sum keeps the sign).
__device__ __forceinline__ uint32_t score_key(float s) {
  return min(max(okey(s + 0.0f), 0x007FFFFFu), 0xFF800000u);
}

__global__ void topk_zero(uint32_t* __restrict__ p, size_t n) {
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) p[i] = 0u;
}

constexpr int kCutWords = 8;   // three (bin, rank) steps, padded
struct LgCtx {
  int T, B;
  const float* sc;
  uint32_t* hist;
  uint32_t* cuts;
  uint32_t* tcnt;
};

__device__ __forceinline__ LgCtx lg_ctx(const Dims& dm, const float* scores, const int32_t* kv_lens,
                                        const int32_t* budgets, uint32_t* ws, int n_tiles) {
  const int kv = blockIdx.y, b = blockIdx.z;
  LgCtx c;
  c.T = max(0, min(kv_lens[b * dm.ls], dm.T_cap));
  c.B = max(0, min(min(budgets[b * dm.ls], c.T), dm.B_max));
  const size_t head = (size_t)(b * dm.n_kv + kv);
  c.sc = scores + head * dm.T_max;
  const size_t per_head = 3 * (size_t)kBins + kCutWords + 2 * (size_t)n_tiles;
  c.hist = ws + head * per_head;
  c.cuts = c.hist + 3 * kBins;
  c.tcnt = c.cuts + kCutWords;
  return c;
}

template <int PASS>
__global__ __launch_bounds__(kLgThreads) void topk_hist(Dims dm, const float* __restrict__ scores,
                                                       const int32_t* __restrict__ kv_lens,
                                                       const int32_t* __restrict__ budgets, uint32_t* __restrict__ ws,
                                                       int n_tiles) {
  __shared__ uint32_t lh[kBins];
  __shared__ uint32_t sh[kLgThreads + 2];
  const LgCtx c = lg_ctx(dm, scores, kv_lens, budgets, ws, n_tiles);
  const int t0 = blockIdx.x * kLgTile;
  if (c.B == 0 || c.B >= c.T || t0 >= c.T) return;   // block-uniform
  const Cut cut = derive_cut(c.hist, c.cuts, PASS, false, (uint32_t)c.B, sh);
  for (int i = threadIdx.x; i < kBins; i += kLgThreads) lh[i] = 0;
  __syncthreads();
  const int sft = radix_shift(PASS);
  const uint32_t bm = radix_bins(PASS) - 1u;
  const int t1 = min(t0 + kLgTile, c.T);
  float v[kLgTile / kLgThreads];   // all requested before the first is used
#pragma unroll
  for (int j = 0; j < kLgTile / kLgThreads; ++j) v[j] = c.sc[min(t0 + (int)threadIdx.x + kLgThreads * j, t1 - 1)];
#pragma unroll
  for (int j = 0; j < kLgTile / kLgThreads; ++j) {
    const uint32_t k = score_key(v[j]);
    if (t0 + (int)threadIdx.x + kLgThreads * j < t1 && (k & cut.mask) == cut.prefix) atomicAdd(&lh[(k >> sft) & bm], 1u);
  }
  __syncthreads();
  uint32_t* gh = c.hist + PASS * kBins;
  for (int i = threadIdx.x; i < kBins; i += kLgThreads) {
    const uint32_t v = lh[i];
    if (v) atomicAdd(&gh[i], v);
  }
}

// EMIT == false: per-tile counts of (key > cut, key == cut).  EMIT == true: ordered output.
template <bool EMIT>
__global__ __launch_bounds__(kLgThreads) void topk_finish(Dims dm, const float* __restrict__ scores,
                                                         const int32_t* __restrict__ kv_lens,
                                                         const int32_t* __restrict__ budgets,
                                                         uint32_t* __restrict__ ws, int n_tiles,
                                                         int32_t* __restrict__ k_idx, int32_t* __restrict__ k_cnt) {
  __shared__ uint32_t sh[kLgThreads + 2];
  const LgCtx c = lg_ctx(dm, scores, kv_lens, budgets, ws, n_tiles);
  const int kv = blockIdx.y, b = blockIdx.z;
  const int t0 = blockIdx.x * kLgTile;
  int32_t* out = k_idx + (size_t)(b * dm.n_kv + kv) * dm.B_max;
  if (EMIT && blockIdx.x == 0 && threadIdx.x == 0) k_cnt[b * dm.n_kv + kv] = c.B;
  if (c.B == 0 || t0 >= c.T) return;
  const int t1 = min(t0 + kLgTile, c.T);
  if (c.B >= c.T) {
    if (EMIT)
      for (int i = t0 + threadIdx.x; i < t1; i += kLgThreads) out[i] = i;
    return;
  }
  const Cut cut = derive_cut(c.hist, c.cuts, 3, EMIT, (uint32_t)c.B, sh);   // the count pass leaves the last step for the emit pass
  const uint32_t tau = cut.prefix, need_eq = cut.need;
  // thread t owns kLgTile / kLgThreads consecutive scores
  constexpr int IPT = kLgTile / kLgThreads;
  const int lo = t0 + threadIdx.x * IPT;
  uint32_t kreg[IPT];
  uint32_t cnt = 0;   // keys above the cut in the high half, keys equal to it in the low half (at most 2048 per tile)
#pragma unroll
  for (int i = 0; i < IPT; ++i) {
    const int t = lo + i;
    const uint32_t k = t < t1 ? score_key(c.sc[t]) : 0u;   // 0 is below every key image
    kreg[i] = k;
    cnt += ((t < t1) && (k > tau) ? 0x10000u : 0u) + ((t < t1) && (k == tau) ? 1u : 0u);
  }
  uint32_t tot;
  const uint32_t before = block_excl_scan<kLgThreads>(cnt, sh, &tot);
  if (!EMIT) {
    if (threadIdx.x == 0) {
      c.tcnt[2 * blockIdx.x] = tot >> 16;
      c.tcnt[2 * blockIdx.x + 1] = tot & 0xFFFFu;
    }
    return;
  }
  const uint32_t p_gt = before >> 16;
  uint32_t p_eq = before & 0xFFFFu;
  // counts of all earlier tiles (fixed order; at most a few hundred tiles): per-thread partial sums, one wave scan
  // each, the four wave totals through LDS
  uint32_t e_gt = 0, e_eq = 0;
  for (int i = threadIdx.x; i < (int)blockIdx.x; i += kLgThreads) {
    e_gt += c.tcnt[2 * i];
    e_eq += c.tcnt[2 * i + 1];
  }
  e_gt = wave_incl_scan_u32(e_gt);
  e_eq = wave_incl_scan_u32(e_eq);
  __syncthreads();   // sh is free again
  if ((threadIdx.x & 63) == 63) {
    sh[threadIdx.x >> 6] = e_gt;
    sh[kLgThreads / 64 + (threadIdx.x >> 6)] = e_eq;
  }
  __syncthreads();
  uint32_t before_gt = 0, before_eq = 0;
#pragma unroll
  for (int i = 0; i < kLgThreads / 64; ++i) {
    before_gt += sh[i];
    before_eq += sh[kLgThreads / 64 + i];
  }
  p_eq += before_eq;
  uint32_t pos = before_gt + p_gt + min(p_eq, need_eq);
#pragma unroll
  for (int i = 0; i < IPT; ++i) {
    const int t = lo + i;
    if (t < t1) {
      const uint32_t k = kreg[i];
      bool take = k > tau;
      if (k == tau) {
        take = p_eq < need_eq;
        ++p_eq;
      }
      if (take) {
        if (pos < (uint32_t)c.B) out[pos] = t;
        ++pos;
      }
    }
  }
}

// ---------------------------------------------------------------------------------------------
static inline int lg_tiles(const Dims& dm) { return (dm.T_max + kLgTile - 1) / kLgTile; }

size_t topk_ws_words(const Dims& dm) {
  if (dm.T_max <= kSmallMax) return 0;
  return (size_t)dm.b * dm.n_kv * (3 * (size_t)kBins + kCutWords + 2 * (size_t)lg_tiles(dm));
}

bool topk_uses_ws(const Dims& dm) { return dm.T_cap > kSmallMax; }

hipError_t launch_topk_keys(const Dims& dm, const float* scores, const int32_t* kv_lens, const int32_t* budgets,
                            int32_t* k_idx, int32_t* k_cnt, uint32_t* ws, hipStream_t st, bool ws_is_zero) {
  if (!topk_uses_ws(dm)) {
    const dim3 block(kSmallThreads);
    const int ipt = (dm.T_cap + kSmallThreads - 1) / kSmallThreads;
    auto launch = [&](auto kernel, int blocks_per_head) {
      hipLaunchKernelGGL(kernel, dim3(dm.n_kv, dm.b, blocks_per_head), block, 0, st, dm, scores, kv_lens, budgets, k_idx, k_cnt);
    };
    // (The time goes with the keys a thread holds, so above 16 the variants lie close together: 12 heads of up to 19999
    // scores 12.3 -> 9.3 us, 8 of 24000 12.4 -> 10.3 against 32 keys a thread.  12 instead of 16 gave 0.2 us only.)
    if (ipt <= 1) {
      launch(topk_small<1, 1>, 1);
    } else if (ipt <= 2) {
      launch(topk_small<2, 1>, 1);
    } else if (ipt <= 4) {
      launch(topk_small<4, 1>, 1);
    } else if (ipt <= 8) {
      launch(topk_small<8, 1>, 1);
    } else if (ipt <= 16) {
      launch(topk_small<16, 2>, 2);
    } else if (ipt <= 20) {
      launch(topk_small<20, 4>, 4);
    } else if (ipt <= 24) {
      launch(topk_small<24, 4>, 4);
    } else if (ipt <= 28) {
      launch(topk_small<28, 4>, 4);
    } else {
      launch(topk_small<32, 4>, 4);
    }
    return hipGetLastError();
  }
  const int n_tiles = lg_tiles(dm);
  const size_t words = topk_ws_words(dm);
  if (!ws_is_zero) hipLaunchKernelGGL(topk_zero, dim3(256), dim3(256), 0, st, ws, words);
  dim3 grid((dm.T_cap + kLgTile - 1) / kLgTile, dm.n_kv, dm.b);
  hipLaunchKernelGGL((topk_hist<0>), grid, dim3(kLgThreads), 0, st, dm, scores, kv_lens, budgets, ws, n_tiles);
  hipLaunchKernelGGL((topk_hist<1>), grid, dim3(kLgThreads), 0, st, dm, scores, kv_lens, budgets, ws, n_tiles);
  hipLaunchKernelGGL((topk_hist<2>), grid, dim3(kLgThreads), 0, st, dm, scores, kv_lens, budgets, ws, n_tiles);
  hipLaunchKernelGGL((topk_finish<false>), grid, dim3(kLgThreads), 0, st, dm, scores, kv_lens, budgets, ws, n_tiles,
                     k_idx, k_cnt);
  hipLaunchKernelGGL((topk_finish<true>), grid, dim3(kLgThreads), 0, st, dm, scores, kv_lens, budgets, ws, n_tiles,
                     k_idx, k_cnt);
  return hipGetLastError();
}

}  // namespace quoka
