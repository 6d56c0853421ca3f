// Top-B key selection per (sequence, KV head) (Alg. 1: I = topk(S-hat, B_SA); Eq. 3).
//
// The cut (the B-th largest score) is found exactly, and an ordered compaction emits the positions of the scores above it
// and of the first ones equal to it: ascending, equal scores to the lower position.  Scores are compared as floats (-0
// equals +0, a NaN ranks as the infinity of its sign), or as order-preserving images that compare alike, so the result is
// deterministic and does not depend on the launch shape.
//
//   T_max <= kSmallMax : one to four blocks per head, scores held in registers, one launch; the cut from a
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
// bin than are ranked (cut_keys), or the scores admit no such bins, the block-wide radix select decides.
// The ordered compaction needs no scan over threads: per register, one wave ballot (two where only some of the keys
// equal to the cut are taken) gives every lane the number of earlier taken positions of its wave; how many earlier waves
// take follows from their counts above the cut's bin and from the positions in the list of that bin's keys.
//
// What bounds it: one compute unit's instruction rate (four passes over the keys, and 16 waves that each do what is done per
// wave: letting every wave scan the histogram for itself to save two barriers took 1 - 2 us more).  So from 8 keys per
// thread on, several blocks take a head: all of them find the cut, each emits its share of the waves' ranges.
// Measured (us, radix select on key bits and one block a head -> histogram -> now: wave reductions on integer images, bins kept,
// counts in the pass that lists the candidates): 8 heads of 8192 scores 7.9 -> 6.4 -> 6.1, 8 of 32768 20.4 -> 13.2 -> 12.0, of
// 12000 8.1 -> 7.0.
constexpr int kCutBins = 2048;
// Candidates a block ranks; more are radix-selected, which goes over all keys of a thread again.  Ranking takes NT / (their number,
// rounded up) lanes a key.  Measured (us, ranked / radix-selected): 512 threads, 1000 scores, 96 candidates 4.7 / 5.3, 160 5.9 / 5.4;
// 1024 threads, 4 keys each, 200 7.3 / 7.6, 300 11.1 / 7.7; 16 keys 256 14.3 / 15.1, 350 16.3 / 15.3; 24 keys 400 19.5 / 20.3; 32 keys
// 460 23.4 / 25.7.
constexpr int cut_keys(int nt, int ipt) { return nt == 512 ? 128 : ipt <= 12 ? 256 : ipt <= 28 ? 64 + 16 * ipt : 512; }
template <int NT, int KEYS>
struct __align__(16) CutLds {
  uint32_t hist[kCutBins];
  float key[KEYS];                     // (read 16 bytes at a time)
  int pos[KEYS];
  uint32_t wmin[NT / 64], wmax[NT / 64], wsum[NT / 64];
  uint32_t above[NT / 64];             // a wave's scores in the bins above the cut's
  uint32_t n, bin, need, need_eq;
  float tau;
};

// Inverse of okey.
__device__ __forceinline__ float okey_value(uint32_t k) {
  return __uint_as_float((k & 0x80000000u) ? k & 0x7FFFFFFFu : ~k);
}

template <int NT, int IPT, int NB>
__global__ __launch_bounds__(NT) void topk_small(Dims dm, const float* __restrict__ scores,
                                                const int32_t* __restrict__ kv_lens,
                                                const int32_t* __restrict__ budgets,
                                                int32_t* __restrict__ k_idx, int32_t* __restrict__ k_cnt) {
  constexpr int NW = NT / 64;
  constexpr int BPT = kCutBins / NT;   // bins per thread
  constexpr bool kKeepBins = IPT <= 16;
  __shared__ RadixSelectLds rs;
  constexpr int kCutKeys = cut_keys(NT, IPT);
  __shared__ CutLds<NT, kCutKeys> cl;
  __shared__ uint32_t wgt[NW], weq[NW];
  const int kv = blockIdx.x, b = blockIdx.y;
  const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const float* sc = scores + (size_t)(b * dm.n_kv + kv) * dm.T_max;
  const int w_lo = w * 64 * IPT, lo = w_lo + lane;   // positions of the wave, of register 0; register j is 64*j further
  // The scores are requested before the cache length is known (the row has T_max entries; those past the length
  // are discarded below), so the two fetches overlap instead of queueing behind each other.
  uint32_t rb[IPT];   // the scores' bits (the radix select borrows the registers for key images)
  auto val = [&](int j) __attribute__((always_inline)) { return __uint_as_float(rb[j]); };
#pragma unroll
  for (int j = 0; j < IPT; ++j) rb[j] = 0u;
  if (w_lo < dm.T_cap) {   // (wave-uniform)
#pragma unroll
    for (int j = 0; j < IPT; ++j) rb[j] = __float_as_uint(sc[min(lo + 64 * j, dm.T_cap - 1)]);
  }
  const int T = max(0, min(kv_lens[b * dm.ls], dm.T_cap));
  const int B = max(0, min(min(budgets[b * dm.ls], T), dm.B_max));
  int32_t* out = k_idx + (size_t)(b * dm.n_kv + kv) * dm.B_max;
  if (tid == 0 && blockIdx.z == 0) k_cnt[b * dm.n_kv + kv] = B;
  if (B == 0) return;
  if (B >= T) {
    for (int i = blockIdx.z * NT + tid; i < T; i += NB * NT) out[i] = i;
    return;
  }
#pragma unroll
  for (int i = 0; i < BPT; ++i) cl.hist[i * NT + tid] = 0u;
  if (tid == 0) cl.n = 0u;
  // positions past the length become NaN: minima and maxima pass over them and no comparison holds for them
  const bool full = w_lo + 64 * IPT <= T;   // (wave-uniform) no position of this wave is past the length
  float vmin = INFINITY, vmax = -INFINITY;
  bool nan = false;   // among the scores proper
  if (full) {
#pragma unroll
    for (int j = 0; j < IPT; ++j) {
      nan |= val(j) != val(j);
      vmin = fminf(vmin, val(j));
      vmax = fmaxf(vmax, val(j));
    }
  } else {
#pragma unroll
    for (int j = 0; j < IPT; ++j) {
      const bool past = lo + 64 * j >= T;
      nan |= !past && val(j) != val(j);
      if (past) rb[j] = 0x7FC00000u;
      vmin = fminf(vmin, val(j));
      vmax = fmaxf(vmax, val(j));
    }
  }
  {   // (as order-preserving images, whose reductions take one instruction a step; a NaN has the largest: no bins then)
    const uint32_t kmin = wave_min_u32(okey(vmin)), kmax = wave_max_u32(nan ? 0xFFFFFFFFu : okey(vmax));
    if (lane == 0) {
      cl.wmin[w] = kmin;
      cl.wmax[w] = kmax;
    }
  }
  __syncthreads();
  vmin = okey_value(row16_min_u32(cl.wmin[lane % NW]));
  vmax = okey_value(row16_max_u32(cl.wmax[lane % NW]));
  // monotone in v (a rounded product and a truncation of non-negative values), the largest score lands in the last bin
  const float per = ((float)kCutBins - 0.5f) / (vmax - vmin);
  const bool binned = per > 0.f && per < 1e30f;   // false for equal or infinite extremes, and where a score is NaN
  auto bin_of = [&](float v) __attribute__((always_inline)) { return min((int)((v - vmin) * per), kCutBins - 1); };
  float tau = 0.f;
  uint32_t need_eq = 0u, n_in = kCutKeys + 1, need = (uint32_t)B;
  int cut_bin = 0;
  if (binned) {   // block-uniform
    int bins[kKeepBins ? IPT : 1];   // (more of them would not fit the registers: they are worked out again)
#pragma unroll
    for (int j = 0; j < IPT; ++j) {
      const int bin = bin_of(val(j));
      if constexpr (kKeepBins) bins[j] = full || val(j) >= vmin ? bin : -1;
      if (full || val(j) >= vmin) atomicAdd(&cl.hist[bin], 1u);   // (not for a NaN)
    }
    __syncthreads();
    uint32_t hv[BPT], mine = 0;   // thread 0 has the highest bins
#pragma unroll
    for (int i = 0; i < BPT; ++i) {
      hv[i] = cl.hist[kCutBins - 1 - (tid * BPT + i)];
      mine += hv[i];
    }
    const uint32_t upto = wave_incl_scan_u32(mine);
    if (lane == 63) cl.wsum[w] = upto;
    __syncthreads();
    const uint32_t earlier = lane % 16 < NW && lane % 16 < w ? cl.wsum[lane % 16] : 0u;
    uint32_t above = row16_sum_u32(earlier) + upto - mine;
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
    if constexpr (!kKeepBins) asm volatile("" : "+v"(vmin));
    uint32_t n_above = 0;
#pragma unroll
    for (int j = 0; j < IPT; ++j) {
      int bin;
      if constexpr (kKeepBins) {
        bin = bins[j];
      } else {
        bin = full || val(j) >= vmin ? bin_of(val(j)) : -1;
      }
      n_above += bin > cut_bin ? 1u : 0u;
      if (bin == cut_bin) {
        const uint32_t slot = atomicAdd(&cl.n, 1u);
        if (slot < (uint32_t)kCutKeys) {
          cl.key[slot] = val(j);
          cl.pos[slot] = lo + 64 * j;
        }
      }
    }
    n_above = wave_incl_scan_u32(n_above);
    if (lane == 63) cl.above[w] = n_above;
    __syncthreads();
    n_in = cl.n;
  }
  uint32_t n_gt, n_eq, all_eq;     // taken candidates at earlier positions, above the cut / equal to it; all that are equal to it
  if (n_in <= (uint32_t)kCutKeys) {   // block-uniform
    // the cut: `need` of the bin's keys are taken, the largest.  P neighbouring lanes rank one key.
    int cap = NT / 16;
    while (cap < (int)n_in) cap <<= 1;
    const int P = NT / cap;   // 16 .. 2
    static_assert(kCutKeys <= NT / 2 && kCutKeys % 4 == 0, "");
    const int e = tid / P, part = tid % P;
    const float k = cl.key[min(e, (int)n_in - 1)];
    uint32_t cnt = 0;   // keys greater (low half), greater or equal (high half)
    auto count = [&](float o) __attribute__((always_inline)) { cnt += (o > k ? 1u : 0u) + (o >= k ? 0x10000u : 0u); };
    int j = part;
    if (n_in > NT / 16u) {   // four at a time
      for (j = 4 * part; j + 3 < (int)n_in; j += 4 * P) {
        const float4 o = *reinterpret_cast<const float4*>(&cl.key[j]);
        count(o.x); count(o.y); count(o.z); count(o.w);
      }
      j = ((int)n_in & ~3) + part;
    }
    for (; j < (int)n_in; j += P) count(cl.key[j]);
    for (int o = 1; o < P; o <<= 1) cnt += (uint32_t)__shfl_xor((int)cnt, o, kWave);
    if (e < (int)n_in && (cnt & 0xFFFFu) < need && need <= (cnt >> 16)) {   // (equal keys all write the same)
      cl.tau = k;
      cl.need_eq = need - (cnt & 0xFFFFu);
    }
    __syncthreads();
    if (NB > 1 && w / (NW / NB) != (int)blockIdx.z) return;   // (no barrier follows) another block emits this wave's range
    tau = cl.tau;
    need_eq = cl.need_eq;
    uint32_t gt = lane < w ? cl.above[min(lane, NW - 1)] : 0u, eq = 0;
    for (int i = lane; i < (int)n_in; i += kWave) {
      const float k = cl.key[i];
      const bool earlier = cl.pos[i] < w_lo;
      gt += earlier && k > tau ? 1u : 0u;
      eq += (earlier && k == tau ? 1u : 0u) + (k == tau ? 0x10000u : 0u);   // (at most kCutKeys each)
    }
    n_gt = (uint32_t)__builtin_amdgcn_readlane((int)wave_incl_scan_u32(gt), 63);
    eq = (uint32_t)__builtin_amdgcn_readlane((int)wave_incl_scan_u32(eq), 63);
    n_eq = eq & 0xFFFFu;
    all_eq = eq >> 16;
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
    block_radix_select<IPT, true, NT>(rb, in_bin, need, rs, &tau_key, &need_eq);
    tau = okey_value(tau_key);
#pragma unroll
    for (int j = 0; j < IPT; ++j) rb[j] = __float_as_uint(okey_value(rb[j]));
    // wave totals of scores above the cut and equal to it
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
    __syncthreads();
    if (NB > 1 && w / (NW / NB) != (int)blockIdx.z) return;   // (as above)
    all_eq = wave_incl_scan_u32(lane < NW ? weq[lane] : 0u);
    n_gt = wave_incl_scan_u32(lane < w ? wgt[lane] : 0u);
    n_eq = wave_incl_scan_u32(lane < w ? weq[lane] : 0u);
    all_eq = (uint32_t)__builtin_amdgcn_readlane((int)all_eq, 63);
    n_gt = (uint32_t)__builtin_amdgcn_readlane((int)n_gt, 63);
    n_eq = (uint32_t)__builtin_amdgcn_readlane((int)n_eq, 63);
  }
  const bool take_all_eq = all_eq == need_eq;
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
    auto launch = [&](auto kernel, int threads, int blocks_per_head) {
      hipLaunchKernelGGL(kernel, dim3(dm.n_kv, dm.b, blocks_per_head), dim3(threads), 0, st, dm, scores, kv_lens, budgets, k_idx,
                         k_cnt);
    };
    // (The time goes with the keys a thread holds, so above 8 the variants lie close together: 8 heads of 12000 scores 7.6 us with
    // 16 keys a thread, 7.0 with 12; 8 of 24000 11.0 with 32, 9.9 with 24.  Half the threads for short heads: 8 of 512 4.5 -> 4.2,
    // of 2048 4.9 -> 4.7; longer ones want the other half back, 8 of 8192 6.0 against 6.6.)
    const int T = dm.T_cap;
    if (T <= 512) {
      launch(topk_small<512, 1, 1>, 512, 1);
    } else if (T <= 1024) {
      launch(topk_small<512, 2, 1>, 512, 1);
    } else if (T <= 2048) {
      launch(topk_small<512, 4, 1>, 512, 1);
    } else if (T <= 4096) {
      launch(topk_small<1024, 4, 1>, 1024, 1);
    } else if (T <= 8192) {
      launch(topk_small<1024, 8, 1>, 1024, 1);
    } else if (T <= 12288) {
      launch(topk_small<1024, 12, 2>, 1024, 2);
    } else if (T <= 16384) {
      launch(topk_small<1024, 16, 2>, 1024, 2);
    } else if (T <= 20480) {
      launch(topk_small<1024, 20, 4>, 1024, 4);
    } else if (T <= 24576) {
      launch(topk_small<1024, 24, 4>, 1024, 4);
    } else if (T <= 28672) {
      launch(topk_small<1024, 28, 4>, 1024, 4);
    } else {
      launch(topk_small<1024, 32, 4>, 1024, 4);
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
