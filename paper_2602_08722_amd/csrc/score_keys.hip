// Key scoring (Alg. 1: K normalisation, S = Qbar K^T, S-hat = max over the query axis; Sec. 3.2-3.3).
//
// scores[b,kv,t] = max_r <Qbar[b,kv,r,:], K[b,kv,t,:]> / max(||K[b,kv,t,:]||, eps).
// The 1/||k|| factor is positive, so it is applied after the max; S itself is never stored.
//
// bf16 keys: the K cache is streamed once from HBM in 128-key tiles (coalesced 16-byte loads, double
// buffered through LDS).  Qbar (float32) is split into three bf16 terms hi + mid + lo that add up to the
// float32 value exactly, so with bf16 keys every MFMA product is exact and only the float32
// accumulation rounds.  Queries are the M side of v_mfma_f32_32x32x16_bf16, keys the N side: a lane
// owns one key column and 16 query rows, so the max over queries is in-register plus one
// half-wave exchange.
// float32 keys: float32 MFMA, operands straight from global memory; few queries: plain FMAs, one key per thread.
#include <type_traits>

#include "common.hip.h"
#include "kernels.h"
#include "qbar_row.hip.h"
#include "score_tile.hip.h"
#include "select_ws.hip.h"

namespace quoka {

// EXACT: Qbar enters as the three-term split (float32-exact products).  Otherwise it is rounded to bf16 once and
// only that term is multiplied: a third of the matrix work, scores within 2^-9 * sum|qbar_i| of the exact ones.
// PACK (QB = 1, EXACT): at most kPackRows queries, all three terms in one operand.
// FUSE (PACK, every query retained): Qbar is not there yet.  Every block works its head's few rows out for itself, in
// place of reading them (8 heads, 8192 keys, one query: a launch of 3.4 us saved, 1 us added here; call 26.1 -> 25.0 us).
// HIST: the scores are also counted in the head's histogram of kScoreBins bins (hist_ws: the zeroed head of the selection's
// workspace), in LDS first, so that the selection starts from the finished histogram.  Its blocks share out what the caches
// hold, not what there is room for: a sequence's blocks its tiles, and in a batch a KV head's blocks the tiles of all sequences
// (with a fixed share of T_cap most had nothing to do in a long cache that is not full yet, or in the shorter ones of a batch).
// Whole calls, fixed share -> this: 8 heads, room for 131072 keys, 64 queries, over 8000 keys 74.6 -> 42.1 us, 33000 74.1 -> 53.9,
// 131072 93.4 -> 92.9; 2 heads of 13 sequences, one of 42306 keys and twelve of 2000 82.5 -> 56.9; batches of equal lengths
// 0.99 - 1.02 of the time.
// TERMS: the query operands lie ready in `terms`.  (A template parameter: as a run-time choice it cost the calls that
// convert Qbar themselves 1.5 us, 2 x 8 heads of 8337 keys 12.0 -> 13.7.)
template <int D, int QB, bool EXACT, bool PACK, bool FUSE, bool TERMS, bool HIST>
__global__ __launch_bounds__(kScThreads, 2) void score_bf16(Dims dm, const float* __restrict__ qbar,
                                                           const uint16_t* __restrict__ kc,
                                                           const int32_t* __restrict__ kv_lens,
                                                           float* __restrict__ scores, int n_keep, int tiles_per_wg,
                                                           uint32_t* __restrict__ zero, uint32_t zero_words,
                                                           FusedQbar fq, const uint16_t* __restrict__ terms,
                                                           uint32_t* __restrict__ hist_ws) {
  using Cfg = ScoreCfg<D, QB>;
  const int len = HIST ? 0 : kv_lens[blockIdx.z * dm.ls];
  constexpr int LD = Cfg::LD, CG = Cfg::CG, RPI = Cfg::RPI, NLD = Cfg::NLD;
  extern __shared__ __align__(16) unsigned char smem[];
  uint16_t* tile0p = reinterpret_cast<uint16_t*>(smem);
  uint16_t* tile1p = reinterpret_cast<uint16_t*>(smem + Cfg::kTileBytes);
  float* ssq = reinterpret_cast<float*>(smem + 2 * Cfg::kTileBytes);   // [3][kScTile]
  float* smax = ssq + 3 * kScTile;                                       // [3][QB][kScTile]
  uint32_t* bins = reinterpret_cast<uint32_t*>(smem + Cfg::kLdsBytes);   // HIST: two bins a word
  if constexpr (HIST) {
    for (int i = threadIdx.x; i < kScoreBins / 2; i += kScThreads) bins[i] = 0u;   // (a barrier follows before the first count)
  }

  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int qb = w % QB, kg = w / QB;
  const int li = lane & 31, hf = lane >> 5;

  const int kv = blockIdx.y;
  int b = blockIdx.z;
  int t_begin = blockIdx.x * tiles_per_wg * kScTile;
  // (HIST: `zero_words` is the number of blocks of a KV head, or with tiles_per_wg == 0 of all its sequences together, among which
  // they are shared out; as grid sizes these would be fetched by a load of their own, a call of one head 1 us longer)
  const bool shared = HIST && tiles_per_wg == 0;
  const int blocks = (int)zero_words;
  if (shared) {
    const uint32_t tiles = lane < dm.b ? (uint32_t)(max(min(kv_lens[lane * dm.ls], dm.T_cap), 0) + kScTile - 1) / kScTile : 0u;
    const uint32_t total = max((uint32_t)__builtin_amdgcn_readlane((int)wave_incl_scan_u32(tiles), 63), 1u);
    const uint32_t n = min(tiles, 1u + tiles * (uint32_t)(blocks - dm.b) / total);   // (2^17 keys and 512 blocks at most)
    const uint32_t upto = wave_incl_scan_u32(n);
    const unsigned long long mine = __builtin_amdgcn_ballot_w64(blockIdx.x >= upto - n && blockIdx.x < upto);
    if (mine == 0) return;   // block-uniform
    b = (int)__builtin_ctzll(mine);
    const int nb = __builtin_amdgcn_readlane((int)n, b), first = __builtin_amdgcn_readlane((int)(upto - n), b);
    tiles_per_wg = (__builtin_amdgcn_readlane((int)tiles, b) + nb - 1) / nb;
    t_begin = ((int)blockIdx.x - first) * tiles_per_wg * kScTile;
  }

  // rows of this (batch, KV head) are addressed as base + 32-bit byte offset (the host checks the 4 GiB span)
  const char* kbase = reinterpret_cast<const char*>(kc + b * dm.kvs[0] + kv * dm.kvs[1]);
  opaque(kbase);
  const uint32_t row_bytes = (uint32_t)dm.kvs[2] * 2u;
  float* sc = scores + (size_t)(b * dm.n_kv + kv) * dm.T_max;
  const int cg = tid % CG, r0 = tid / CG;

  // two tiles are kept in flight: even tiles travel through RA, odd tiles through RB
  u32x4 RA[NLD], RB[NLD];
  auto issue = [&](int it, u32x4 (&R)[NLD]) __attribute__((always_inline)) {
    const int t0 = t_begin + it * kScTile;
#pragma unroll
    for (int i = 0; i < NLD; ++i) {
      // rows are clamped to the cache extent, not to the sequence length: loads then do not wait for the length, and
      // rows past it (allocated, arbitrary content) only produce scores that are never stored
      const int row = min(t0 + r0 + RPI * i, dm.T_max - 1);
      R[i] = *reinterpret_cast<const u32x4*>(kbase + ((uint32_t)row * row_bytes + (uint32_t)cg * 16u));
    }
  };
  // FUSE: the queries of the wave's first row, ahead of the keys (fetches arrive in order, and these are few)
  QbarRows<D> q_first;
  if constexpr (FUSE) q_first.load(dm, static_cast<const uint16_t*>(fq.q), min(w, n_keep - 1), kv, b, lane);
  // The first K tile is in flight while the length arrives and the query operands are prepared.  (Past the end of a sequence it is fetched
  // for nothing: in ten random batches with lengths up to eight times apart this launch takes 1.025 of the time that it takes with the fetch
  // behind the length; in the other 71 calls 0.995, and a prompt of 16000 466.7 us without and 458.5 with it.)
  if constexpr (!HIST) {
    issue(0, RA);
    asm volatile("" ::: "memory");   // (or the compiler moves these fetches behind the length's arrival)
    clear_words(zero, zero_words);
  }
  const int T = min(HIST ? kv_lens[b * dm.ls] : len, dm.T_cap);
  if constexpr (HIST) {
    if (!shared && T != dm.T_cap) {   // the cache is not full
      tiles_per_wg = (max(T, 0) + kScTile * blocks - 1) / (kScTile * blocks);
      t_begin = blockIdx.x * tiles_per_wg * kScTile;
    }
    if (t_begin >= T) return;   // block-uniform
    issue(0, RA);
  }
  const float* qhead = qbar + (size_t)(b * dm.n_kv + kv) * n_keep * D;
  if constexpr (FUSE) {
    __shared__ __align__(16) float qrows[kPackRows * D];   // (read 16 bytes at a time)
    if (t_begin >= T && blockIdx.x != 0) return;   // block-uniform
    constexpr int EPL = D / 64;
    for (int r = w; r < n_keep; r += kScThreads / 64) {
      float row[EPL];
      const uint16_t* q = static_cast<const uint16_t*>(fq.q);
      if (r != w) q_first.load(dm, q, r, kv, b, lane);
      if (dm.g <= 4) {
        qbar_row<uint16_t, D, kIdentity, 4, true>(dm, q, fq.q_idx, n_keep, r, kv, b, lane, blockIdx.x == 0, row, &q_first);
      } else {
        qbar_row<uint16_t, D, kIdentity, 8, false>(dm, q, fq.q_idx, n_keep, r, kv, b, lane, blockIdx.x == 0, row, &q_first);
      }
#pragma unroll
      for (int e = 0; e < EPL; ++e) {
        qrows[r * D + lane * EPL + e] = row[e];
        if (blockIdx.x == 0) fq.qbar[((size_t)(b * dm.n_kv + kv) * n_keep + r) * D + lane * EPL + e] = row[e];
      }
    }
    __syncthreads();
    qhead = qrows;
  }
  if (t_begin >= T) return;  // block-uniform
  const int n_tiles = min(tiles_per_wg, (T - t_begin + kScTile - 1) / kScTile);
  // The second K tile: ahead of operands that are converted here, and so waited for; behind those that lie ready, which the first tile's
  // products need.
  if (!TERMS && n_tiles > 1) issue(1, RB);

  const bool dot_mode = (dm.flags & 1) != 0, mean_mode = (dm.flags & 2) != 0;   // ablation scorers
  typename std::conditional<PACK, PackedTerms<D>, QueryTerms<D, EXACT>>::type qt;   // this wave's 32 query rows
  if constexpr (PACK) {
    qt.load(qhead, n_keep, li, hf);
  } else if constexpr (TERMS) {
    qt.load_terms(terms + (size_t)(b * dm.n_kv + kv) * TermsLayout<D>::head_elems(n_keep), n_keep, qb, li, hf);
  } else {
    qt.load(qhead, n_keep, qb, li, hf, mean_mode);
  }
  if (TERMS && n_tiles > 1) issue(1, RB);

  // scores of tile `it` from the maxima and squared norms of generation it % 3
  auto finish = [&](int it) {
    if (tid < kScTile) {
      const int key = t_begin + it * kScTile + tid;
      if (key < T) {
        const float s = tile_score<QB>(smax + (it % 3) * QB * kScTile, ssq + (it % 3) * kScTile, tid, dot_mode, mean_mode,
                                       n_keep);
        sc[key] = s;
        if constexpr (HIST) {
          const int bin = coarse_bin<kScoreBins>(s);
          atomicAdd(&bins[bin >> 1], 1u << (16 * (bin & 1)));
        }
      }
    }
  };

  auto tile_step = [&](int it, u32x4 (&R)[NLD]) __attribute__((always_inline)) {
    uint16_t* tl = (it & 1) ? tile1p : tile0p;
    float* ssq_g = ssq + (it % 3) * kScTile;
    float* smax_g = smax + (it % 3) * QB * kScTile;
#pragma unroll
    for (int i = 0; i < NLD; ++i) {
      const int rl = r0 + RPI * i;
      *reinterpret_cast<u32x4*>(tl + rl * LD + cg * 8) = R[i];
      if constexpr (!PACK) {
        const float ss = row_sumsq<CG>(R[i]);
        if (cg == 0) ssq_g[rl] = ss;
      }
    }
    // One barrier per tile.  It publishes tile `it` (and its squared norms) and the maxima of tile it-1.  The K tile
    // buffer written above was last read two steps ago, before the previous barrier; the norm / maximum generation
    // written in this step was last read (by finish) three steps ago, two barriers back.
    __syncthreads();
    if (it + 2 < n_tiles) issue(it + 2, R);  // the registers are free again: fetch the tile after the next
    if (it > 0) finish(it - 1);

    if constexpr (PACK) {
      const int key = w * 32 + li;
      const uint16_t* kp = tl + key * LD + hf * (D / 2);
      bf16x8 kop[D / 16];
#pragma unroll
      for (int ks = 0; ks < D / 16; ++ks) kop[ks] = *reinterpret_cast<const bf16x8*>(kp + ks * 8);
      float ss;
      const float m = packed_products<D>(kop, qt, &ss);
      if (hf == 0) {
        smax_g[key] = m;
        ssq_g[key] = ss;
      }
    } else {
      tile_products<D, QB, EXACT>(tl, qt, qb, kg, li, hf, mean_mode, smax_g);
    }
  };
  for (int it = 0; it < n_tiles; it += 2) {
    tile_step(it, RA);
    if (it + 1 < n_tiles) tile_step(it + 1, RB);
  }
  __syncthreads();
  finish(n_tiles - 1);
  if constexpr (HIST) {
    __syncthreads();
    const int heads = dm.b * dm.n_kv;
    uint32_t* hist = exact_hist(hist_ws, heads, b * dm.n_kv + kv, (int)blockIdx.x % exact_hist_copies(heads));
    for (int i = tid; i < kScoreBins / 2; i += kScThreads) {
      const uint32_t c = bins[i];
      if (c & 0xFFFFu) atomicAdd(&hist[2 * i], c & 0xFFFFu);
      if (c >> 16) atomicAdd(&hist[2 * i + 1], c >> 16);
    }
  }
}

// ---------------------------------------------------------------------------------------------
// float32 keys: float32 matrix instructions (v_mfma_f32_32x32x2_f32), so only the accumulation rounds.  A wave owns one
// block of 32 queries (operand held in registers) and takes 32 keys at a time, straight from global memory: lane
// (li, hf) reads dims 8i + 4*hf .. +4 of key li for i = 0 .. D/8-1, and step (i, e) contracts dims 8i + e and 8i + 4 + e.
// Bound by the latency of one row fetch and the D instructions of 64 clocks that follow it; measured at 2 x 4096 keys,
// 64 queries, d 128: 45 us for one key per thread with plain FMAs, 9 us here.
template <int D, int QB>
__global__ __launch_bounds__(kScThreads) void score_f32(Dims dm, const float* __restrict__ qbar,
                                                       const float* __restrict__ kc,
                                                       const int32_t* __restrict__ kv_lens, float* __restrict__ scores,
                                                       int n_keep, uint32_t* __restrict__ zero, uint32_t zero_words) {
  constexpr int NI = D / 8;
  constexpr int KPB = 32 * (4 / QB);   // keys per block and step
  typedef float f32x4 __attribute__((ext_vector_type(4)));
  __shared__ float smax[2][QB][KPB];
  const int kv = blockIdx.y, b = blockIdx.z;
  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int qb = w % QB, kb = w / QB;
  const int li = lane & 31, hf = lane >> 5;
  const bool dot_mode = (dm.flags & 1) != 0, mean_mode = (dm.flags & 2) != 0;   // ablation scorers
  const int len = kv_lens[b * dm.ls];
  const char* khead = reinterpret_cast<const char*>(kc + b * dm.kvs[0] + kv * dm.kvs[1]);
  opaque(khead);
  const char* kbase = khead + 16 * hf;
  const uint32_t row_bytes = (uint32_t)dm.kvs[2] * 4u;
  f32x4 kreg[NI];
  auto load_k = [&](int t0) __attribute__((always_inline)) {   // clamped to the cache extent: no wait for the length
    const uint32_t off = (uint32_t)min(t0 + kb * 32 + li, dm.T_max - 1) * row_bytes;
#pragma unroll
    for (int i = 0; i < NI; ++i) kreg[i] = *reinterpret_cast<const f32x4*>(kbase + off + 32 * i);
  };
  int t0 = blockIdx.x * KPB;
  load_k(t0);
  // query operand: row qb*32 + li (rows past n_keep repeat a real query, or are zero where a mean is taken), fetched beside the keys
  // and the length
  f32x4 qreg[NI];
  const int r = qb * 32 + li;
  const bool pad = r >= n_keep;
  {
    const float* qhead = qbar + (size_t)(b * dm.n_kv + kv) * n_keep * D;
    opaque(qhead);
    const float* qrow = qhead + (pad ? n_keep - 1 : r) * D + 4 * hf;
#pragma unroll
    for (int i = 0; i < NI; ++i) qreg[i] = *reinterpret_cast<const f32x4*>(qrow + 8 * i);
  }
  asm volatile("" ::: "memory");   // (or the compiler moves all of these fetches behind the length's arrival)
  clear_words(zero, zero_words);
  const int T = min(len, dm.T_cap);
  if (t0 >= T) return;   // block-uniform
  const bool round_q = (dm.flags & QUOKA_SCORE_QBAR_BF16) != 0;   // reduced-precision scorer: Qbar as bf16 values
  if (round_q || mean_mode) {   // (kernel-uniform)
#pragma unroll
    for (int i = 0; i < NI; ++i) {
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        if (round_q) qreg[i][e] = bf16_bits_to_f32(f32_to_bf16_bits(qreg[i][e]));
        if (mean_mode && pad) qreg[i][e] = 0.f;
      }
    }
  }
  float* sc = scores + (size_t)(b * dm.n_kv + kv) * dm.T_max;
  for (int par = 0; t0 < T; t0 += gridDim.x * KPB, par ^= 1) {
    float ss = 0.f;
    f32x16 c;
#pragma unroll
    for (int v = 0; v < 16; ++v) c[v] = 0.f;
#pragma unroll
    for (int i = 0; i < NI; ++i)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        c = __builtin_amdgcn_mfma_f32_32x32x2f32(qreg[i][e], kreg[i][e], c, 0, 0, 0);
        ss = fmaf(kreg[i][e], kreg[i][e], ss);
      }
    if (t0 + (int)gridDim.x * KPB < T) load_k(t0 + gridDim.x * KPB);
    ss += other_half(ss);
    float m = mean_mode ? 0.f : -INFINITY;
#pragma unroll
    for (int v = 0; v < 16; ++v) m = mean_mode ? m + c[v] : fmaxf(m, c[v]);
    m = mean_mode ? m + other_half(m) : fmaxf(m, other_half(m));
    const int k = kb * 32 + li;
    if constexpr (QB > 1) {   // the waves of the other query blocks hold the same keys; the buffers alternate, so one
      if (hf == 0) smax[par][qb][k] = m;   // barrier a step is enough
      __syncthreads();
      m = smax[par][0][k];
#pragma unroll
      for (int j = 1; j < QB; ++j) m = mean_mode ? m + smax[par][j][k] : fmaxf(m, smax[par][j][k]);
    }
    if (mean_mode) m /= (float)n_keep;
    if (qb == 0 && hf == 0 && t0 + k < T) sc[t0 + k] = m / (dot_mode ? 1.0f : fmaxf(sqrtf(ss), kNormEps)) + 0.0f;
  }
}

// The same for few queries, of which a matrix instruction would hold 32 whatever their number: one key per thread, its row in
// registers, Qbar from LDS.  Bound by the fetch of the rows, and by D FMAs a query where the keys are few.  Measured,
// matrix instructions -> this kernel: 8 x 8 heads of 4000 keys, d 128, 2 queries 39.2 -> 22.3 us, 16 queries 40.9 -> 33.4;
// 8 of 100000, d 64, 4 queries 58.6 -> 33.3; 2 of 4096, d 64, 2 queries 4.7 -> 4.2.
constexpr int kFewQueries = 26;
template <int D>
__global__ __launch_bounds__(kScThreads) void score_f32_few(Dims dm, const float* __restrict__ qbar,
                                                           const float* __restrict__ kc,
                                                           const int32_t* __restrict__ kv_lens,
                                                           float* __restrict__ scores, int n_keep,
                                                           uint32_t* __restrict__ zero, uint32_t zero_words) {
  __shared__ float qs[kFewQueries * D];
  clear_words(zero, zero_words);
  const int kv = blockIdx.y, b = blockIdx.z;
  const int T = min(kv_lens[b * dm.ls], dm.T_cap);
  if ((int)(blockIdx.x * kScThreads) >= T) return;   // block-uniform
  const float* qhead = qbar + (size_t)(b * dm.n_kv + kv) * n_keep * D;
  const bool round_q = (dm.flags & QUOKA_SCORE_QBAR_BF16) != 0;   // reduced-precision scorer: Qbar as bf16 values
  for (int i = threadIdx.x; i < n_keep * D; i += kScThreads)
    qs[i] = round_q ? bf16_bits_to_f32(f32_to_bf16_bits(qhead[i])) : qhead[i];
  __syncthreads();
  const int t = blockIdx.x * kScThreads + threadIdx.x;
  if (t >= T) return;
  const float* krow = kc + b * dm.kvs[0] + kv * dm.kvs[1] + (size_t)t * dm.kvs[2];
  float k[D];
  float ss = 0.f;
#pragma unroll
  for (int i = 0; i < D; i += 4) {
    const float4 x = *reinterpret_cast<const float4*>(krow + i);
    k[i] = x.x; k[i + 1] = x.y; k[i + 2] = x.z; k[i + 3] = x.w;
    ss += x.x * x.x; ss += x.y * x.y; ss += x.z * x.z; ss += x.w * x.w;
  }
  const bool dot_mode = (dm.flags & 1) != 0, mean_mode = (dm.flags & 2) != 0;   // ablation scorers
  float m = mean_mode ? 0.f : -INFINITY;
  for (int r = 0; r < n_keep; ++r) {
    const float* qr = qs + r * D;
    float dot = 0.f;
#pragma unroll
    for (int i = 0; i < D; ++i) dot += qr[i] * k[i];
    m = mean_mode ? m + dot : fmaxf(m, dot);
  }
  if (mean_mode) m /= (float)n_keep;
  scores[(size_t)(b * dm.n_kv + kv) * dm.T_max + t] = m / (dot_mode ? 1.0f : fmaxf(sqrtf(ss), kNormEps)) + 0.0f;
}

// Which of the two: the more keys, the more of the matrix instructions' time is not hidden, so the line rises with the keys.
// Both sides equal at 3 - 4 queries up to 32768 keys over all heads (one block of 128 for each compute unit); d 64: at 8 - 9 up
// to 98304, 26 - 28 from 262144 on; d 128: at 10 - 12 up to 65536, 18 - 20 at 98304, 22 - 25 from 262144 on.  The last bits of
// the scores depend on it: in a prompt it goes by the prompt's length and the batch of the whole call, like score_packs.
static bool score_f32_by_key(const Dims& dm, int n_keep) {
  const long long keys = (long long)(dm.prompt_chunks ? dm.ls : dm.b) * dm.n_kv * dm.T_max;
  if (keys <= 32768) return n_keep <= 3;
  if (dm.d == 64) return n_keep <= (keys <= 81920 ? 8 : keys < 10240 * kFewQueries ? keys / 10240 : kFewQueries);
  return n_keep <= (keys <= 65536 ? 10 : keys < 10240 * 13 ? 10 + keys / 10240 : 23);
}

template <int D>
static void launch_f32_d(const Dims& dm, const float* qbar, const float* kc, const int32_t* kv_lens, float* scores,
                         int n_keep, hipStream_t st, uint32_t* zero, uint32_t zero_words) {
  if (score_f32_by_key(dm, n_keep)) {
    const dim3 grid((dm.T_cap + kScThreads - 1) / kScThreads, dm.n_kv, dm.b);
    hipLaunchKernelGGL((score_f32_few<D>), grid, dim3(kScThreads), 0, st, dm, qbar, kc, kv_lens, scores, n_keep, zero,
                       zero_words);
    return;
  }
  const int qblocks = n_keep <= 32 ? 1 : (n_keep <= 64 ? 2 : 4);
  const int keys = 32 * (4 / qblocks);
  // one step per block up to four blocks a compute unit; longer caches keep the query operand over several steps
  int gx = (dm.T_cap + keys - 1) / keys;
  const int most = (1024 + dm.b * dm.n_kv - 1) / (dm.b * dm.n_kv);
  gx = gx < most ? gx : most;
  const dim3 grid(gx, dm.n_kv, dm.b);
  if (qblocks == 1) {
    hipLaunchKernelGGL((score_f32<D, 1>), grid, dim3(kScThreads), 0, st, dm, qbar, kc, kv_lens, scores, n_keep, zero,
                       zero_words);
  } else if (qblocks == 2) {
    hipLaunchKernelGGL((score_f32<D, 2>), grid, dim3(kScThreads), 0, st, dm, qbar, kc, kv_lens, scores, n_keep, zero,
                       zero_words);
  } else {
    hipLaunchKernelGGL((score_f32<D, 4>), grid, dim3(kScThreads), 0, st, dm, qbar, kc, kv_lens, scores, n_keep, zero,
                       zero_words);
  }
}

// ---------------------------------------------------------------------------------------------
// Tiles of a block, and blocks of a head.  Two blocks per compute unit are resident at once: aim for one round of 512 blocks, so
// the query operands (prepared once per block) are amortised over as many tiles as the launch allows
// -- except where the batch entries are chunks of a prompt, which share one cache of which the earlier ones see little:
// four rounds of shorter blocks even that out (prompt of 16000 in chunks of 1024, this launch 84 -> 57 us; 1024 blocks
// 84, 4096 64; for caches of one length each, 2048 blocks cost 10-17 %).  Whole calls, 512 -> 2048 blocks: 2 such prompts
// 1133 -> 1088 us, 30000 tokens, d 64 956 -> 923, 24000 in chunks of 2048 446 -> 432, 20000 in chunks of 500, 14/2 heads
// 364 -> 355, 9000 in chunks of 333, 12/4 heads 131 -> 124; 3000 - 6000 tokens within 0.5 %.
static int tiles_per_block(const Dims& dm) {
  const int nt = (dm.T_cap + kScTile - 1) / kScTile;
  const int heads = dm.b * dm.n_kv;
  const int wg_per_head = ((dm.prompt_chunks ? 2048 : 512) + heads - 1) / heads;
  const int tpw = (nt + wg_per_head - 1) / wg_per_head;
  return tpw < 1 ? 1 : tpw;
}

template <int D, int QB, bool EXACT, bool PACK = false, bool FUSE = false, bool TERMS = false, bool HIST = false>
static hipError_t launch_bf16(const Dims& dm, const float* qbar, const void* kc, const int32_t* kv_lens, float* scores,
                              int n_keep, hipStream_t st, uint32_t* zero, uint32_t zero_words, const FusedQbar& fq = {},
                              const uint16_t* terms = nullptr, uint32_t* hist_ws = nullptr) {
  using Cfg = ScoreCfg<D, QB>;
  constexpr size_t lds = Cfg::kLdsBytes + (HIST ? kScoreBins / 2 * sizeof(uint32_t) : 0);
  static_assert(lds <= 81920, "two blocks a compute unit");
  static std::atomic<uint64_t> lds_done{0};
  const hipError_t e =
      ensure_dynamic_lds(reinterpret_cast<const void*>(&score_bf16<D, QB, EXACT, PACK, FUSE, TERMS, HIST>), lds, lds_done);
  if (e != hipSuccess) return e;
  const int nt = (dm.T_cap + kScTile - 1) / kScTile;
  int tpw = tiles_per_block(dm);
  dim3 grid((nt + tpw - 1) / tpw, dm.n_kv, dm.b);
  if (HIST) {
    if (dm.b > 1 && dm.b <= kWave && 512 / dm.n_kv >= 2 * dm.b) {
      grid = dim3(512 / dm.n_kv, dm.n_kv, 1);
      tpw = 0;
    }
    zero_words = grid.x;
  }
  hipLaunchKernelGGL((score_bf16<D, QB, EXACT, PACK, FUSE, TERMS, HIST>), grid, dim3(kScThreads), lds, st, dm, qbar,
                     static_cast<const uint16_t*>(kc), kv_lens, scores, n_keep, tpw, zero, zero_words, fq,
                     terms, hist_ws);
  return hipGetLastError();
}

template <int D>
static hipError_t launch_bf16_d(const Dims& dm, const float* qbar, const void* kc, const int32_t* kv_lens,
                                float* scores, int n_keep, hipStream_t st, uint32_t* zero, uint32_t zero_words,
                                const FusedQbar& fq, const uint16_t* terms) {
  const int qblocks = (n_keep + 31) / 32;
  if (dm.flags & QUOKA_SCORE_QBAR_BF16) {
    if (qblocks <= 1) return launch_bf16<D, 1, false>(dm, qbar, kc, kv_lens, scores, n_keep, st, zero, zero_words);
    if (qblocks == 2) return launch_bf16<D, 2, false>(dm, qbar, kc, kv_lens, scores, n_keep, st, zero, zero_words);
    return launch_bf16<D, 4, false>(dm, qbar, kc, kv_lens, scores, n_keep, st, zero, zero_words);
  }
  if (fq.q != nullptr)
    return launch_bf16<D, 1, true, true, true>(dm, qbar, kc, kv_lens, scores, n_keep, st, zero, zero_words, fq);
  if (score_packs(dm)) return launch_bf16<D, 1, true, true>(dm, qbar, kc, kv_lens, scores, n_keep, st, zero, zero_words);
  if (terms != nullptr) {
    if (qblocks <= 1)
      return launch_bf16<D, 1, true, false, false, true>(dm, qbar, kc, kv_lens, scores, n_keep, st, zero, zero_words, {}, terms);
    if (qblocks == 2)
      return launch_bf16<D, 2, true, false, false, true>(dm, qbar, kc, kv_lens, scores, n_keep, st, zero, zero_words, {}, terms);
    return launch_bf16<D, 4, true, false, false, true>(dm, qbar, kc, kv_lens, scores, n_keep, st, zero, zero_words, {}, terms);
  }
  if (qblocks <= 1) return launch_bf16<D, 1, true>(dm, qbar, kc, kv_lens, scores, n_keep, st, zero, zero_words);
  if (qblocks == 2) return launch_bf16<D, 2, true>(dm, qbar, kc, kv_lens, scores, n_keep, st, zero, zero_words);
  return launch_bf16<D, 4, true>(dm, qbar, kc, kv_lens, scores, n_keep, st, zero, zero_words);
}

// The exact scores and their histogram, from `terms`.
template <int D>
static hipError_t launch_hist_d(const Dims& dm, const float* qbar, const void* kc, const int32_t* kv_lens, float* scores,
                                int n_keep, hipStream_t st, const uint16_t* terms, uint32_t* ws) {
  const int qblocks = (n_keep + 31) / 32;
  if (qblocks <= 1)
    return launch_bf16<D, 1, true, false, false, true, true>(dm, qbar, kc, kv_lens, scores, n_keep, st, nullptr, 0, {}, terms, ws);
  if (qblocks == 2)
    return launch_bf16<D, 2, true, false, false, true, true>(dm, qbar, kc, kv_lens, scores, n_keep, st, nullptr, 0, {}, terms, ws);
  return launch_bf16<D, 4, true, false, false, true, true>(dm, qbar, kc, kv_lens, scores, n_keep, st, nullptr, 0, {}, terms, ws);
}

hipError_t launch_score_hist(const Dims& dm, const float* qbar, const void* k_cache, const int32_t* kv_lens, float* scores,
                             hipStream_t st, const uint16_t* terms, uint32_t* hist_ws) {
  const int n_keep = dm.n_ret < dm.C ? dm.n_ret : dm.C;
  return dm.d == 64 ? launch_hist_d<64>(dm, qbar, k_cache, kv_lens, scores, n_keep, st, terms, hist_ws)
                    : launch_hist_d<128>(dm, qbar, k_cache, kv_lens, scores, n_keep, st, terms, hist_ws);
}

bool score_reads_terms(const Dims& dm, int dtype) {
  return dtype == QUOKA_BF16 && dm.T_cap > 0 && !score_packs(dm) && (dm.flags & (QUOKA_SCORE_MEAN | QUOKA_SCORE_QBAR_BF16)) == 0;
}

bool score_forms_qbar(const Dims& dm, int dtype) {
  return dtype == QUOKA_BF16 && dm.T_cap > 0 && dm.C <= dm.n_ret && score_packs(dm);
}

hipError_t launch_score_keys(const Dims& dm, int dtype, const float* qbar, const void* k_cache, const int32_t* kv_lens,
                             float* scores, hipStream_t st, uint32_t* zero, size_t zero_words_sz, const FusedQbar& fq,
                             const uint16_t* terms) {
  if (dm.T_cap <= 0) return hipSuccess;   // (then the top-k that follows takes no workspace either)
  const uint32_t zero_words = (uint32_t)zero_words_sz;
  const int n_keep = dm.n_ret < dm.C ? dm.n_ret : dm.C;
  if (dtype == QUOKA_BF16) {
    return dm.d == 64 ? launch_bf16_d<64>(dm, qbar, k_cache, kv_lens, scores, n_keep, st, zero, zero_words, fq, terms)
                      : launch_bf16_d<128>(dm, qbar, k_cache, kv_lens, scores, n_keep, st, zero, zero_words, fq, terms);
  }
  const float* kf = static_cast<const float*>(k_cache);
  if (dm.d == 64) {
    launch_f32_d<64>(dm, qbar, kf, kv_lens, scores, n_keep, st, zero, zero_words);
  } else {
    launch_f32_d<128>(dm, qbar, kf, kv_lens, scores, n_keep, st, zero, zero_words);
  }
  return hipGetLastError();
}

}  // namespace quoka
