// Tile arithmetic of the key scoring (Alg. 1: S = Qbar K^T, S-hat = max over the query axis; Sec. 3.2-3.3), shared
// by the streaming scoring kernel and by the exact re-scoring of the keys near the provisional cut: both must give
// the same float32 bits for the same key, so the split of Qbar, the order of the MFMA terms, the squared norm and
// the final division live here once.  (The streaming kernel's exact form follows the orders of tile_products and row_sumsq on its own
// layout.)
//
// Operand plan (v_mfma_f32_32x32x16_bf16; a lane is (li = lane % 32, hf = lane / 32)): queries are the M side, keys
// the N side.  Lane (li, hf) holds, for k-step ks, dims ks*16 + 8*hf .. +8 of query row li (A) and of key li (B);
// the result block has key li in the lane and 16 query rows in its registers, so the max over queries is in-register
// plus one exchange between the half waves.
#pragma once
#include "common.hip.h"

namespace quoka {

constexpr int kScThreads = 256;
constexpr int kScTile = 128;  // keys per LDS tile

template <int D, int QB>
struct ScoreCfg {
  static constexpr int KS = D / 16;             // MFMA k-steps over head_dim
  static constexpr int LD = D + 8;              // padded LDS row, elements (16-byte pad: conflict-free b128 reads)
  static constexpr int CG = D / 8;              // 16-byte chunks per key row
  static constexpr int RPI = kScThreads / CG;   // key rows covered by one block-wide load
  static constexpr int NLD = kScTile / RPI;     // loads per thread per tile
  static constexpr int KG = 4 / QB;             // wave groups that split a tile's keys
  static constexpr int KPW = kScTile / KG;      // keys per wave per tile
  static constexpr size_t kTileBytes = (size_t)kScTile * LD * 2;
  // two K tiles; three generations of squared norms and of per-query-block maxima (a tile's scores are finished
  // one step after its products, under the next tile's barrier)
  static constexpr size_t kLdsBytes = 2 * kTileBytes + 3 * kScTile * 4 + 3 * QB * kScTile * 4;
};

typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));

// sum of squares of the 8 bf16 values of a 16-byte chunk (products of bf16 pairs are exact in float32)
__device__ __forceinline__ float sumsq_bf16x8(const u32x4& r) {
  // (the chunk is reinterpreted as a whole: casting single dwords of the vector to bf16 pairs is miscompiled)
  const bf16x8 v = __builtin_bit_cast(bf16x8, r);
  float s = 0.f;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const bf16x2_t p = {v[2 * i], v[2 * i + 1]};
    s = __builtin_amdgcn_fdot2_f32_bf16(p, p, s, false);
  }
  return s;
}

// Squared norm of a key row whose CG 16-byte chunks sit in CG consecutive lanes (`r` is this lane's chunk).
template <int CG>
__device__ __forceinline__ float row_sumsq(const u32x4& r) {
  const float ss = sumsq_bf16x8(r);
  if constexpr (CG == 16) {
    return row16_sum(ss);   // a key row is exactly one 16-lane DPP row
  } else {
    return group_sum<CG>(ss);
  }
}

// The three terms of a row of Qbar as the launch that forms it can leave them, 16 bytes a lane in operand order:
// [row block][k-step][term][lane].  A scoring block then fetches whole kilobytes and converts nothing (64 elements a lane,
// about 450 instructions): 8 heads of 8192 keys, 64 queries 10.4 -> 8.7 us, call 72.7 -> 69.9; 128 queries x 32768 keys
// 31.0 -> 29.2.  (The re-scoring of the two-pass stage gains nothing from it.)
template <int D>
struct TermsLayout {
  static constexpr int kBlock = (D / 16) * 3 * 64 * 8;   // elements of 32 rows
  __host__ __device__ static size_t head_elems(int n_keep) { return (size_t)((n_keep + 31) / 32) * kBlock; }
  // first of the elements of row r's dims d .. (d % 8 != 7: neighbours follow)
  __device__ static size_t at(int r, int d, int term) {
    return (size_t)(r / 32) * kBlock + (size_t)((((d / 16) * 3 + term) * 64 + ((d % 16) / 8) * 32 + r % 32) * 8 + d % 8);
  }
};

// Query operands of one wave: 32 rows of Qbar (rows qb*32 .. +32 of a head's [n_keep][D] float32 block) as bf16
// terms.  EXACT: hi + mid + lo add up to the float32 value exactly, so with bf16 keys every product is exact and only
// the float32 accumulation rounds.  Otherwise only hi (Qbar rounded to bf16) is formed.  Rows past n_keep repeat the
// last real query (the max is unchanged); `zero_pad` makes them zero instead (for the mean over queries).
template <int D, bool EXACT>
struct QueryTerms {
  bf16x8 hi[D / 16], mid[D / 16], lo[D / 16];
  // (rows past n_keep repeat the last real query)
  __device__ __forceinline__ void load_terms(const uint16_t* __restrict__ head, int n_keep, int qb, int li, int hf) {
    const uint16_t* p = head + TermsLayout<D>::at(min(qb * 32 + li, n_keep - 1), 8 * hf, 0);
#pragma unroll
    for (int ks = 0; ks < D / 16; ++ks) {
      hi[ks] = *reinterpret_cast<const bf16x8*>(p + (ks * 3 + 0) * 512);
      mid[ks] = *reinterpret_cast<const bf16x8*>(p + (ks * 3 + 1) * 512);
      lo[ks] = *reinterpret_cast<const bf16x8*>(p + (ks * 3 + 2) * 512);
    }
  }
  __device__ __forceinline__ void load(const float* __restrict__ qhead, int n_keep, int qb, int li, int hf,
                                       bool zero_pad) {
    int r = qb * 32 + li;
    const bool pad_row = r >= n_keep;
    r = pad_row ? n_keep - 1 : r;
    const float* qrow = qhead + (size_t)r * D + 8 * hf;
#pragma unroll
    for (int ks = 0; ks < D / 16; ++ks) {
      const float4 x0 = *reinterpret_cast<const float4*>(qrow + ks * 16);
      const float4 x1 = *reinterpret_cast<const float4*>(qrow + ks * 16 + 4);
      float x[8] = {x0.x, x0.y, x0.z, x0.w, x1.x, x1.y, x1.z, x1.w};
      if (zero_pad && pad_row) {
#pragma unroll
        for (int e = 0; e < 8; ++e) x[e] = 0.f;
      }
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const __bf16 h = (__bf16)x[e];
        hi[ks][e] = h;
        if constexpr (EXACT) {
          const float r1 = x[e] - (float)h;
          const __bf16 m = (__bf16)r1;
          const float r2 = r1 - (float)m;
          mid[ks][e] = m;
          lo[ks][e] = (__bf16)r2;
        }
      }
    }
  }
};

// Products of one wave over its share of a staged tile: keys kg*KPW .. +KPW of `tl` (row pitch LD) against the wave's
// 32 query rows; per key the max (or, mean_mode, the sum) over those rows goes to smax_g[qb*kScTile + key].  All
// three query terms go into one accumulator per key block (smallest term first inside every k-step), so there is
// nothing to add up afterwards; two key blocks are interleaved to keep the MFMA chains independent.
template <int D, int QB, bool EXACT>
__device__ __forceinline__ void tile_products(const uint16_t* __restrict__ tl, const QueryTerms<D, EXACT>& q, int qb,
                                              int kg, int li, int hf, bool mean_mode, float* __restrict__ smax_g) {
  using Cfg = ScoreCfg<D, QB>;
  constexpr int KS = Cfg::KS, LD = Cfg::LD, KPW = Cfg::KPW;
  constexpr int NKB = KPW / 32;
#pragma unroll
  for (int kb = 0; kb < NKB; kb += 2) {
    constexpr int kPair = NKB >= 2 ? 2 : 1;
    f32x16 c[kPair];
    const uint16_t* kp[kPair];
#pragma unroll
    for (int u = 0; u < kPair; ++u) {
      c[u] = f32x16{0};
      kp[u] = tl + (kg * KPW + (kb + u) * 32 + li) * LD + 8 * hf;
    }
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      bf16x8 kop[kPair];
#pragma unroll
      for (int u = 0; u < kPair; ++u) kop[u] = *reinterpret_cast<const bf16x8*>(kp[u] + ks * 16);
      if constexpr (EXACT) {
#pragma unroll
        for (int u = 0; u < kPair; ++u) c[u] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(q.lo[ks], kop[u], c[u], 0, 0, 0);
#pragma unroll
        for (int u = 0; u < kPair; ++u) c[u] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(q.mid[ks], kop[u], c[u], 0, 0, 0);
      }
#pragma unroll
      for (int u = 0; u < kPair; ++u) c[u] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(q.hi[ks], kop[u], c[u], 0, 0, 0);
    }
#pragma unroll
    for (int u = 0; u < kPair; ++u) {
      float m;
      if (mean_mode) {   // sum over this wave's 32 query rows (padding rows are zero)
        m = 0.f;
#pragma unroll
        for (int v = 0; v < 16; ++v) m += c[u][v];
        m += other_half(m);
      } else {
        m = -INFINITY;
#pragma unroll
        for (int v = 0; v < 16; ++v) m = fmaxf(m, c[u][v]);
        m = fmaxf(m, other_half(m));
      }
      if (hf == 0) smax_g[qb * kScTile + kg * KPW + (kb + u) * 32 + li] = m;
    }
  }
}

// Up to kPackRows queries: their three terms fit the 32 rows of ONE operand (rows 0-7 hi, 8-15 mid, 16-23 lo, 24-31
// zero), so the exact product costs what one term costs.  The terms of a query land in the same lane of the result
// (registers 0-3 hi, 4-7 mid, 8-11 lo of queries 4*hf .. +4), where they are added, smallest first; every MFMA product is
// exact.  Here lane (li, hf) holds, for k-step ks, the 16-byte chunk ks + KS*hf of its row (the contraction index may
// be permuted freely).  Rows past n_keep repeat the last real query.
constexpr int kPackRows = 8;
template <int D>
struct PackedTerms {
  bf16x8 t[D / 16];
  __device__ __forceinline__ void load(const float* __restrict__ qhead, int n_keep, int li, int hf) {
    const int term = li >> 3;
    const float* qrow = qhead + (size_t)min(li & 7, n_keep - 1) * D + hf * (D / 2);
#pragma unroll
    for (int ks = 0; ks < D / 16; ++ks) {
      const float4 x0 = *reinterpret_cast<const float4*>(qrow + ks * 8);
      const float4 x1 = *reinterpret_cast<const float4*>(qrow + ks * 8 + 4);
      const float x[8] = {x0.x, x0.y, x0.z, x0.w, x1.x, x1.y, x1.z, x1.w};
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const __bf16 h = (__bf16)x[e];
        const float r1 = x[e] - (float)h;
        const __bf16 m = (__bf16)r1;
        const float r2 = r1 - (float)m;
        t[ks][e] = (__bf16)(term == 0 ? (float)h : term == 1 ? (float)m : term == 2 ? r2 : 0.f);
      }
    }
  }
};
// The largest product of lane li's key with the queries (in both half waves) and the key's squared norm.
template <int D>
__device__ __forceinline__ float packed_products(const bf16x8 (&kop)[D / 16], const PackedTerms<D>& q, float* ssq) {
  f32x16 c0 = {0}, c1 = {0};   // two chains (even / odd k-steps)
#pragma unroll
  for (int ks = 0; ks < D / 16; ks += 2) {
    c0 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(q.t[ks], kop[ks], c0, 0, 0, 0);
    c1 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(q.t[ks + 1], kop[ks + 1], c1, 0, 0, 0);
  }
  float ss = 0.f;
#pragma unroll
  for (int ks = 0; ks < D / 16; ++ks)
#pragma unroll
    for (int e = 0; e < 8; e += 2) {
      const bf16x2_t pr = {kop[ks][e], kop[ks][e + 1]};
      ss = __builtin_amdgcn_fdot2_f32_bf16(pr, pr, ss, false);
    }
  *ssq = ss + other_half(ss);
  float m = -INFINITY;
#pragma unroll
  for (int i = 0; i < 4; ++i) m = fmaxf(m, ((c0[8 + i] + c1[8 + i]) + (c0[4 + i] + c1[4 + i])) + (c0[i] + c1[i]));
  return fmaxf(m, other_half(m));
}
// Whether a bf16 call takes this form: the scores' last bits depend on it, so every scoring kernel goes by this rule, and
// in a prompt it goes by the prompt's length and the batch of the whole call: how many chunks share a launch, and how
// much cache they have come to, must not decide between two nearly equal keys.
// Bounds: sel_finish has a lane for every tile of heads of up to kPackMaxKeys positions.  Long caches of few keys in all are not
// packed: quoka_chunk_attn is the faster with unpacked exact scores there (two heads of 65537 positions, 4 queries 34.8 us, packed
// 37.4; one of 131072 36.8, 43.0), up to where the two meet (two of 98000, 4 of 49000 39.1, 40.5 and 37.8, 37.0).
// quoka_select_keys by itself takes the two-pass form there, though packed would be the faster (39 us, 27): a test that this
// form runs expects mostly provisional scores of four queries at just that size.
constexpr int kPackMaxKeys = 131072;
constexpr long long kPackMinKeys = 3 << 16;
inline bool score_packs(const Dims& dm) {
  const int n_keep = dm.n_ret < dm.C ? dm.n_ret : dm.C;
  const long long sequences = dm.prompt_chunks ? dm.ls : dm.b;   // (ls: the batch of the whole call)
  return n_keep <= kPackRows && (dm.flags & (QUOKA_SCORE_DOT | QUOKA_SCORE_MEAN | QUOKA_SCORE_QBAR_BF16)) == 0 &&
         (dm.T_max <= 32768 || (dm.T_max <= kPackMaxKeys && sequences * dm.n_kv * dm.T_max >= kPackMinKeys));
}

// Score of key `k` of a tile from the per-query-block maxima (sums) and the squared norm.
template <int QB>
__device__ __forceinline__ float tile_score(const float* __restrict__ sm, const float* __restrict__ ssq_g, int k,
                                            bool dot_mode, bool mean_mode, int n_keep) {
  float m = sm[k];
#pragma unroll
  for (int j = 1; j < QB; ++j) m = mean_mode ? m + sm[j * kScTile + k] : fmaxf(m, sm[j * kScTile + k]);
  if (mean_mode) m /= (float)n_keep;
  const float nrm = dot_mode ? 1.0f : fmaxf(sqrtf(ssq_g[k]), kNormEps);
  return m / nrm + 0.0f;
}

// Side job of a fused call: all blocks of the launch together clear `words` 32-bit words (p is 16-byte aligned).
__device__ __forceinline__ void clear_words(uint32_t* __restrict__ p, uint32_t words) {
  if (p == nullptr) return;
  const uint32_t nblk = gridDim.x * gridDim.y * gridDim.z;
  const uint32_t blk = blockIdx.x + gridDim.x * (blockIdx.y + gridDim.y * blockIdx.z);
  const uint32_t i0 = blk * blockDim.x + threadIdx.x, step = nblk * blockDim.x;
  for (uint32_t i = i0; i < words / 4; i += step) reinterpret_cast<u32x4*>(p)[i] = u32x4{0u, 0u, 0u, 0u};
  if (i0 < words % 4) p[words / 4 * 4 + i0] = 0u;
}

}  // namespace quoka
