// Attention for decode-sized chunks (Sec. 4.4: generation uses the same selection with B_CP = 1; Alg. 1 keeps every
// query when B_CP <= N_Q): the g * C query rows of one KV head fit one 32-row MFMA block, so the work is split over
// the KEY axis instead (split-KV): block (split, kv, b) attends its rows over one contiguous range of the key list
// [gathered cache rows | chunk rows] and writes an un-normalised partial (m, l, O); a second kernel merges the
// partials with the usual log-sum-exp rescale (Eq. 2-3 are unchanged, only the summation is regrouped).
//
// Rows: row r = c * g + j is chunk token c of q-head kv * g + j.  Keys: list slot n < n_cache is a cache row
// (k_idx[n] on the sparse path, n itself on the dense path), slot n_cache + p is chunk row p, visible to token c
// iff p <= c.
//
// Bound by memory: every row of K and V is used once, by one wave.  So a wave works by itself -- it fetches 32 slots at a
// time (index two tiles ahead, rows one tile ahead, whole rows by 16 lanes), turns them in its own piece of LDS and needs
// no barrier until its block's four waves are merged at the end -- and two blocks share a compute unit, which keeps
// 128 KiB of rows on the way.  The key list of a sequence is cut in proportion to its length, so the blocks of a ragged
// batch take equally long.
// Measured (kernel without the merge launch; 128-slot tiles that a block staged together, index and row fetched in turn,
// equal numbers of blocks per sequence -> now): 8 sequences x 8 heads, 12 % of 13000 - 65536 tokens, 157 MB: 77 -> 37 us;
// one sequence, 983 keys: 10.1 -> 6.1 us.
// MFMA operand plan as in the prefill kernel: S^T = K Q^T (query rows on lanes), O^T += V^T P^T with V^T fetched
// by the transposing LDS read.
#include <type_traits>

#include "common.hip.h"
#include "kernels.h"

namespace quoka {

typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef short s16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef s16x4 __attribute__((address_space(3))) * tr_ptr;

constexpr int kDcWaves = 4;
constexpr int kDcThreads = 64 * kDcWaves;
constexpr int kDcTile = 32;       // list slots a wave handles at a time
constexpr int kMaxSplits = 64;    // blocks per (sequence, KV head)
// (at most 32 rows of the chunk's own)
static_assert(((long long)kMaxKv / kDcTile + 2) * kMaxSplits < 1ll << 32, "tiles times shares in 32 bits");

template <int D>
struct DecodeCfg {
  static constexpr int KS = D / 16;
  static constexpr int LD = D + 8;        // K rows: 16 bytes of padding (conflict-free b128 reads)
  static constexpr int LDV = D + 32;      // V rows: 64 bytes apart modulo 256 (transposing reads)
  static constexpr int CG = D / 8;        // lanes per row (16 bytes each)
  static constexpr int RPI = 64 / CG;     // rows per wave-wide load
  static constexpr int NLD = kDcTile / RPI;
  static constexpr int DB = D / 32;
  static constexpr size_t kKBytes = (size_t)kDcTile * LD * 2;
  static constexpr size_t kWaveBytes = kKBytes + (size_t)kDcTile * LDV * 2;
  static constexpr int kRec = 32 * (D + 2);   // floats of a block's partial: O[32][D], m[32], l[32]
  static constexpr int LDO = D + 4;       // LDS pitch of a wave's output rows (floats): 16-byte writes, no conflicts
  static constexpr size_t kMergeBytes = (size_t)kDcWaves * 32 * (LDO + 3) * 4;   // output rows, m, l and weight of each
  static constexpr size_t kLdsBytes = kDcWaves * kWaveBytes > kMergeBytes ? kDcWaves * kWaveBytes : kMergeBytes;
};

// The blocks of one KV head, `n_slots` of them, over the sequences: sequence b gets 1 + floor(share * (n_slots - batch))
// of them, share its part of all tiles (never more than there are tiles for four waves each; more than 64 sequences:
// an equal number each).  Every wave works it out for itself; all lanes return the same.
struct DecodeShare {
  int n_splits;   // of sequence b
  int first;      // its first slot
};
struct DecodeWork {
  int b, split, n_splits;   // b < 0: nothing to do
};
__device__ __forceinline__ int decode_cache(const Dims& dm, const AttnArgs& a, int b, int kv) {
  const int n = a.k_idx != nullptr ? min(a.n_cache[b * dm.n_kv + kv], dm.B_max) : min(a.n_cache[b * dm.ls], dm.T_max);
  return max(n, 0);
}
__device__ __forceinline__ int decode_tiles(const Dims& dm, const AttnArgs& a, int b, int kv) {
  return (decode_cache(dm, a, b, kv) + dm.C + kDcTile - 1) / kDcTile;
}
// the splits of a call's only sequence
__device__ __forceinline__ int decode_splits_of_one(int tiles, int n_slots) {
  return min(min(n_slots, (tiles + kDcWaves - 1) / kDcWaves), kMaxSplits);
}
// lane i of the wave: the splits of sequence i, and the sum over the earlier ones in *before
__device__ __forceinline__ uint32_t decode_lane_splits(const Dims& dm, const AttnArgs& a, int kv, int n_slots,
                                                       uint32_t* before) {
  const int lane = threadIdx.x & 63;
  const uint32_t tiles = lane < dm.b ? (uint32_t)decode_tiles(dm, a, lane, kv) : 0u;
  const uint32_t total = (uint32_t)__builtin_amdgcn_readlane((int)wave_incl_scan_u32(tiles), 63);
  uint32_t n = lane < dm.b ? 1u + (uint32_t)((unsigned long long)tiles * (uint32_t)(n_slots - dm.b) / total) : 0u;
  n = min(n, max((tiles + kDcWaves - 1) / kDcWaves, lane < dm.b ? 1u : 0u));
  n = min(n, (uint32_t)kMaxSplits);
  *before = wave_incl_scan_u32(n) - n;
  return n;
}
__device__ __forceinline__ DecodeShare decode_share(const Dims& dm, const AttnArgs& a, int b, int kv, int n_slots) {
  if (dm.b == 1) return {decode_splits_of_one(decode_tiles(dm, a, 0, kv), n_slots), 0};
  if (dm.b > 64) return {n_slots / dm.b, b * (n_slots / dm.b)};
  uint32_t before;
  const uint32_t n = decode_lane_splits(dm, a, kv, n_slots, &before);
  return {__builtin_amdgcn_readlane((int)n, b), __builtin_amdgcn_readlane((int)before, b)};
}
__device__ __forceinline__ DecodeWork decode_work(const Dims& dm, const AttnArgs& a, int slot, int kv, int n_slots) {
  if (dm.b > 64) {
    const int n = n_slots / dm.b;
    return {slot < n * dm.b ? slot / n : -1, slot % n, n};
  }
  uint32_t before;
  const uint32_t n = decode_lane_splits(dm, a, kv, n_slots, &before);
  const unsigned long long mine = __builtin_amdgcn_ballot_w64((uint32_t)slot >= before && (uint32_t)slot < before + n);
  if (mine == 0) return {-1, 0, 0};
  const int b = (int)__builtin_ctzll(mine);
  return {b, slot - __builtin_amdgcn_readlane((int)before, b), __builtin_amdgcn_readlane((int)n, b)};
}

// part: [n_kv, n_slots, kRec] float32
// ONE: one sequence and a list.  The list mostly has the B_max entries that there is room for, so the first tile of such a list is
// looked up while the list's length travels: one fetch less in the chain, here and in the merge (32/8 heads, d 128, whole calls: 1 token
// over 983 keys 23.6 -> 22.6 us, this kernel alone 22.7; 5 over 4000 75.4 -> 74.5; batches, whose shares go by all the lengths,
// lost 1.4 % to it and stay as they were).
// LONG: waves with more than two tiles.  The queries have arrived before a tile's successor is requested.  Otherwise they count as on
// their way wherever the loop is entered again, and every tile's products wait for all that was requested after them, which is the next
// tile.  With two tiles and fewer that wait is the shorter one: the second tile leaves before the queries are there.  (32/8 heads, d 128, 1
// token: 8 sequences, 12 % of 16384 keys each 18.7 -> 17.3 us, of 4096 - 65536 33.1 -> 32.3; one, 12 % of 131072 18.3 -> 17.0; both launches.)
template <int D, bool ONE, bool LONG>
__global__ __launch_bounds__(kDcThreads, 2) void attn_decode_bf16(Dims dm, AttnArgs a, float* __restrict__ part,
                                                                  int n_slots) {
  using Cfg = DecodeCfg<D>;
  constexpr int KS = Cfg::KS, LD = Cfg::LD, LDV = Cfg::LDV, CG = Cfg::CG, RPI = Cfg::RPI, NLD = Cfg::NLD, DB = Cfg::DB,
                LDO = Cfg::LDO;
  extern __shared__ __align__(16) unsigned char smem[];
  const int kv = blockIdx.y;
  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int li = lane & 31, hf = lane >> 5;
  const int C = dm.C, g = dm.g;
  const int n_rows = C * g;   // <= 32, checked by the launcher
  const bool sparse = a.k_idx != nullptr;
  DecodeWork work{0, (int)blockIdx.x, 0};
  if constexpr (!ONE) {
    work = decode_work(dm, a, blockIdx.x, kv, n_slots);
    if (work.b < 0) return;   // block-uniform
  }
  const int b = work.b;
  int n_cache, n_keys, t_end, t;   // cache slots and all slots of the list; this wave's tiles: every fourth
  auto share_out = [&](int n) __attribute__((always_inline)) {
    n_cache = n;
    n_keys = n + C;
    const int tiles = (n_keys + kDcTile - 1) / kDcTile;
    if constexpr (ONE) work.n_splits = decode_splits_of_one(tiles, n_slots);
    // (as 64-bit quotients they took 260 instructions ahead of the first fetch)
    t_end = (int)((uint32_t)tiles * (uint32_t)(work.split + 1) / (uint32_t)work.n_splits);
    t = ONE && work.split >= work.n_splits ? t_end : (int)((uint32_t)tiles * (uint32_t)work.split / (uint32_t)work.n_splits) + w;
  };
  const int n_given = decode_cache(dm, a, b, kv), n_most = min(dm.B_max, dm.T_max);
  share_out(ONE ? n_most : n_given);

  const char* kcache = reinterpret_cast<const char*>(static_cast<const uint16_t*>(a.k_cache) + b * dm.kvs[0] + kv * dm.kvs[1]);
  const char* vcache = reinterpret_cast<const char*>(static_cast<const uint16_t*>(a.v_cache) + b * dm.kvs[0] + kv * dm.kvs[1]);
  const char* kchunk = reinterpret_cast<const char*>(static_cast<const uint16_t*>(a.k_chunk) + b * dm.cks[0] + kv * dm.cks[1]);
  const char* vchunk = reinterpret_cast<const char*>(static_cast<const uint16_t*>(a.v_chunk) + b * dm.cks[0] + kv * dm.cks[1]);
  const int32_t* kidx = sparse ? a.k_idx + (size_t)(b * dm.n_kv + kv) * dm.B_max : nullptr;
  const uint32_t cache_row_bytes = (uint32_t)dm.kvs[2] * 2u, chunk_row_bytes = (uint32_t)dm.cks[2] * 2u;
  const uint64_t k_cache_u = reinterpret_cast<uint64_t>(kcache), v_cache_u = reinterpret_cast<uint64_t>(vcache);
  const uint64_t k_chunk_delta = reinterpret_cast<uint64_t>(kchunk) - k_cache_u;   // modulo 2^64
  const uint64_t v_chunk_delta = reinterpret_cast<uint64_t>(vchunk) - v_cache_u;

  const int cg = lane % CG, r0 = lane / CG;
  uint32_t src[NLD];        // list entries of the tile whose rows are fetched next
  u32x4 RK[NLD], RV[NLD];   // rows on the way
  // (Every slot fetches an entry, also where it is a chunk row and has none: with a choice between an entry and the slot's own number, the
  // fetches of a tile waited for each other two by two.)
  auto resolve = [&](int tt) __attribute__((always_inline)) {
    if (!sparse) return;
#pragma unroll
    for (int i = 0; i < NLD; ++i) src[i] = (uint32_t)kidx[max(min(tt * kDcTile + r0 + RPI * i, n_cache - 1), 0)];
  };
  auto issue = [&](int tt) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < NLD; ++i) {
      // addresses as integers (cache base, plus the distance to the chunk tensor for chunk rows): a per-lane choice
      // between two pointers would be kept as a table in scratch memory
      const int n = min(tt * kDcTile + r0 + RPI * i, n_keys - 1);   // tail slots repeat a real row; they are masked below
      const bool from_cache = n < n_cache;
      // (the clamp: a malformed list cannot leave the cache)
      const uint32_t row = from_cache ? (sparse ? min(src[i], (uint32_t)(dm.T_max - 1)) : (uint32_t)n) : (uint32_t)(n - n_cache);
      const uint64_t off = (uint64_t)(row * (from_cache ? cache_row_bytes : chunk_row_bytes) + (uint32_t)cg * 16u);
      // (named as global memory: through generic pointers the products' LDS operands wait for the rows of the tile after)
      typedef const u32x4 __attribute__((address_space(1))) * global_rows;
      RK[i] = *(global_rows)(k_cache_u + (from_cache ? 0ull : k_chunk_delta) + off);
      RV[i] = *(global_rows)(v_cache_u + (from_cache ? 0ull : v_chunk_delta) + off);
    }
  };
  if (t < t_end) resolve(t);
  if constexpr (ONE) {
    if (n_given != n_most) {   // block-uniform
      share_out(n_given);
      if (t < t_end) resolve(t);
    }
    if (work.split >= work.n_splits) return;   // block-uniform
  }
  if (t < t_end) {
    issue(t);
    if (t + kDcWaves < t_end) resolve(t + kDcWaves);
  }

  // Q operand: row li -> (token li / g, head li % g); padding rows repeat row 0 and are never stored
  const int row = li < n_rows ? li : 0;
  const int tok = row / g, hj = row % g;
  bf16x8 qreg[KS];
  {
    const uint16_t* qrow = static_cast<const uint16_t*>(a.q) + b * dm.qs[0] + (size_t)(kv * g + hj) * dm.qs[1] +
                           (size_t)tok * dm.qs[2] + 8 * hf;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) qreg[ks] = *reinterpret_cast<const bf16x8*>(qrow + ks * 16);
  }

  f32x16 o[DB];
#pragma unroll
  for (int c = 0; c < DB; ++c)
#pragma unroll
    for (int v = 0; v < 16; ++v) o[c][v] = 0.f;
  float m_run = -INFINITY, l_run = 0.f;
  const float sl2 = 1.4426950408889634f / sqrtf((float)D);
  uint16_t* kt = reinterpret_cast<uint16_t*>(smem + (size_t)w * Cfg::kWaveBytes);
  uint16_t* vt = reinterpret_cast<uint16_t*>(smem + (size_t)w * Cfg::kWaveBytes + Cfg::kKBytes);

  for (; t < t_end; t += kDcWaves) {
    // (this wave's own piece of LDS: its accesses stay in order, no barrier)
#pragma unroll
    for (int i = 0; i < NLD; ++i) {
      const int rl = r0 + RPI * i;
      *reinterpret_cast<u32x4*>(kt + rl * LD + cg * 8) = RK[i];
      *reinterpret_cast<u32x4*>(vt + rl * LDV + cg * 8) = RV[i];
    }
    __builtin_amdgcn_wave_barrier();
    if constexpr (LONG) {   // (named as changed, so that they are waited for here, where the tile's entries are waited for next)
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) asm volatile("" : "+v"(qreg[ks]));
    }
    if (t + kDcWaves < t_end) {
      issue(t + kDcWaves);
      if (t + 2 * kDcWaves < t_end) resolve(t + 2 * kDcWaves);
    }
    const int slot0 = t * kDcTile;
    // ---- S^T = K Q^T ----
    f32x16 s;
#pragma unroll
    for (int v = 0; v < 16; ++v) s[v] = 0.f;
    const uint16_t* kp = kt + li * LD + 8 * hf;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      const bf16x8 kop = *reinterpret_cast<const bf16x8*>(kp + ks * 16);
      s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kop, qreg[ks], s, 0, 0, 0);
    }
    // ---- mask: slots past the list; chunk rows in the token's future ----
    // slot n is visible iff it is a cache slot or its chunk position n - n_cache is <= tok, i.e. iff
    // n < n_cache + tok + 1: one lane-private limit, as in the prefill kernel
    const int limit = n_cache + tok + 1 - slot0;   // keys kk < limit of the tile are visible
    if (slot0 + kDcTile > n_cache) {   // wave-uniform: the tile touches the chunk rows or the end
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const int kk = 8 * (v / 4) + 4 * hf + (v % 4);
        if (kk >= limit) s[v] = -INFINITY;
      }
    }
    // ---- online softmax ----
    float mx = -INFINITY;
#pragma unroll
    for (int v = 0; v < 16; ++v) mx = fmaxf(mx, s[v]);
    mx = fmaxf(mx, other_half(mx)) * sl2;
    // the reference point only moves when the tile maximum exceeds it by more than 2^8 (as in the prefill kernel)
    constexpr float kLazy = 8.0f;
    if (__builtin_amdgcn_ballot_w64(mx > m_run + kLazy) != 0) {   // wave-uniform branch
      const float m_new = (mx > m_run + kLazy) ? mx : m_run;
      const float m_fin = (m_new == -INFINITY) ? 0.f : m_new;
      const float alpha = __builtin_amdgcn_exp2f(m_run - m_fin);
      m_run = m_new;
      l_run *= alpha;
#pragma unroll
      for (int c = 0; c < DB; ++c)
#pragma unroll
        for (int v = 0; v < 16; ++v) o[c][v] *= alpha;
    }
    const float m_use = (m_run == -INFINITY) ? 0.f : m_run;
#pragma unroll
    for (int v = 0; v < 16; ++v) s[v] = __builtin_amdgcn_exp2f(fmaf(s[v], sl2, -m_use));
    // ---- O^T += V^T P^T ----
    const tr_ptr vtr = (tr_ptr)(vt + (4 * hf + ((lane & 15) >> 2)) * LDV + 16 * ((lane >> 4) & 1) + 4 * (lane & 3));
    float psum = 0.f;
#pragma unroll
    for (int t2 = 0; t2 < 2; ++t2) {
      bf16x8 pb;
#pragma unroll
      for (int e = 0; e < 8; ++e) pb[e] = (__bf16)s[8 * t2 + e];
#pragma unroll
      for (int e = 0; e < 8; e += 2) {
        const bf16x2 pp = {pb[e], pb[e + 1]};
        psum = __builtin_amdgcn_fdot2_f32_bf16(pp, bf16x2{(__bf16)1.0f, (__bf16)1.0f}, psum, false);
      }
#pragma unroll
      for (int c = 0; c < DB; ++c) {
        const int e0 = (16 * t2) * LDV + c * 32;
        const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16(vtr + e0 / 4);
        const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16(vtr + (e0 + 8 * LDV) / 4);
        const s16x8 both = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
        o[c] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, both), pb, o[c], 0, 0, 0);
      }
    }
    l_run += psum;
    __builtin_amdgcn_wave_barrier();
  }

  // ---- merge the four waves' partials of the real rows through LDS, then write the block's partial ----
  // Every block pays for this whatever its share of the keys, and a call of many tokens has 32 rows: weights once per wave
  // and row, rows by 16 bytes.  (A weight per element and single floats: 2 sequences of 8192, 8 KV heads, kernel 17.8 us
  // at 4 rows and 23.8 at 32.)
  const float l_wave = l_run + other_half(l_run);
  __syncthreads();   // the waves' pieces may be reused
  float* mo = reinterpret_cast<float*>(smem);      // [4 waves][32 rows][LDO]
  float* mm = mo + kDcWaves * 32 * LDO;             // [4][32]
  float* ml = mm + kDcWaves * 32;
  float* mw = ml + kDcWaves * 32;
  if (li < n_rows) {
    if (hf == 0) {
      mm[w * 32 + li] = m_run;
      ml[w * 32 + li] = l_wave;
    }
    float* rec = mo + ((size_t)w * 32 + li) * LDO + 4 * hf;
#pragma unroll
    for (int c = 0; c < DB; ++c)
#pragma unroll
      for (int v4 = 0; v4 < 4; ++v4)   // registers 4*v4 .. 4*v4+3 are four consecutive dims
        *reinterpret_cast<float4*>(rec + 32 * c + 8 * v4) =
            make_float4(o[c][4 * v4], o[c][4 * v4 + 1], o[c][4 * v4 + 2], o[c][4 * v4 + 3]);
  }
  __syncthreads();
  float* my_part = part + ((size_t)kv * n_slots + blockIdx.x) * Cfg::kRec;
  if (tid < kDcWaves * 32 && li < n_rows) {   // thread (wave tid / 32, row tid % 32 == li)
    float m = mm[li];
#pragma unroll
    for (int u = 1; u < kDcWaves; ++u) m = fmaxf(m, mm[u * 32 + li]);
    mw[tid] = mm[tid] == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(mm[tid] - m);
    if (tid < 32) my_part[32 * D + li] = m;
  }
  __syncthreads();
  if (tid < n_rows) {
    float l = 0.f;
#pragma unroll
    for (int u = 0; u < kDcWaves; ++u) l += mw[u * 32 + tid] * ml[u * 32 + tid];
    my_part[32 * D + 32 + tid] = l;
  }
  for (int i = tid; i < n_rows * (D / 4); i += kDcThreads) {
    const int r = i / (D / 4), c4 = i % (D / 4);
    float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
    for (int u = 0; u < kDcWaves; ++u) {
      const float wgt = mw[u * 32 + r];
      const float4 x = *reinterpret_cast<const float4*>(mo + ((size_t)u * 32 + r) * LDO + 4 * c4);
      acc.x += wgt * x.x;
      acc.y += wgt * x.y;
      acc.z += wgt * x.z;
      acc.w += wgt * x.w;
    }
    *reinterpret_cast<float4*>(my_part + r * D + 4 * c4) = acc;
  }
}

// One block per (row, kv, b).  The splits' (m, l) go through LDS once; then thread (dim e, split group sg) adds up the
// O partials of its splits (independent, coalesced loads, unrolled), and the groups are combined through LDS.
// The summation order is fixed by the indices alone, so the result does not depend on scheduling.
// ONE: as in attn_decode_bf16; the first partials are requested while the list's length travels.
template <int D, bool ONE>
__global__ __launch_bounds__(kDcThreads) void attn_decode_merge(Dims dm, AttnArgs a, const float* __restrict__ part,
                                                                int n_slots) {
  constexpr int NG = kDcThreads / D;   // split groups
  __shared__ float wgt[kMaxSplits];
  __shared__ float red[NG][D];
  __shared__ float s_m, s_l;
  const int r = blockIdx.x, kv = blockIdx.y, b = blockIdx.z;
  const int tid = threadIdx.x;
  DecodeShare share{0, 0};
  int n_splits;
  const int n_given = ONE ? decode_cache(dm, a, 0, kv) : 0, n_most = min(dm.B_max, dm.T_max);
  auto splits_of = [&](int n) __attribute__((always_inline)) { return decode_splits_of_one((n + dm.C + kDcTile - 1) / kDcTile, n_slots); };
  if constexpr (ONE) {
    n_splits = splits_of(n_most);
  } else {
    share = decode_share(dm, a, b, kv, n_slots);
    n_splits = share.n_splits;
  }
  constexpr size_t sstride = DecodeCfg<D>::kRec;   // split s is s * sstride further
  const float* base = part + ((size_t)kv * n_slots + share.first) * sstride;
  // a thread's first eight outputs are requested together with (m, l), the next eight before these are used
  const int e = tid % D, sg = tid / D;
  float v[8];
  auto load_v = [&](int s0) __attribute__((always_inline)) {
#pragma unroll
    for (int u = 0; u < 8; ++u) v[u] = base[min(s0 + u * NG, n_splits - 1) * sstride + r * D + e];
  };
  float m_s, l_s;
  auto load_ml = [&]() __attribute__((always_inline)) {
    m_s = -INFINITY;
    l_s = 0.f;
    if (tid < n_splits) {
      m_s = base[tid * sstride + 32 * D + r];
      l_s = base[tid * sstride + 32 * D + 32 + r];
    }
  };
  load_ml();
  load_v(sg);
  if (ONE && n_given != n_most) {   // block-uniform
    n_splits = splits_of(n_given);
    load_ml();
    load_v(sg);
  }
  if (tid < 64) {   // n_splits <= 64: one wave holds all of them
    const float m = wave64_max(m_s);
    const float w = (m_s == -INFINITY) ? 0.f : __builtin_amdgcn_exp2f(m_s - m);
    const float l = wave64_sum(w * l_s);
    wgt[tid] = w;
    if (tid == 0) {
      s_m = m;
      s_l = l;
    }
  }
  __syncthreads();
  float acc = 0.f;
  for (int s0 = sg; s0 < n_splits; s0 += 8 * NG) {
    float x[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) x[u] = v[u];
    if (s0 + 8 * NG < n_splits) load_v(s0 + 8 * NG);
#pragma unroll
    for (int u = 0; u < 8; ++u)
      if (s0 + u * NG < n_splits) acc += wgt[s0 + u * NG] * x[u];
  }
  red[sg][e] = acc;
  __syncthreads();
  if (tid < D) {
    float o = red[0][tid];
#pragma unroll
    for (int g2 = 1; g2 < NG; ++g2) o += red[g2][tid];
    const int tok = r / dm.g, h = kv * dm.g + r % dm.g;
    uint16_t* orow = static_cast<uint16_t*>(a.out) + b * dm.os[0] + h * dm.os[1] + (size_t)tok * dm.os[2];
    orow[tid] = (uint16_t)f32_to_bf16_bits(o / s_l);
    if (tid == 0 && a.lse != nullptr) a.lse[(size_t)(b * dm.n_q + h) * dm.C + tok] = (s_m + log2f(s_l)) * 0.6931471805599453f;
  }
}

// ---------------------------------------------------------------------------------------------
bool attn_decode_applies(const Dims& dm) { return dm.C * dm.g <= 32; }

// Blocks per KV head: in all two for every compute unit, which are resident together.  (One more for every sequence puts the
// last of them into a second round: 3 sequences of 10000 - 20000 tokens, 8 KV heads, dense 43.0 us a call, 35.9 so; 8 of
// mixed length 33.1 / 29.6.  Only where a sequence has fewer than four blocks of a head to itself is that the smaller loss:
// every sequence has one, and the others go by length.)
static int decode_slots(const Dims& dm) {
  const long long n = (512 + dm.n_kv - 1) / dm.n_kv, most = (long long)kMaxSplits * dm.b;
  const long long want = dm.b > 64 ? (n + dm.b - 1) / dm.b * dm.b : (4 * dm.b <= n ? n : n + dm.b);
  return (int)(want < most ? want : most);
}
// One block a compute unit instead where the waves of two would have two tiles each or fewer: every block pays for its
// start and for the merge of its rows (2 sequences of 5286 and 3653 tokens, 8 KV heads, d 128: 1 token 15.5 us a call, 14.7
// so; 8 tokens 18.8 / 16.3.  About as fast at twice the keys, slower from there on).
static int decode_launch_slots(const Dims& dm, bool sparse) {
  const int n = decode_slots(dm), half = (n + 1) / 2;
  const long long tiles = ((long long)attended_cap(dm, sparse) + dm.C + kDcTile - 1) / kDcTile * dm.b;   // of a KV head
  return 4 * dm.b <= half && tiles <= 2 * kDcWaves * (long long)n ? half : n;
}

size_t attn_decode_ws_floats(const Dims& dm) {
  // independent of the chunk length (a prompt's last chunk may be decode-sized when the others are not)
  return (size_t)dm.n_kv * decode_slots(dm) * 32 * (2 + dm.d);
}

template <int D, bool ONE>
static hipError_t launch_decode_d(const Dims& dm, const AttnArgs& a, float* part, hipStream_t st) {
  using Cfg = DecodeCfg<D>;
  const int n_slots = decode_launch_slots(dm, a.k_idx != nullptr);
  // blocks that a short list leaves without work are not launched where the host can tell
  const long long tiles = ((long long)attended_cap(dm, a.k_idx != nullptr) + dm.C + kDcTile - 1) / kDcTile;
  const long long most = dm.b > 64 ? n_slots : dm.b * ((tiles + kDcWaves - 1) / kDcWaves);
  auto launch = [&](auto is_long) -> hipError_t {
    constexpr bool kLong = decltype(is_long)::value;
    static std::atomic<uint64_t> lds_done{0};
    const hipError_t e = ensure_dynamic_lds(reinterpret_cast<const void*>(&attn_decode_bf16<D, ONE, kLong>), Cfg::kLdsBytes, lds_done);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((attn_decode_bf16<D, ONE, kLong>), dim3(n_slots < most ? n_slots : (int)most, dm.n_kv), dim3(kDcThreads),
                       Cfg::kLdsBytes, st, dm, a, part, n_slots);
    return hipSuccess;
  };
  // More than two tiles a wave.  (160 random calls, both launches: LONG takes 0.93 - 1.00 of the time above the line, 0.97 on the mean,
  // and 1.00 - 1.03 at it and below, 1.01 with more than eight rows.)
  const hipError_t e = tiles * dm.b > 2LL * kDcWaves * n_slots ? launch(std::true_type{}) : launch(std::false_type{});
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((attn_decode_merge<D, ONE>), dim3(dm.C * dm.g, dm.n_kv, dm.b), dim3(kDcThreads), 0, st, dm, a, part,
                     n_slots);
  return hipGetLastError();
}

hipError_t launch_attn_decode_bf16(const Dims& dm, const AttnArgs& a, float* part, hipStream_t st) {
  if (dm.b == 1 && a.k_idx != nullptr)
    return dm.d == 64 ? launch_decode_d<64, true>(dm, a, part, st) : launch_decode_d<128, true>(dm, a, part, st);
  return dm.d == 64 ? launch_decode_d<64, false>(dm, a, part, st) : launch_decode_d<128, false>(dm, a, part, st);
}

}  // namespace quoka
