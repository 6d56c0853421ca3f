// Chunk attention in float32 (Alg. 2 attention step; Eq. 2-3) for the float32 storage type: float32 matrix
// instructions (v_mfma_f32_32x32x2_f32: float32 operands, float32 accumulation), online softmax in float32.  Serves the
// sparse path (cache rows through k_idx) and the dense baseline.
//
// What bounds it: the float32 matrix rate (64 clocks for 32x32x2, twice the rate of plain FMAs); a 32-row, 32-key unit
// takes D such instructions and reads only 2 * 32 * D floats, so V, and K of short lists and at d 64, come straight from global
// memory (the cache rows of one KV head stay in L2); no key tile is shared by waves.
//
// Rows: the C * g query rows of a KV head are numbered r = token * g + head-in-group, so the 32 rows of a block span few
// tokens and decode-sized chunks of all heads fill one row block.  Keys: the cache list and the chunk are cut into
// units of 32 keys.  A block of eight waves owns one row block; its waves take the units in turn, each with its own
// running (m, l, O), and are merged through LDS.  Row blocks that leave compute units idle are also split over the grid
// along the key list: such blocks write partial (m, l, O) and attn_f32_merge adds them up.
// Measured (8/2 heads, d 128, 512 tokens over 491 + 512 keys): 423 us for one wave per row with plain FMAs, 27 + 4 us here;
// (2/1 heads, d 64, 128 tokens over 128 + 128 keys): 47 us and 10 us.
//
// Short lists of a few tokens keep one wave per row (attn_f32_short).
//
// Operand plan (a lane is (li = lane % 32, hf = lane / 32)); the contraction index may be permuted freely:
//   S^T[key, row]: A = K row of key li, B = Q row li from LDS; step (i, e) contracts dims 8i + e (hf 0) and 8i + 4 + e.
//     Register v of the result holds key 8*(v/4) + 4*hf + v%4 of the unit for query row li.
//   O^T[dim, row]: step v contracts exactly the two keys that register v holds, so B = P is that register; A = V of the
//     lane's key, M index m of block c standing for dim DB*m + c, so one contiguous load gives all DB blocks.
#include <type_traits>

#include "common.hip.h"
#include "kernels.h"

namespace quoka {

constexpr int kFaWaves = 8;
constexpr int kFaThreads = 64 * kFaWaves;
constexpr int kFaMaxSplits = 64;

template <int D>
struct FaCfg {
  static constexpr int NI = D / 8;        // 16-byte operand loads per lane of a K row
  static constexpr int DB = D / 32;       // dim blocks of the PV product
  static constexpr int QLD = D + 4;       // LDS pitch of the Q rows (floats): 16 bytes of padding
  static constexpr int OLD = D + 4;       // LDS pitch of a wave's partial output rows
  static constexpr int REC = D + 2;       // floats per row of a partial: O[D], m, l
  static constexpr size_t kLdsBytes =
      (size_t)32 * QLD * 4 + (size_t)kFaWaves * 32 * OLD * 4 + (size_t)kFaWaves * 32 * 2 * 4 + (size_t)kFaWaves * 32 * 4;
};

template <int DB>
struct FaVec;
template <>
struct FaVec<2> {
  typedef float type __attribute__((ext_vector_type(2)));
};
template <>
struct FaVec<4> {
  typedef float type __attribute__((ext_vector_type(4)));
};

struct FaRow {
  int tok, head;   // chunk token and head-in-group of a flattened row
};
__device__ __forceinline__ FaRow fa_row(int r, int g) { return {r / g, r % g}; }

// STAGED: K rows go to the wave's own piece of LDS (where its output rows go in the end), whole.  As operands straight from memory a load
// takes 32 bytes of each of 32 rows, eight waves' rows do not fit the first-level cache, and every line is fetched four times (8/2 heads, d
// 128, 512 tokens over 491 + 512 keys: the launches 31.5 -> 27.8 us; dense over 4096 101 -> 89).  Up to four units their waves' lines
// stay, and the way through LDS costs 0.5 us (5 tokens over 45 keys 8.9 / 9.4; eight waves of one unit, 60 tokens over 360 keys 18.2 /
// 16.7), and at d 64, with half the lines, 4 - 7 % throughout: those take the operands as they come.
template <int D, bool STAGED>
__global__ __launch_bounds__(kFaThreads, 2) void attn_f32(Dims dm, AttnArgs a, float* __restrict__ part, int n_splits) {
  using Cfg = FaCfg<D>;
  constexpr int NI = Cfg::NI, DB = Cfg::DB, QLD = Cfg::QLD, OLD = Cfg::OLD, REC = Cfg::REC;
  static_assert(OLD >= D, "a unit's K rows in the place of a wave's output rows");
  typedef typename FaVec<DB>::type vrow;
  typedef float f32x4 __attribute__((ext_vector_type(4)));
  extern __shared__ __align__(16) unsigned char smem[];
  float* qs = reinterpret_cast<float*>(smem);                 // [32][QLD]
  float* os = qs + 32 * QLD;                                    // [kFaWaves][32][OLD]
  float* ml = os + kFaWaves * 32 * OLD;                         // [kFaWaves][32][2]
  uint32_t* offs = reinterpret_cast<uint32_t*>(ml + kFaWaves * 64);   // [kFaWaves][32] row offsets of the wave's unit

  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int li = lane & 31, hf = lane >> 5;
  const int rb = gridDim.x - 1 - blockIdx.x;   // longest causal ranges first
  const int split = blockIdx.y;
  const int kv = blockIdx.z % dm.n_kv, b = blockIdx.z / dm.n_kv;
  const int g = dm.g, n_rows = dm.C * g, row0 = rb * 32;

  const bool sparse = a.k_idx != nullptr;
  int n_cache = sparse ? min(a.n_cache[b * dm.n_kv + kv], dm.B_max) : min(a.n_cache[b * dm.ls], dm.T_max);
  n_cache = max(n_cache, 0);
  const int n_chunk = fa_row(min(row0 + 31, n_rows - 1), g).tok + 1;   // chunk keys any row of the block can see
  const int cache_units = (n_cache + 31) / 32, units = cache_units + (n_chunk + 31) / 32;
  const int u_begin = (int)((long long)units * split / n_splits), u_end = (int)((long long)units * (split + 1) / n_splits);

  // Q rows of the block to LDS (rows past the end repeat the last one and are never stored)
  for (int i = tid; i < 32 * (D / 4); i += kFaThreads) {
    const int r = i / (D / 4), c4 = i % (D / 4);
    const FaRow fr = fa_row(min(row0 + r, n_rows - 1), g);
    const float* src = static_cast<const float*>(a.q) + b * dm.qs[0] + (size_t)(kv * g + fr.head) * dm.qs[1] +
                       (size_t)fr.tok * dm.qs[2] + 4 * c4;
    *reinterpret_cast<f32x4*>(qs + r * QLD + 4 * c4) = *reinterpret_cast<const f32x4*>(src);
  }

  const int32_t* kidx = sparse ? a.k_idx + (size_t)(b * dm.n_kv + kv) * dm.B_max : nullptr;
  const char* kcache = reinterpret_cast<const char*>(static_cast<const float*>(a.k_cache) + b * dm.kvs[0] + kv * dm.kvs[1]);
  const char* vcache = reinterpret_cast<const char*>(static_cast<const float*>(a.v_cache) + b * dm.kvs[0] + kv * dm.kvs[1]);
  const char* kchunk = reinterpret_cast<const char*>(static_cast<const float*>(a.k_chunk) + b * dm.cks[0] + kv * dm.cks[1]);
  const char* vchunk = reinterpret_cast<const char*>(static_cast<const float*>(a.v_chunk) + b * dm.cks[0] + kv * dm.cks[1]);
  const uint32_t cache_rb = (uint32_t)dm.kvs[2] * 4u, chunk_rb = (uint32_t)dm.cks[2] * 4u;

  // The list's entry for slot li of unit u: fetched a unit ahead, before the unit's V rows (fetches arrive in order), and first used, and
  // so waited for, behind the unit's first product.  (Looked up and turned into an offset in one place, the wave waited for it, and for all
  // of its V rows, ahead of that product.)  A chunk unit and a dense call find some number, which is not used: asked for lists only, the
  // launch over 491 + 512 keys takes 29.8 us instead of 27.5, at d 64 19.3 and 18.8, and a dense one over 4096 the same 88.8.
  const int32_t* list = sparse ? kidx : a.n_cache;
  const int list_last = sparse ? max(n_cache - 1, 0) : 0;
  auto look_up = [&](int u) __attribute__((always_inline)) { return (uint32_t)list[min(u * 32 + li, list_last)]; };
  // byte offset of the row that slot li of unit u names (slots past the list repeat its last row; they are masked)
  auto row_offset = [&](int u, uint32_t entry) __attribute__((always_inline)) -> uint32_t {
    if (u < cache_units)   // (the clamp: a malformed list cannot leave the cache)
      return (sparse ? min(entry, (uint32_t)(dm.T_max - 1)) : (uint32_t)min(u * 32 + li, n_cache - 1)) * cache_rb;
    return (uint32_t)min((u - cache_units) * 32 + li, n_chunk - 1) * chunk_rb;
  };
  // Slot c of row r holds chunk c ^ (r & 15), so that 16 lanes read a chunk of 16 rows without conflicts.
  constexpr int CG = D / 4, RPL = 64 / CG;   // 16-byte chunks of a row, rows of a load
  const float* kt = os + (size_t)w * 32 * OLD;
  const uint32_t kt_lds = (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) void*)kt;
  f32x4 kreg[STAGED ? 1 : NI];
  auto request_k = [&](int u, uint32_t off) __attribute__((always_inline)) {
    const char* base = u < cache_units ? kcache : kchunk;
    if constexpr (!STAGED) {
#pragma unroll
      for (int i = 0; i < NI; ++i) kreg[i] = *reinterpret_cast<const f32x4*>(base + 16 * hf + off + 32 * i);
      return;
    }
#pragma unroll
    for (int i = 0; i < 32 / RPL; ++i) {
      const int r = i * RPL + lane / CG;
      uint32_t row = (uint32_t)__builtin_amdgcn_readlane((int)off, i * RPL);   // (lane r has the offset of row r)
#pragma unroll
      for (int j = 1; j < RPL; ++j) row = lane / CG == j ? (uint32_t)__builtin_amdgcn_readlane((int)off, i * RPL + j) : row;
      dma16(base, row + (uint32_t)(lane % CG ^ (r & 15)) * 16u, kt_lds + (uint32_t)i * 1024u);
    }
  };

  f32x16 o[DB];
#pragma unroll
  for (int c = 0; c < DB; ++c)
#pragma unroll
    for (int v = 0; v < 16; ++v) o[c][v] = 0.f;
  float m_run = -INFINITY, l_run = 0.f;   // of row li; l_run is this half wave's share
  const float scale2 = 1.4426950408889634f / sqrtf((float)D);   // softmax scale and the change to base 2
  const int tok = fa_row(min(row0 + li, n_rows - 1), g).tok;

  int u = u_begin + w;
  uint32_t off = 0;
  if (u < u_end) {
    off = row_offset(u, sparse ? look_up(u) : 0u);
    request_k(u, off);
  }
  __syncthreads();   // Q rows are in LDS
  uint32_t* my_offs = offs + w * 32;
  const float* qrow = qs + li * QLD + 4 * hf;
  for (; u < u_end; u += kFaWaves) {
    if constexpr (STAGED) wait_vmcnt<0>();   // K of this unit is there
    const bool is_chunk = u >= cache_units;
    // the rows of the unit's 16 V loads: slot 8*(v/4) + 4*hf + v%4 belongs to another lane (only this wave uses its row
    // of `offs`, and a wave's LDS accesses stay in order)
    if (hf == 0) my_offs[li] = off;
    __builtin_amdgcn_wave_barrier();
    uint32_t voff[16];
#pragma unroll
    for (int q4 = 0; q4 < 4; ++q4) {
      const u32x4 t = *reinterpret_cast<const u32x4*>(my_offs + 8 * q4 + 4 * hf);
#pragma unroll
      for (int e = 0; e < 4; ++e) voff[4 * q4 + e] = t[e];
    }
    const uint32_t entry_next = look_up(u + kFaWaves);
    vrow vreg[16];   // in flight during the first product
    const char* vbase = (is_chunk ? vchunk : vcache) + (DB * 4) * li;
#pragma unroll
    for (int v = 0; v < 16; ++v) vreg[v] = *reinterpret_cast<const vrow*>(vbase + voff[v]);
    __builtin_amdgcn_sched_barrier(0);   // (or they leave behind the product)

    f32x16 s;
#pragma unroll
    for (int v = 0; v < 16; ++v) s[v] = 0.f;
    // (Q, read a step ahead of its products.  With K in LDS too that is the slower: 512 tokens over 491 + 512 keys 27.8 / 29.4 us.)
    f32x4 qv[2];
    auto read_q = [&](int i) __attribute__((always_inline)) { qv[i % 2] = *reinterpret_cast<const f32x4*>(qrow + 8 * i); };
    if constexpr (!STAGED) read_q(0);
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      f32x4 kop;
      if constexpr (STAGED) {
        read_q(i);
        kop = *reinterpret_cast<const f32x4*>(kt + li * D + ((2 * i + hf) ^ (li & 15)) * 4);
      } else {
        if (i + 1 < NI) read_q(i + 1);
        kop = kreg[i];
        __builtin_amdgcn_sched_barrier(0);
      }
#pragma unroll
      for (int e = 0; e < 4; ++e) s = __builtin_amdgcn_mfma_f32_32x32x2f32(kop[e], qv[i % 2][e], s, 0, 0, 0);
      if constexpr (!STAGED) __builtin_amdgcn_sched_barrier(0);
    }
    if (u + kFaWaves < u_end) {   // travels during the softmax and the second product
      off = row_offset(u + kFaWaves, entry_next);
      if constexpr (STAGED) asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // (K of this unit has been read)
      request_k(u + kFaWaves, off);
    }

    const int limit = is_chunk ? tok + 1 - (u - cache_units) * 32 : n_cache - u * 32;   // slots kk < limit are visible
    float mx = -INFINITY;
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      const int kk = 8 * (v / 4) + 4 * hf + (v % 4);
      if (kk >= limit) s[v] = -INFINITY;
      mx = fmaxf(mx, s[v]);
    }
    mx = fmaxf(mx, other_half(mx)) * scale2;
    // the reference point moves only when the unit's maximum exceeds it by more than 2^8
    const bool moves = m_run == -INFINITY ? mx > -INFINITY : mx > m_run + 8.0f;
    if (__builtin_amdgcn_ballot_w64(moves) != 0) {   // wave-uniform branch
      const float m_new = moves ? mx : m_run;
      const float alpha = __builtin_amdgcn_exp2f(m_run - (m_new == -INFINITY ? 0.f : m_new));
      m_run = m_new;
      l_run *= alpha;
#pragma unroll
      for (int c = 0; c < DB; ++c)
#pragma unroll
        for (int v = 0; v < 16; ++v) o[c][v] *= alpha;
    }
    const float neg_m = m_run == -INFINITY ? 0.f : -m_run;
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      s[v] = __builtin_amdgcn_exp2f(fmaf(s[v], scale2, neg_m));
      l_run += s[v];
    }
#pragma unroll
    for (int v = 0; v < 16; ++v)
#pragma unroll
      for (int c = 0; c < DB; ++c) o[c] = __builtin_amdgcn_mfma_f32_32x32x2f32(vreg[v][c], s[v], o[c], 0, 0, 0);
  }

  // ---- merge the waves: every wave leaves (m, l) and its output rows, all threads add them up ----
  const float l_wave = l_run + other_half(l_run);
  if (hf == 0) {
    ml[(w * 32 + li) * 2] = m_run;
    ml[(w * 32 + li) * 2 + 1] = l_wave;
  }
  float* my_os = os + (size_t)(w * 32 + li) * OLD;
#pragma unroll
  for (int v = 0; v < 16; ++v) {
    const int m = 8 * (v / 4) + 4 * hf + (v % 4);
    vrow t;
#pragma unroll
    for (int c = 0; c < DB; ++c) t[c] = o[c][v];
    *reinterpret_cast<vrow*>(my_os + DB * m) = t;   // dims DB*m .. +DB
  }
  __syncthreads();
  float* my_part = part + ((size_t)(blockIdx.z * gridDim.x + rb) * n_splits + split) * 32 * REC;
  for (int i = tid; i < 32 * (D / 4); i += kFaThreads) {
    const int r = i / (D / 4), c4 = i % (D / 4);
    float m = -INFINITY;
#pragma unroll
    for (int j = 0; j < kFaWaves; ++j) m = fmaxf(m, ml[(j * 32 + r) * 2]);
    const float m_fin = m == -INFINITY ? 0.f : m;
    float l = 0.f;
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int j = 0; j < kFaWaves; ++j) {
      const float wgt = __builtin_amdgcn_exp2f(ml[(j * 32 + r) * 2] - m_fin);   // 0 for a wave that saw no key of this row
      l += wgt * ml[(j * 32 + r) * 2 + 1];
      const f32x4 x = *reinterpret_cast<const f32x4*>(os + (size_t)(j * 32 + r) * OLD + 4 * c4);
#pragma unroll
      for (int e = 0; e < 4; ++e) acc[e] += wgt * x[e];
    }
    if (n_splits > 1) {   // block-uniform
      *reinterpret_cast<f32x4*>(my_part + r * D + 4 * c4) = acc;
      if (c4 == 0) {
        my_part[32 * D + r] = m;
        my_part[32 * D + 32 + r] = l;
      }
    } else if (row0 + r < n_rows) {
      const FaRow fr = fa_row(row0 + r, g);
      const int h = kv * g + fr.head;
      float* orow = static_cast<float*>(a.out) + b * dm.os[0] + h * dm.os[1] + (size_t)fr.tok * dm.os[2];
#pragma unroll
      for (int e = 0; e < 4; ++e) acc[e] /= l;
      *reinterpret_cast<f32x4*>(orow + 4 * c4) = acc;
      if (c4 == 0 && a.lse != nullptr)
        a.lse[(size_t)(b * dm.n_q + h) * dm.C + fr.tok] = (m + log2f(l)) * 0.6931471805599453f;
    }
  }
}

// Sum of the splits' partials: D / 4 threads per row, four dims each, the splits of a row shared by G such groups (neighbouring
// splits each), whose sums meet in LDS.  All of a thread's records, at most eight, are requested before the first is used.  The maximum
// over all splits comes first, so that every partial is weighted once and added by one fused multiply-add, in a fixed order; the
// groups' sums are added in pairs.  (Sums rescaled to a running maximum, products rounded before they are added: 0.1 - 0.5 % further
// from float64.)  What bounds it is the chain of fetches: with one group that walked the splits one by one two KV heads of one,
// d 128, 2 tokens over 7362 keys took 33 us in all, and take 19; 4 heads, d 64, 48 tokens 27 and 14.
constexpr int kFmThreads = 256, kFmRun = 4;
template <int D, int G>
__global__ __launch_bounds__(kFmThreads) void attn_f32_merge(Dims dm, AttnArgs a, const float* __restrict__ part, int n_rb,
                                                            int n_splits) {
  constexpr int REC = FaCfg<D>::REC, TPR = D / 4, ROWS = kFmThreads / (TPR * G);
  constexpr int RUNS = G > 1 ? kFaMaxSplits / (G * kFmRun) : 1;   // (G == 1: at most kFmRun splits)
  static_assert(G == 1 || RUNS * G * kFmRun == kFaMaxSplits, "");
  typedef float f32x4 __attribute__((ext_vector_type(4)));
  __shared__ __align__(16) f32x4 sum[G > 1 ? kFmThreads : 1];
  __shared__ float ms_all[G > 1 ? kFmThreads : 1], ls_all[G > 1 ? kFmThreads : 1];
  const int c4 = threadIdx.x % TPR, grp = threadIdx.x / TPR % G;
  const int row = blockIdx.x * ROWS + threadIdx.x / (TPR * G);
  const int kv = blockIdx.y % dm.n_kv, b = blockIdx.y / dm.n_kv;
  const bool row_on = row < dm.C * dm.g;
  const int r = row % 32, rb = row_on ? row / 32 : 0;
  const float* rec = part + ((size_t)blockIdx.y * n_rb + rb) * n_splits * 32 * REC;
  const int s0 = n_splits * grp / G, s1 = n_splits * (grp + 1) / G;
  float ms[RUNS * kFmRun], ls[RUNS * kFmRun];
  f32x4 x[RUNS * kFmRun];
#pragma unroll
  for (int u = 0; u < RUNS; ++u) {
    if (u > 0 && n_splits <= u * kFmRun * G) break;   // block-uniform
#pragma unroll
    for (int i = u * kFmRun; i < (u + 1) * kFmRun; ++i) {   // (the group's last record again where it has fewer, or none)
      const float* p = rec + (size_t)max(min(s0 + i, s1 - 1), 0) * 32 * REC;
      ms[i] = p[32 * D + r];
      ls[i] = p[32 * D + 32 + r];
      x[i] = *reinterpret_cast<const f32x4*>(p + r * D + 4 * c4);
    }
  }
  __builtin_amdgcn_sched_barrier(0);   // all of them in flight
  float m = -INFINITY;
#pragma unroll
  for (int i = 0; i < RUNS * kFmRun; ++i) m = s0 + i < s1 ? fmaxf(m, ms[i]) : m;
  if constexpr (G > 1) {
    ms_all[threadIdx.x] = m;
    __syncthreads();
#pragma unroll
    for (int i = 0; i < G; ++i) m = fmaxf(m, ms_all[threadIdx.x + TPR * (i - grp)]);
  }
  float l = 0.f;
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int i = 0; i < RUNS * kFmRun; ++i) {
    if (s0 + i < s1) {
      const float wgt = __builtin_amdgcn_exp2f(ms[i] - m);   // (every row sees at least its own key: m is finite)
      l += wgt * ls[i];
#pragma unroll
      for (int e = 0; e < 4; ++e) acc[e] += wgt * x[i][e];
    }
  }
  if constexpr (G > 1) {
    sum[threadIdx.x] = acc;
    ls_all[threadIdx.x] = l;
    __syncthreads();
    if (grp > 0) return;
    float lg[G];
    f32x4 ag[G];
#pragma unroll
    for (int i = 0; i < G; ++i) {
      lg[i] = ls_all[threadIdx.x + TPR * i];
      ag[i] = sum[threadIdx.x + TPR * i];
    }
#pragma unroll
    for (int o = 1; o < G; o *= 2)   // in pairs
#pragma unroll
      for (int i = 0; i < G; i += 2 * o) {
        lg[i] += lg[i + o];
        ag[i] += ag[i + o];
      }
    l = lg[0];
    acc = ag[0];
  }
  if (!row_on) return;
  const FaRow fr = fa_row(row, dm.g);
  const int h = kv * dm.g + fr.head;
  float* orow = static_cast<float*>(a.out) + b * dm.os[0] + h * dm.os[1] + (size_t)fr.tok * dm.os[2];
#pragma unroll
  for (int e = 0; e < 4; ++e) acc[e] /= l;
  *reinterpret_cast<f32x4*>(orow + 4 * c4) = acc;
  if (c4 == 0 && a.lse != nullptr)
    a.lse[(size_t)(b * dm.n_q + h) * dm.C + fr.tok] = (m + log2f(l)) * 0.6931471805599453f;
}

// ---------------------------------------------------------------------------------------------
// Short lists of a few tokens: one wave per query row, lanes take 64 keys at a time for the logits and own head_dim / 64
// output dims each for the values; no unit of 32 rows and 32 keys is formed, which takes a wave of attn_f32 5 us at d 128
// whatever there is in it.  Bound by a chain of three fetches and one step a key.  Measured (attn_f32 -> this kernel): 32/8
// heads, d 128, 1 token over 8 keys 8.8 -> 4.8 us, 8 tokens over 16 keys 9.4 -> 7.5; d 64, 1 token over 16 keys 6.3 -> 5.3.
constexpr int kFsThreads = 256;

template <int D>
__global__ __launch_bounds__(kFsThreads) void attn_f32_short(Dims dm, AttnArgs a) {
  constexpr int EPL = D / 64;
  __shared__ float qs[kFsThreads / 64][D];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int i = blockIdx.x * (kFsThreads / 64) + w;   // chunk position of this wave's row
  const int h = blockIdx.y, b = blockIdx.z;
  const bool row_on = i < dm.C;
  if (row_on) {
    const float* qsrc = static_cast<const float*>(a.q) + b * dm.qs[0] + h * dm.qs[1] + (size_t)i * dm.qs[2];
#pragma unroll
    for (int e = 0; e < EPL; ++e) qs[w][lane + 64 * e] = qsrc[lane + 64 * e];
  }
  __syncthreads();
  if (!row_on) return;   // wave-uniform; no barrier follows
  const int kv = h / dm.g;
  const bool sparse = a.k_idx != nullptr;
  int n_cache = sparse ? min(a.n_cache[b * dm.n_kv + kv], dm.B_max) : min(a.n_cache[b * dm.ls], dm.T_max);
  n_cache = max(n_cache, 0);
  const int32_t* kidx = sparse ? a.k_idx + (size_t)(b * dm.n_kv + kv) * dm.B_max : nullptr;
  const float* kcache = static_cast<const float*>(a.k_cache) + b * dm.kvs[0] + kv * dm.kvs[1];
  const float* vcache = static_cast<const float*>(a.v_cache) + b * dm.kvs[0] + kv * dm.kvs[1];
  const float* kchunk = static_cast<const float*>(a.k_chunk) + b * dm.cks[0] + kv * dm.cks[1];
  const float* vchunk = static_cast<const float*>(a.v_chunk) + b * dm.cks[0] + kv * dm.cks[1];
  const float scale = 1.0f / sqrtf((float)D);
  const int total = n_cache + i + 1;
  float m_run = -INFINITY, l_run = 0.f;
  float acc[EPL];
#pragma unroll
  for (int e = 0; e < EPL; ++e) acc[e] = 0.f;

  for (int j0 = 0; j0 < total; j0 += 64) {
    const int j = j0 + lane;
    const bool valid = j < total;
    const int jj = valid ? j : total - 1;
    int is_chunk, row;
    if (jj < n_cache) {
      is_chunk = 0;
      row = sparse ? (int)min((uint32_t)kidx[jj], (uint32_t)(dm.T_max - 1)) : jj;   // a malformed list cannot leave the cache
    } else {
      is_chunk = 1;
      row = jj - n_cache;
    }
    const float* kp = is_chunk ? kchunk + (size_t)row * dm.cks[2] : kcache + (size_t)row * dm.kvs[2];
    float dot = 0.f;
#pragma unroll 8
    for (int d0 = 0; d0 < D; d0 += 4) {
      const float4 kx = *reinterpret_cast<const float4*>(kp + d0);
      dot += qs[w][d0] * kx.x;
      dot += qs[w][d0 + 1] * kx.y;
      dot += qs[w][d0 + 2] * kx.z;
      dot += qs[w][d0 + 3] * kx.w;
    }
    const float s = valid ? dot * scale : -INFINITY;
    const float m_new = fmaxf(m_run, wave64_max(s));   // finite: key j0 is always visible
    const float alpha = expf(m_run - m_new);
    const float p = valid ? expf(s - m_new) : 0.f;
    l_run = l_run * alpha + wave64_sum(p);
    m_run = m_new;
#pragma unroll
    for (int e = 0; e < EPL; ++e) acc[e] *= alpha;
    const int cnt = min(64, total - j0);
    for (int t = 0; t < cnt; ++t) {
      // t is wave-uniform: lane reads through the scalar path instead of LDS shuffles
      const float pt = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(p), t));
      const int ct = __builtin_amdgcn_readlane(is_chunk, t);
      const int rt = __builtin_amdgcn_readlane(row, t);
      const float* vp = ct ? vchunk + (size_t)rt * dm.cks[2] : vcache + (size_t)rt * dm.kvs[2];
#pragma unroll
      for (int e = 0; e < EPL; ++e) acc[e] += pt * vp[lane + 64 * e];
    }
  }
  float* orow = static_cast<float*>(a.out) + b * dm.os[0] + h * dm.os[1] + (size_t)i * dm.os[2];
#pragma unroll
  for (int e = 0; e < EPL; ++e) orow[lane + 64 * e] = acc[e] / l_run;
  if (a.lse != nullptr && lane == 0) a.lse[(size_t)(b * dm.n_q + h) * dm.C + i] = m_run + logf(l_run);
}

// Both sides equal at 24 (C = 1) to 16 (C = 8) cached keys at d 64, 46 to 26 at d 128 and about 10 at C = 16 (32/8 heads, no
// cached key: 9.4 -> 6.3); longer chunks have the rows for attn_f32.
static bool attn_f32_is_short(const Dims& dm, bool sparse) {
  return dm.C <= 16 && attended_cap(dm, sparse) + 2 * dm.C <= (dm.d == 64 ? 26 : 42);
}

// ---------------------------------------------------------------------------------------------
// Splits of the key list: as many as give every compute unit a block, but at least one unit of 32 keys for every wave
// of a block (a split costs 16 KiB of partials and a share of the merge launch).
static long long f32_blocks(const Dims& dm) { return (long long)dm.b * dm.n_kv * ((dm.C * dm.g + 31) / 32); }
static long long f32_units(const Dims& dm, bool sparse) {   // of the longest key list
  return ((long long)attended_cap(dm, sparse) + 31) / 32 + (dm.C + 31) / 32;
}
static int f32_most_splits(const Dims& dm, bool sparse) {
  const long long n = (f32_units(dm, sparse) + kFaWaves - 1) / kFaWaves;
  return (int)(n > kFaMaxSplits ? kFaMaxSplits : n);
}
static int f32_splits(const Dims& dm, bool sparse) {
  const long long blocks = f32_blocks(dm), n = (256 + blocks - 1) / blocks;
  const int most = f32_most_splits(dm, sparse);
  return n < most ? (int)n : most;
}

// Fewer than 256 row blocks are split into at most 2 * 256 blocks; the other bound grows with the chunk length.  So the
// partials of a shorter chunk of the same shape (a prompt's last one) fit as well.
size_t attn_f32_ws_floats(const Dims& dm) {
  const long long most = f32_blocks(dm) * f32_most_splits(dm, false);
  return (size_t)(most < 2 * 256 ? most : 2 * 256) * 32 * (dm.d + 2);
}

template <int D>
static hipError_t launch_f32_d(const Dims& dm, const AttnArgs& a, float* part, hipStream_t st) {
  if (attn_f32_is_short(dm, a.k_idx != nullptr)) {
    const dim3 grid((dm.C + kFsThreads / 64 - 1) / (kFsThreads / 64), dm.n_q, dm.b);
    hipLaunchKernelGGL((attn_f32_short<D>), grid, dim3(kFsThreads), 0, st, dm, a);
    return hipGetLastError();
  }
  const int n_splits = f32_splits(dm, a.k_idx != nullptr), n_rb = (dm.C * dm.g + 31) / 32;
  auto launch = [&](auto staged) -> hipError_t {
    constexpr bool kStaged = decltype(staged)::value;
    static std::atomic<uint64_t> lds_done{0};
    const hipError_t e = ensure_dynamic_lds(reinterpret_cast<const void*>(&attn_f32<D, kStaged>), FaCfg<D>::kLdsBytes, lds_done);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((attn_f32<D, kStaged>), dim3(n_rb, n_splits, dm.b * dm.n_kv), dim3(kFaThreads), FaCfg<D>::kLdsBytes, st, dm,
                       a, part, n_splits);
    return hipSuccess;
  };
  hipError_t e;
  if constexpr (D == 128) {
    // at most four waves of the block have a unit (a list of so few is never split)
    e = f32_units(dm, a.k_idx != nullptr) <= 4 ? launch(std::false_type{}) : launch(std::true_type{});
  } else {
    e = launch(std::false_type{});
  }
  if (e != hipSuccess) return e;
  if (n_splits > 1) {
    const int rows = dm.C * dm.g;
    auto merge = [&](auto kernel, int rows_per_block) {
      hipLaunchKernelGGL(kernel, dim3((rows + rows_per_block - 1) / rows_per_block, dm.b * dm.n_kv), dim3(kFmThreads), 0, st, dm, a,
                         part, n_rb, n_splits);
    };
    if (n_splits <= kFmRun) {
      merge(attn_f32_merge<D, 1>, kFmThreads / (D / 4));
    } else {
      merge(attn_f32_merge<D, 8>, kFmThreads / (D / 4 * 8));
    }
  }
  return hipGetLastError();
}

hipError_t launch_attn_f32(const Dims& dm, const AttnArgs& a, float* part, hipStream_t st) {
  return dm.d == 64 ? launch_f32_d<64>(dm, a, part, st) : launch_f32_d<128>(dm, a, part, st);
}

}  // namespace quoka
