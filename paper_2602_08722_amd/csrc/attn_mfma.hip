// Chunk attention on bf16 MFMA (Alg. 2 attention step; Eq. 2-3): flash-style online softmax over
// [gathered cache rows | chunk rows], causal inside the chunk.  One kernel serves the sparse path
// (rows gathered through k_idx while the tile is staged into LDS -- the reduced cache of Eq. 3 is
// never materialised) and the dense baseline of Eq. 2 (rows 0..kv_len).
//
// Work split: a wave owns a row block: 32 query rows of one q-head.  Row blocks of a KV head are numbered
// (token tile, head-in-group).  In a launch of one round a block takes half of its row blocks from the front of that
// list and half from the back, so every block (and every SIMD, which hosts one wave of each kind) gets the same mix of
// short and long causal ranges; in a launch of several rounds a block takes neighbouring row blocks and the blocks
// with the longest ranges come first.  A block is two sets of four waves that share every staged K/V tile.
//
// MFMA operand plan (v_mfma_f32_32x32x16_bf16; a lane is (li = lane % 32, hf = lane / 32)):
//   S^T[key, row] = K[key, :] . Q[row, :]      A = K tile rows from LDS, B = Q held in registers.
//     Result layout: lane li = query row, 16 registers = keys 8*(v/4) + 4*hf + v%4 of a 32-key block.
//     Row max / row sum are therefore in-lane plus one exchange between the two half waves.
//   O^T[dim, row] += V[key, dim] . P[row, key]  B = P: exactly the registers S^T left in the lane
//     (the contraction index may be permuted freely, so no transpose or shuffle is needed),
//     A = V^T, fetched from the row-major LDS tile with the transposing LDS read (ds_read_b64_tr_b16):
//     in every group of 16 lanes, lane s supplies the address of 4 consecutive dims of one key, and
//     lane L receives dim (L % 4) of the four lanes L/4, L/4 + 4, L/4 + 8, L/4 + 12.  With lane s
//     pointing at key row0 + s/4, dims dim0 + 4*(s%4), lane L ends up with dim dim0 + L of keys
//     row0 .. row0+3: a quarter of an MFMA A operand, with no register shuffling.
//     Accumulator block c, register v of lane li holds O[row li, dim 32*c + 8*(v/4) + 4*hf + v%4].
//
// Schedule: a wave works through its keys in units of 32 and keeps the matrix core and the vector unit busy at once: while the
// products of unit u+1 (S = K Q^T) are formed, the scores of unit u become probabilities; while those of unit u (O += P V) are
// formed, the maximum of unit u+1 is taken.  Operands are read from LDS half a unit before their product, and the next tiles are
// stored and requested between products.  The order is written out, instruction group by instruction group, and held there.
// One barrier per tile of 64 keys, K running one tile ahead of V.
// What bounds it: the loop alone (operands from LDS, nothing staged) keeps the matrix core busy for 73 % of its clocks, at
// 1.73 of 2.4 GHz, the clock that the power limit leaves (1.27 PFLOP/s; without the operand reads 1.44, without the conversion and sum
// of the probabilities 1.44).  Against two wave sets half a step apart, one forming S while the other ran softmax and P V behind
// it (two barriers a tile, staging through registers), attention by itself, us: 32/8 heads, d 128, 4096 tokens over 8192 keys 622 -> 551
// (1.25 PFLOP/s), 2048 over 3932 172 -> 147, 1024 over 983 38.1 -> 31.7, 1024 over 8192 161 -> 135; d 64, 1500 over 2400 70 -> 59.
#include "common.hip.h"
#include "kernels.h"

#include <type_traits>

namespace quoka {

typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef short s16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef s16x4 __attribute__((address_space(3))) * tr_ptr;   // LDS address of one lane's 8 bytes of a transposing read

constexpr int kComputeUnits = 256;   // MI355X
constexpr int kSetThreads = 256;   // four waves
constexpr int kSub = 64;           // keys a wave set consumes per step
constexpr int kMaxKeySplits = 32;          // blocks that share a key list,
constexpr long long kMaxRecords = 2048;   // and their partials of 32 rows (16.6 KiB each at d = 128)
// What attn_bf16 divides without a division: row blocks of a KV head by the group, blocks by the shares of a list (of which there are no
// more than partials); and its tiles times shares stay within 32 bits.
static_assert(quotients_hold(kMaxGroup, kMaxGroup * ((kMaxChunk + 31) / 32) - 1), "row blocks by the group");
static_assert(quotients_hold(kMaxKeySplits, kMaxRecords - 1), "blocks by the shares");
static_assert(((long long)kMaxKv / kSub + kMaxChunk / kSub + 2) * kMaxKeySplits < 1ll << 32, "tiles times shares");

// SPLIT = false: the sets own different row blocks (8 per block) and both consume every 64-key tile.
// SPLIT = true:  both sets own the same 4 row blocks; a staged tile has 128 keys, set s consumes keys 64*s..64*s+63,
//                and the two partial results are merged through LDS at the end.  Used when 8 row blocks per block
//                would leave compute units without a block.
// Index of the sequence whose length has descending rank `rank` among lens[0], lens[stride], ... (nb <= 64 of them; ties
// keep batch order).  Every wave works it out for itself: one load, nb lane reads, a ballot.
__device__ __forceinline__ int seq_of_rank(const int32_t* __restrict__ lens, int stride, int nb, int rank) {
  const int lane = threadIdx.x & 63;
  const int mine = lane < nb ? lens[lane * stride] : -1;
  int r = 0;
  for (int j = 0; j < nb; ++j) {
    const int other = __builtin_amdgcn_readlane(mine, j);
    r += (other > mine) || (other == mine && j < lane);
  }
  const unsigned long long hit = __builtin_amdgcn_ballot_w64(lane < nb && r == rank);
  return hit ? (int)__builtin_ctzll(hit) : rank;
}

// Two floats as bf16, rounded to nearest even by one instruction.  (In integer arithmetic the rows' way out takes 300 more: 32/8 heads, d
// 128, 300 tokens over 1080 keys 23.9 -> 23.6 us, 3000 over 2400 200.5 -> 199.4.)
__device__ __forceinline__ uint32_t bf16_pair(float lo, float hi) {
  const bf16x2 p = {(__bf16)lo, (__bf16)hi};
  return __builtin_bit_cast(uint32_t, p);
}

template <int D>
__device__ __forceinline__ int k_swizzle(int row) { return D == 128 ? row & 3 : (row >> 1) & 3; }
template <int D>
__device__ __forceinline__ int v_swizzle(int row) { return D == 128 ? 4 * (row & 3) : 4 * ((row >> 1) & 1); }

template <int D>
__device__ __forceinline__ int q_swizzle(int row) { return D == 128 ? row & 15 : (row >> 1) & 7; }

template <int D, bool SPLIT>
struct AttnCfg {
  static constexpr int KT = SPLIT ? 2 * kSub : kSub;  // keys per staged tile
  static constexpr int KS = D / 16;                   // k-steps of the QK^T product
  static constexpr int CG = D / 8;                    // 16-byte chunks per row
  static constexpr int RPI = kSetThreads / CG;        // rows per set-wide load
  static constexpr int NLD = KT / RPI;                // loads per thread per tile (set 0 loads K, set 1 loads V)
  static constexpr int DB = D / 32;                   // dim blocks of the PV product
  static constexpr int HW = SPLIT ? 2 : 4;            // front (= back) row blocks per block
  // LDS: a wave-wide load fills a group of RPW rows, 1 KiB.  The 16-byte chunks of a row are permuted by the fetch (k_swizzle,
  // v_swizzle), and K's groups lie 64 bytes apart modulo 256: the 16 rows that lanes read a chunk of at a time (K), and the four rows x
  // 64 bytes of a transposing read by half a wave (V), are 256 bytes on distinct banks.
  // Tiles go straight from memory to LDS, except with blocks of eight row blocks at d 64, whose steps are the shortest (1 us): through
  // registers a load has two steps' time, not one (d 64, 333 tokens over 5000 keys 37.1 -> 36.0 us, 1500 over 2400 61.1 -> 59.9).
  // Elsewhere the stores to LDS were what staging cost (by leaving them out, blocks of eight 7 %, of four 17 - 22 %), and direct loads take
  // them off the waves: 32/8 heads, d 128, 1024 tokens over 8192 keys 140.7 -> 133.2 us, 1024 over 983 33.6 -> 31.7, 4096 over 8192
  // 576 -> 560.  (Three stages, so that every load has two steps: 1 - 3 % slower throughout.)
  static constexpr bool DMA = D == 128 || SPLIT;
  static constexpr int RPW = 64 / CG, ROW = D * 2;
  static constexpr int KG = 1024 + 64, VG = 1024;   // pitches of a group
  static constexpr int kKTileBytes = KT / RPW * KG;
  static constexpr int kStageBytes = kKTileBytes + KT / RPW * VG;   // one K tile and one V tile
  static constexpr size_t kOutBytes = (size_t)8 * 32 * (D + 8) * 2;   // what the rows go out through
  static constexpr size_t kQBytes = SPLIT ? 0 : (size_t)8 * 32 * ROW;   // (SPLIT: in the place of a V tile)
  static constexpr size_t kInBytes = (size_t)2 * kStageBytes + kQBytes;
  static constexpr size_t kLdsBytes = kInBytes > kOutBytes ? kInBytes : kOutBytes;
  static_assert(!SPLIT || KT / RPW * VG == 4 * 32 * ROW, "the rows of four row blocks in the place of a V tile");
  static constexpr int kRecFloats = 32 * (D + 2);     // partial of a row block: O as the registers lie, m, l
};

// XS (QUOKA_ATTN_SCALE_F32): the softmax scale is applied to the float32 products, one fused multiply-add per score
// together with the subtraction of the reference point.  Otherwise the factor log2(e)/sqrt(d) is folded into the bf16 Q
// operand once and the accumulator of K Q^T starts from minus the reference point, so that the matrix core hands back
// what the exponential takes and no vector instruction is spent on either -- 3-13 % faster, at the price of rounding Q a
// second time: an error of the logits of relative size 2^-9, which shows in the output once the logits are several
// times those of unit-variance inputs (0.03 absolute at four times, 0.06 at eight).
// KSPLIT: the key list is shared by a.n_splits blocks, each of which writes a partial result.  (A template parameter: as
// a run-time switch it cost the unsplit launches 1.5-2 %.)
// WHOLE (not KSPLIT): rows go out whole, 16 bytes a lane, through the wave's own piece of LDS; as the registers lie, a store covers
// 16 bytes of each of 32 rows (32/8 heads, d 128, 1024 tokens over 983 keys 40.6 -> 39.2 us, 443 over 43 17.3 -> 16.6, 32 over 40
// 10.9 -> 10.0).  Launches of fewer than 64 rows a KV head are the faster without (2 KV heads of 2, d 64, 17 tokens 6.4 / 6.6 us), and so
// are blocks of eight at d 64 (1 - 1.5 % in launches of many rounds).  (As a run-time choice it cost all others 2 - 5 %.)
template <int D, bool SPLIT, bool XS, bool KSPLIT, bool WHOLE>
__global__ __launch_bounds__(2 * kSetThreads, 2) void attn_bf16(Dims dm, AttnArgs a) {
  using Cfg = AttnCfg<D, SPLIT>;
  constexpr bool DMA = Cfg::DMA;
  constexpr int KT = Cfg::KT, KS = Cfg::KS, CG = Cfg::CG, RPI = Cfg::RPI, NLD = Cfg::NLD,
                DB = Cfg::DB, HW = Cfg::HW;
  extern __shared__ __align__(16) unsigned char smem[];

  const int kv = blockIdx.x;   // KV head fastest: one head's blocks share an XCD's L2
  const bool sparse = a.k_idx != nullptr;
  // Blocks are dispatched in grid order and a block runs as long as its sequence's key list, so in a ragged batch the
  // sequences are taken longest first (grid slice z works on the sequence of rank z by attended cache length);
  // otherwise a long sequence that happens to come last starts when most of the chip has already drained.
  // (The chunks of a prompt lie shortest first: no length to wait for.)
  int b = dm.prompt_chunks ? dm.b - 1 - (int)blockIdx.z : (int)blockIdx.z;
  if (dm.b > 1 && dm.b <= kWave && !dm.prompt_chunks)
    b = seq_of_rank(sparse ? a.n_cache + kv : a.n_cache, sparse ? dm.n_kv : dm.ls, dm.b, blockIdx.z);
  // The list's length and the arguments that the start needs, fetched together: one by one, where each is first used, they are four fetches
  // in a row.
  const int n_given = a.n_cache[sparse ? b * dm.n_kv + kv : b * dm.ls];
  asm volatile("" ::"s"(dm.g), "s"(dm.C), "s"(dm.T_max), "s"(dm.B_max), "s"(dm.C_last),
               "s"(dm.qs[0]), "s"(dm.qs[1]), "s"(dm.qs[2]), "s"(dm.kvs[0]), "s"(dm.kvs[1]), "s"(dm.kvs[2]), "s"(dm.cks[0]), "s"(dm.cks[1]),
               "s"(dm.cks[2]), "s"(a.q), "s"(a.k_cache), "s"(a.v_cache), "s"(a.k_chunk), "s"(a.v_chunk), "s"(a.k_idx),
               "s"(a.n_cache), "s"(a.adjacent), "s"(a.inv_g));
  const int tid = threadIdx.x % kSetThreads, lane = tid & 63;                 // position inside the wave set
  // wave-uniform values are pinned to scalar registers so that everything derived from them (tile kind, base
  // pointers, branches) stays scalar too
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int set = __builtin_amdgcn_readfirstlane(threadIdx.x / kSetThreads);
  const int li = lane & 31, hf = lane >> 5;
  const int C = dm.chunk(b), g = dm.g;
  const int ntt = (C + 31) / 32;
  const int nrb = g * ntt;                       // row blocks of this KV head
  const int half = (nrb + 1) / 2;                // row blocks [0, half) are "front", [half, nrb) "back"
  // SPLIT: slots 0,1 front, 2,3 back, and set 1's waves are rotated by two so that each SIMD hosts a front and a back
  // row block.  Otherwise set 0 is front, set 1 back.
  const int slot = SPLIT ? (w + 2 * set) % 4 : w + 4 * set;
  const bool back = SPLIT ? slot >= 2 : set == 1;
  const int yb = KSPLIT ? (int)((blockIdx.y * a.inv_splits) >> 16) : (int)blockIdx.y;   // group of row blocks
  const int split = KSPLIT ? (int)blockIdx.y - yb * a.n_splits : 0;                               // share of its key list
  const int kf = yb * HW + slot % HW;
  // Row blocks of a block.  Paired (a launch of one round): half from the front of the list, half from the back, so all
  // blocks take equally long.  Adjacent (a launch of several rounds): 2*HW neighbours with nearly the same causal range,
  // so no wave idles while others still have chunk keys to go, and the blocks with the longest ranges come first
  // in the grid: the compute units that finish the short blocks early pick up more of what is left.
  const bool adjacent = a.adjacent != 0;
  const int x = adjacent ? nrb - 1 - (yb * 2 * HW + slot) : (back ? nrb - 1 - kf : kf);
  const bool wave_on = adjacent ? x >= 0 : (back ? (x >= half) : (x < half));
  const int xt = wave_on ? (int)((uint32_t)x * a.inv_g >> 16) : 0;   // x / g
  const int xj = wave_on ? x - xt * g : 0;
  const int tok0 = xt * 32;
  const int h = kv * g + xj;
  const int xb_hi = nrb - 1 - yb * HW;                                     // the block's last row block
  const int x_hi = adjacent ? nrb - 1 - yb * 2 * HW
                            : (xb_hi >= half ? xb_hi : min(yb * HW + HW - 1, half - 1));
  if (adjacent ? x_hi < 0 : yb * HW >= half) return;   // a short chunk has no row blocks here (block-uniform)
  const int c_end_blk = min((int)((uint32_t)x_hi * a.inv_g >> 16) * 32 + 32, C);   // chunk keys any wave of this block can see
  const int sub = SPLIT ? set * kSub : 0;               // first key of this set's share of a staged tile

  // The tensor this set stages (set 0: K, set 1: V) for this (batch, KV head), as byte pointers: every row is
  // addressed as base + 32-bit byte offset (the host checks that a head's rows span less than 4 GiB).
  const void* cache_t = set == 0 ? a.k_cache : a.v_cache;
  const void* chunk_t = set == 0 ? a.k_chunk : a.v_chunk;
  const char* cache_base = reinterpret_cast<const char*>(static_cast<const uint16_t*>(cache_t) + b * dm.kvs[0] + kv * dm.kvs[1]);
  const char* chunk_base = reinterpret_cast<const char*>(static_cast<const uint16_t*>(chunk_t) + b * dm.cks[0] + kv * dm.cks[1]);
  const char* kidx = sparse ? reinterpret_cast<const char*>(a.k_idx + (size_t)(b * dm.n_kv + kv) * dm.B_max) : nullptr;
  const uint32_t cache_row_bytes = (uint32_t)dm.kvs[2] * 2u, chunk_row_bytes = (uint32_t)dm.cks[2] * 2u;
  // Staging.  Thread (r0, cg) fetches slot cg of rows r0 + RPI * k of this set's tensor, k < NLD: a load of a wave fills a group.
  // Source rows of a tile are looked up a step ahead of the loads that use them, so the dependent index -> row fetch of the gather
  // never sits on the critical path.  At d 128 the 16 lanes that carry a row look up NLD rows between them, one each, and take
  // them from each other where they are used: one register instead of NLD.
  constexpr bool kShare = CG == 16;
  constexpr int NI = kShare ? 1 : NLD;
  const int r0 = tid / CG;
  const uint32_t cg_src = (uint32_t)(tid % CG ^ (set == 0 ? k_swizzle<D>(lane / CG) : v_swizzle<D>(lane / CG))) * 16u;
  const uint32_t idx_max = (uint32_t)max(dm.T_max - 1, 0);
  uint32_t src[NI];     // rows of the tile to be requested next, as looked up
  uint32_t off[NI];     // the same as byte offsets, of the tile being requested
  u32x4 R[DMA ? 1 : NLD];   // the tile in flight (not DMA)
  const char* req_base = nullptr;   // of the tile being requested
  const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) void*)smem;
  const uint32_t group_mine = set == 0 ? Cfg::KG : Cfg::VG;
  const uint32_t dst_mine = lds0 + (set == 0 ? 0u : (uint32_t)Cfg::kKTileBytes) + (uint32_t)w * group_mine;
  auto stage_of = [&](int t) __attribute__((always_inline)) { return (t & 1) * Cfg::kStageBytes; };
  auto request = [&](int t, int k) __attribute__((always_inline)) {   // chunk k of tile t
    const uint32_t o = kShare ? row16_lane(off[0], k) + cg_src : off[k % NI];
    if constexpr (DMA) dma16(req_base, o, dst_mine + (uint32_t)stage_of(t) + 4u * k * group_mine);
    else R[k] = *reinterpret_cast<const u32x4*>(req_base + o);
  };
  auto q_area = [&](int t_first) __attribute__((always_inline)) {
    return lds0 + (uint32_t)(SPLIT ? stage_of(t_first + 1) + Cfg::kKTileBytes : 2 * Cfg::kStageBytes);
  };
  // A block's start is a chain of fetches, in a launch of many rounds one for every round, so what does not wait for the list's length
  // leaves at once: the list's first entries, the chunk's first tile and the queries.  The entries are looked up for a list that fills its
  // first tile, and again where it does not.  (Length, queries, entries and tile one after the other took 5.2 us to the first product in
  // 32/8 heads, 1024 tokens over 983 keys, now 3.8, of which 1.3 until the arguments are there.  Attention by itself, 200 random calls of
  // 2 - 4096 tokens: 0.95 of the time, d 128 0.96 - 0.92, d 64 0.99 - 0.96; 54 tokens over 132 keys 10.8 -> 9.5 us, 573 over 2084
  // 37.6 -> 35.4.)
  if constexpr (!KSPLIT) {
    if (sparse) {
#pragma unroll
      for (int i = 0; i < NI; ++i)
        src[i] = *reinterpret_cast<const uint32_t*>(kidx + (uint32_t)min(r0 + RPI * (kShare ? lane % NLD : i), max(dm.B_max - 1, 0)) * 4u);
    }
    req_base = chunk_base;
#pragma unroll
    for (int i = 0; i < NI; ++i)
      off[i] = (uint32_t)min(r0 + RPI * (kShare ? lane % NLD : i), C - 1) * chunk_row_bytes + (kShare ? 0u : cg_src);
#pragma unroll
    for (int k = 0; k < NLD; ++k) request(-1, k);
  }
  // Q goes through LDS too, in whole rows.  (As operands a load takes 16 bytes of each of 64 lines: 1.7 us for a block's.)
  // SPLIT: the two waves of a slot fetch half of its rows each, to where V of the second tile goes later.
  auto request_q = [&](uint32_t area) __attribute__((always_inline)) {
    constexpr int N = 32 / Cfg::RPW / (SPLIT ? 2 : 1);
    const uint16_t* qhead = static_cast<const uint16_t*>(a.q) + b * dm.qs[0] + h * dm.qs[1];
#pragma unroll
    for (int i = 0; i < N; ++i) {
      const int r = ((SPLIT ? set * N : 0) + i) * Cfg::RPW + lane / CG;
      const uint16_t* p = qhead + (size_t)min(tok0 + r, C - 1) * dm.qs[2] + (lane % CG ^ q_swizzle<D>(r)) * 8;
      dma16(p, area + slot * (32 * Cfg::ROW) + (uint32_t)((SPLIT ? set * N : 0) + i) * 1024u);
    }
  };
  if constexpr (!KSPLIT) request_q(q_area(-1));
  const int n_cache = max(min(n_given, sparse ? dm.B_max : dm.T_max), 0);
  // Tile order: the chunk's first tile, the cache tiles, the chunk's other tiles.  What a wave can see is one run of tiles [w0, w1), whose
  // end is where its causal range ends; the first tile needs no index look-up, so its loads leave right at kernel start; and every row
  // of a chunk sees all of it, but for the first rows, so that the reference point taken from it (below) is a maximum over as many keys
  // as a tile has.  (With the chunk's tiles from the last to the first a row met the tile of its diagonal first, of which it may see
  // a single key; the largest probability is then less often 1, the only one that is not rounded: the outputs of a first chunk of 1024
  // tokens lay 0.27 % further from float64, of 2048 0.46 %, of 1024 over 100 keys 0.27 %.)
  const int n_cht = (c_end_blk + KT - 1) / KT;
  const int n_ct = (n_cache + KT - 1) / KT;
  const int n_tiles = n_cht + n_ct;
  // Tiles are numbered from -1, so that the cache tiles are 0 .. n_ct - 1.
  const int t_begin = (KSPLIT ? (int)((uint32_t)n_tiles * (uint32_t)split / (uint32_t)a.n_splits) : 0) - 1;
  const int t_end = (KSPLIT ? (int)((uint32_t)n_tiles * (uint32_t)(split + 1) / (uint32_t)a.n_splits) : n_tiles) - 1;
  auto is_cache = [&](int t) __attribute__((always_inline)) { return (uint32_t)t < (uint32_t)n_ct; };
  // first key (cache slot or chunk position) of tile t
  auto tile_base = [&](int t) __attribute__((always_inline)) { return (is_cache(t) ? t : max(t - (n_ct - 1), 0)) * KT; };
  const int seen = tok0 + 31 >= sub ? (tok0 + 31 - sub) / KT + 1 : 0;   // chunk tiles of whose share for this set the wave sees something
  // Tiles whose unit u has keys that not every row sees: at the end of the cache list, and the last chunk tile (-2: none).
  int tail_tile[2], diag_tile[2];
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    tail_tile[u] = n_ct > 0 && (n_ct - 1) * KT + sub + 32 * u + 32 > n_cache ? n_ct - 1 : -2;
    diag_tile[u] = max(seen - 1, 0) * KT + sub + 32 * u + 31 > tok0 ? (seen <= 1 ? -1 : n_ct + seen - 2) : -2;
  }
  int w0 = seen > 0 ? -1 : 0;
  int w1 = n_ct + max(seen - 1, 0);
  if (seen <= 1 && n_ct > 0 && (n_ct - 1) * KT + sub >= n_cache) --w1;   // (the share of the last cache tile may be empty)
  w0 = max(w0, t_begin);
  w1 = min(w1, t_end);
  if (!wave_on || w0 >= w1) w0 = w1 = t_end + 1;   // sees nothing: stages its part of the tiles only

  // Source rows of tile t.  kShare: only entries of the list are fetched, for a chunk tile too (some entry, which is not used), and other
  // rows are worked out where they are requested: as a choice between a fetch and a number the value changes registers, and the step
  // that asks for an entry waits for it.  (d 64 keeps either: the vector unit sets the pace there.)
  const int list_last = max(n_cache - 1, 0);
  auto row_of = [&](int t, int i) __attribute__((always_inline)) {   // tail slots repeat a real row
    return (uint32_t)min(tile_base(t) + r0 + RPI * (kShare ? lane % NLD : i), (is_cache(t) ? n_cache : C) - 1);
  };
  auto look_up = [&](int t) __attribute__((always_inline)) {
    t = min(t, t_end - 1);   // (past the list's end the last tile is requested again, and nothing reads it)
    if constexpr (kShare) {
      if (!sparse) return;
      src[0] = *reinterpret_cast<const uint32_t*>(kidx + (uint32_t)min(max(t, 0) * KT + r0 + RPI * (lane % NLD), list_last) * 4u);
    } else {
      const bool cache = is_cache(t);
      const int base = tile_base(t), last = cache ? n_cache - 1 : C - 1;
#pragma unroll
      for (int i = 0; i < NI; ++i) src[i] = (uint32_t)min(base + r0 + RPI * i, last);
      if (cache && sparse) {
#pragma unroll
        for (int i = 0; i < NI; ++i) src[i] = *reinterpret_cast<const uint32_t*>(kidx + src[i] * 4u);
      }
    }
  };
  // (the clamp to the cache extent: a malformed list, negative or too large, cannot leave the tensor)
  auto address = [&](int t) __attribute__((always_inline)) {
    t = min(t, t_end - 1);
    const bool cache = is_cache(t);
    req_base = cache ? cache_base : chunk_base;
    const uint32_t row_bytes = cache ? cache_row_bytes : chunk_row_bytes;
    if constexpr (kShare) {
      if (cache && sparse) off[0] = min(src[0], idx_max) * cache_row_bytes;
      else off[0] = row_of(t, 0) * row_bytes;
    } else {
      const uint32_t row_max = cache ? idx_max : 0xffffffffu;
#pragma unroll
      for (int i = 0; i < NI; ++i) off[i] = min(src[i], row_max) * row_bytes + cg_src;
    }
  };
  auto store = [&](int t, int k, u32x4 r) __attribute__((always_inline)) {   // (not DMA)
    *(u32x4 __attribute__((address_space(3)))*)(uintptr_t)(dst_mine + lane * 16u + (uint32_t)stage_of(t) + 4u * k * group_mine) = r;
  };
  // Step j takes chunk k of tile j+2 (K) or j+1 (V) to LDS; through registers it was requested a step earlier.
  auto stage = [&](int j, int k) __attribute__((always_inline)) {
    if constexpr (!DMA) store(j + 2 - set, k, R[k]);
    request(DMA ? j + 2 - set : j + 3 - set, k);
  };

  if constexpr (!KSPLIT) {
    if (n_cache < KT || (!kShare && !sparse)) look_up(0);
  } else if (t_begin < t_end) {   // (a split without tiles contributes the neutral partial)
    request_q(q_area(t_begin));
    look_up(t_begin);
    address(t_begin);
    look_up(t_begin + 1);
#pragma unroll
    for (int k = 0; k < NLD; ++k) request(t_begin, k);
  }
  if (t_begin < t_end && set == 0) {   // K runs one tile ahead of V
    u32x4 first[DMA ? 1 : NLD];
    if constexpr (!DMA) {
#pragma unroll
      for (int k = 0; k < NLD; ++k) first[k] = R[k];
    }
    if (t_begin + 1 < t_end) {
      address(t_begin + 1);
      look_up(t_begin + 2);
      // Not DMA: the queries have arrived before the second tile is requested, into registers, by loads whose number is the compiler's
      // choice.  (It waits here for the entries anyway.  KSPLIT: the queries come ahead of the first tile, which is stored below.)
      if constexpr (!DMA && !KSPLIT) wait_vmcnt<0>();
#pragma unroll
      for (int k = 0; k < NLD; ++k) request(t_begin + 1, k);
    }
    if constexpr (!DMA) {
#pragma unroll
      for (int k = 0; k < NLD; ++k) store(t_begin, k, first[k]);
    }
  }
  // the first tile and the queries have arrived (K of the second tile may be on its way)
  if (set == 0 && t_begin + 1 < t_end) {
    if constexpr (DMA) wait_vmcnt<NLD>();
  } else {
    wait_vmcnt<0>();
  }
  __syncthreads();
  // Q operand: row tok0 + li, chunk ks + KS*hf of 8 dims
  bf16x8 qreg[KS];
#pragma unroll
  for (int ks = 0; ks < KS; ++ks)
    qreg[ks] = *(const bf16x8 __attribute__((address_space(3)))*)(uintptr_t)(q_area(t_begin) + slot * (32 * Cfg::ROW) + li * Cfg::ROW +
                                                                             ((ks + KS * hf) ^ q_swizzle<D>(li)) * 16);
  // the softmax scale and the change to base 2
  const float qscale = 1.4426950408889634f / sqrtf((float)D);
  if constexpr (!XS) {   // into Q once, so K Q^T arrives in the exponent's own units
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
#pragma unroll
      for (int e = 0; e < 8; ++e) qreg[ks][e] = (__bf16)((float)qreg[ks][e] * qscale);
  }

  f32x16 o[DB];
#pragma unroll
  for (int c = 0; c < DB; ++c)
#pragma unroll
    for (int v = 0; v < 16; ++v) o[c][v] = 0.f;
  float m_run = -INFINITY;   // running row max, in the scaled log2 domain
  float l_run = 0.f;         // this half wave's share of the running row sum
  // The reference point m_run only moves when a unit's maximum exceeds it by more than kLazy (in the log2 domain): exp2(s - m_run)
  // then stays below 2^kLazy, and rescaling the accumulators becomes rare.  `moves_above` is what a maximum is compared with (XS: in the
  // scaled log2 domain, else relative to the reference point): any score at all moves a row that has none yet.
  constexpr float kLazy = 8.0f;
  float moves_above = -INFINITY;
  // What the accumulator of K Q^T starts from.  !XS: -m_run in every entry, so the matrix core hands back s - m_run
  // and the exponential needs no subtraction of its own; rewritten only when the reference point moves.  XS: zero.
  f32x16 cinit;
#pragma unroll
  for (int v = 0; v < 16; ++v) cinit[v] = 0.f;
  const int tok = tok0 + li;
  f32x16 s[2];          // S^T of a tile's two units of 32 keys
  bf16x8 kop[KS];       // K operands of the unit whose S is formed next
  s16x4 vop[2 * DB][2]; // V^T operands of the unit whose P V follows: block t2 * DB + c
  bf16x8 p[2];          // P of that unit: k-slot e of this lane is key 16*t2 + 8*(e/4) + 4*hf + e%4

  // Chunk c of row r of a group lies at slot c ^ k_swizzle(r) (K: the low two bits) or c ^ v_swizzle(r) (V: bit 2 and 3).
  uint32_t ka[4];     // K: places of chunks ks % 4 (+ KS for the upper half wave) of row li
#pragma unroll
  for (int q = 0; q < 4; ++q)
    ka[q] = lds0 + (uint32_t)(stage_of(w0) + (sub + li) / Cfg::RPW * Cfg::KG + li % Cfg::RPW * Cfg::ROW +
                              ((q ^ k_swizzle<D>(li % Cfg::RPW)) + KS * hf) * 16);
  // V: the lane's corner of the transposing reads of dim block c: key 4*hf + (lane%16)/4, dims 16*((lane/16)%2) + 4*(lane%4)
  uint32_t va[DB];
#pragma unroll
  for (int c = 0; c < DB; ++c) {
    const int r = 4 * hf + ((lane & 15) >> 2);
    va[c] = lds0 + (uint32_t)(stage_of(w0) + Cfg::kKTileBytes + (sub + r) * Cfg::ROW +
                              (((4 * c) ^ v_swizzle<D>(r % Cfg::RPW)) + 2 * ((lane >> 4) & 1) + ((lane & 3) >> 1)) * 16 + 8 * (lane & 1));
  }
  // (the places move between the two stages by one addition a tile each)
  auto move_k = [&](int t) __attribute__((always_inline)) {   // from tile t to tile t + 1
    const uint32_t by = (uint32_t)((t & 1) ? -Cfg::kStageBytes : Cfg::kStageBytes);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      ka[q] += by;
      asm volatile("" : "+v"(ka[q]));
    }
  };
  auto move_v = [&](int t) __attribute__((always_inline)) {
    const uint32_t by = (uint32_t)((t & 1) ? -Cfg::kStageBytes : Cfg::kStageBytes);
#pragma unroll
    for (int c = 0; c < DB; ++c) {
      va[c] += by;
      asm volatile("" : "+v"(va[c]));
    }
  };
  auto read_k = [&](int u, int i) __attribute__((always_inline)) {
    kop[i] = ((const bf16x8 __attribute__((address_space(3)))*)(uintptr_t)ka[i % 4])[i / 4 * 4 + u * (32 / Cfg::RPW * Cfg::KG / 16)];
  };
  auto qk_step = [&](f32x16& sn, int i) __attribute__((always_inline)) {
    sn = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kop[i], qreg[i], i == 0 ? cinit : sn, 0, 0, 0);
  };
  // scores 2*e, 2*e+1 of a unit as probabilities: rounded to bf16, and added to the row sum as the matrix core sees them
  auto to_p = [&](const f32x16& sc, int e, float psum) __attribute__((always_inline)) {
    const bf16x2 pp = {(__bf16)sc[2 * e], (__bf16)sc[2 * e + 1]};
    p[e / 4][2 * (e % 4)] = pp[0];
    p[e / 4][2 * (e % 4) + 1] = pp[1];
    return __builtin_amdgcn_fdot2_f32_bf16(pp, bf16x2{(__bf16)1.0f, (__bf16)1.0f}, psum, false);
  };

  // First half of a unit: S of the unit after it (`next`), and its own scores become probabilities meanwhile.
  // The order of instructions is fixed: after every MFMA the operand reads of a step of the second half and 16 / KS exponentials.
  auto half_qk = [&](auto next, f32x16& sn, f32x16& sc, int u, auto between) __attribute__((always_inline)) {
    constexpr int E = 16 / KS;
    const float neg_m = XS ? (m_run == -INFINITY ? 0.f : -m_run) : 0.f;   // (a row that has seen nothing yet: all its scores are -inf)
    float psum = 0.f;
#pragma unroll
    for (int i = 0; i < KS; ++i) {
      if constexpr (decltype(next)::value) {
        qk_step(sn, i);
        __builtin_amdgcn_sched_barrier(0);
      }
      const tr_ptr vp_c = (tr_ptr)(uintptr_t)va[i % DB] + (32 * u + 16 * (i / DB)) * Cfg::ROW / 8;
      vop[i][0] = __builtin_amdgcn_ds_read_tr16_b64_v4i16(vp_c);
      vop[i][1] = __builtin_amdgcn_ds_read_tr16_b64_v4i16(vp_c + Cfg::ROW);
#pragma unroll
      for (int e = E * i; e < E * i + E; ++e) sc[e] = __builtin_amdgcn_exp2f(XS ? fmaf(sc[e], qscale, neg_m) : sc[e]);
      if (i > 0) {
#pragma unroll
        for (int e = E / 2 * (i - 1); e < E / 2 * i; ++e) psum = to_p(sc, e, psum);
      }
      between(i);
      __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int e = E / 2 * (KS - 1); e < 8; ++e) psum = to_p(sc, e, psum);
    l_run += psum;
    asm volatile("" : "+v"(p[0]), "+v"(p[1]), "+v"(l_run));   // (or the compiler moves all of it behind the next branch)
    __builtin_amdgcn_sched_barrier(0);
  };
  // Second half of a unit: O^T += V^T P^T; meanwhile the maximum of the next unit's scores, which it returns, and the K operands
  // of the unit after that.
  auto half_pv = [&](auto next, const f32x16& sn, int u, auto between) __attribute__((always_inline)) {
    constexpr int E = 16 / KS;
    float mx = -INFINITY;
#pragma unroll
    for (int i = 0; i < KS; ++i) {
      const s16x8 both = __builtin_shufflevector(vop[i][0], vop[i][1], 0, 1, 2, 3, 4, 5, 6, 7);
      o[i % DB] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, both), p[i / DB], o[i % DB], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
      if constexpr (decltype(next)::value) {
        read_k(u, i);
#pragma unroll
        for (int e = E * i; e < E * i + E; ++e) mx = fmaxf(mx, sn[e]);
        asm volatile("" : "+v"(mx));   // (or all of it ends up behind the last product)
      }
      between(KS + i);
      __builtin_amdgcn_sched_barrier(0);
    }
    return mx;
  };
  // Keys of unit u of tile t that a row does not see (wave-uniform branch).
  auto mask = [&](f32x16& sn, int t, int u) __attribute__((always_inline)) {
    if (t == tail_tile[u] || t == diag_tile[u]) {
      // register v is key 8*(v/4) + v%4 past the lane's first
      const int limit = (is_cache(t) ? n_cache : tok + 1) - (tile_base(t) + sub + 32 * u) - 4 * hf;
#pragma unroll
      for (int v = 0; v < 16; ++v)
        if (8 * (v / 4) + v % 4 >= limit) sn[v] = -INFINITY;
    }
  };
  // Whether any row sees a key of the second unit of tile t: half of all row blocks end in the first unit of their last tile, and so do
  // lists of up to 32 keys (32 heads, 20 tokens over 30 keys: d 64 7.3 -> 6.8 us, d 128 9.3 -> 8.3; 260 tokens alone, d 64 8.0 -> 7.6).
  // (Not asked where the list is shared: the time is that of a block whose tiles are full, and the question cost it 1 %.)
  auto both_units = [&](int t) __attribute__((always_inline)) {
    if constexpr (KSPLIT) return true;
    const int base = tile_base(t) + sub + 32;
    return is_cache(t) ? base < n_cache : base <= tok0 + 31;
  };
  // Moves the reference point where the maximum asks for it (wave-uniform branch, rare).
  auto move_reference = [&](f32x16& sn, float mx) __attribute__((always_inline)) {
    if constexpr (XS) mx *= qscale;   // (the products themselves are raw)
    if (__builtin_amdgcn_ballot_w64(mx > moves_above) != 0) {
      mx = fmaxf(mx, other_half(mx));   // of the row
      const bool moves = mx > moves_above;
      const float m_old = (m_run == -INFINITY) ? 0.f : m_run;    // !XS: what the scores are relative to
      const float m_new = !moves ? m_run : XS ? mx : m_old + mx;
      const float m_fin = (m_new == -INFINITY) ? 0.f : m_new;
      const float alpha = __builtin_amdgcn_exp2f(m_run - m_fin);   // 0 for a row without a reference so far, 1 if unmoved
      m_run = m_new;
      moves_above = m_new == -INFINITY ? -INFINITY : XS ? m_new + kLazy : kLazy;
      l_run *= alpha;
#pragma unroll
      for (int c = 0; c < DB; ++c)
#pragma unroll
        for (int v = 0; v < 16; ++v) o[c][v] *= alpha;
      if constexpr (!XS) {
        const float shift = m_fin - m_old;
#pragma unroll
        for (int v = 0; v < 16; ++v) sn[v] -= shift;
#pragma unroll
        for (int v = 0; v < 16; ++v) cinit[v] = -m_fin;
      }
    }
  };

  using yes = std::integral_constant<bool, true>;
  using no = std::integral_constant<bool, false>;
  // Step j of the block: K of tile j+2 and V of tile j+1 go to LDS (set 0: K, set 1: V) and every wave works on tile j.  One barrier a
  // step.  What step j brings is complete before the barrier of step j+1 (the wait and the fence ahead of it), in which it is first
  // read: the K operands of tile j+1 are read during tile j.  The places it takes held K of tile j and V of tile j-1, whose last reads
  // ended before the barrier of step j (the fence again).  DMA: the first step's tiles are requested ahead of the loop.  (Whether a step
  // can be the first is settled when it is compiled: asked in every step, and with a second tile requested and waited for where a block has
  // only one, d 64 was 2 % slower on the mean of 2000 calls, d 128 1 %; 8 KV heads of 4, d 128, 1074 tokens over 3487 keys
  // 96.1 -> 92.8 us.)
  auto begin_step = [&](int j, auto can_be_first) __attribute__((always_inline)) {
    const bool first = decltype(can_be_first)::value && j < t_begin;   // (its barrier is the one above)
    if constexpr (DMA) {
      if (first) return;
      wait_vmcnt<0>();
    }
    if (!first) __syncthreads();
    if constexpr (!kShare && DMA) {   // (or the new entries are waited for, to be moved to where these are)
#pragma unroll
      for (int i = 0; i < NI; ++i) asm volatile("" : "+v"(src[i]));
    }
    address(DMA ? j + 2 - set : j + 3 - set);
    look_up(DMA ? j + 3 - set : j + 4 - set);
  };
  auto stage_all = [&](int j, auto can_be_first) __attribute__((always_inline)) {
    if (DMA && ((decltype(can_be_first)::value && j < t_begin) || j + 2 - set >= t_end)) return;
#pragma unroll
    for (int k = 0; k < NLD; ++k) stage(j, k);
  };
  auto nothing = [](int) __attribute__((always_inline)) {};
  int j = t_begin < t_end ? t_begin - 1 : t_end;
  for (; j < min(w0 - 1, t_end); ++j) {
    begin_step(j, yes{});
    stage_all(j, yes{});
  }
  if (w0 < w1) {
    // The staging of a step, a load at a time: between the products of the first unit's second half, or, where there are as many
    // chunks as products in it (blocks of four row blocks, d 128), of both its halves.
    auto staging = [&](int i) __attribute__((always_inline)) {
      constexpr int first = NLD == KS ? 0 : KS, every = (2 * KS - first) / NLD;
      if (i >= first && (i - first) % every == 0) stage(j, (i - first) / every);
    };
    begin_step(j, yes{});
    {   // S of the first unit, the operands of the second, the reference point
#pragma unroll
      for (int i = 0; i < KS; ++i) read_k(0, i);
#pragma unroll
      for (int i = 0; i < KS; ++i) qk_step(s[0], i);
#pragma unroll
      for (int i = 0; i < KS; ++i) read_k(1, i);
      mask(s[0], w0, 0);
      float mx = -INFINITY;
#pragma unroll
      for (int v = 0; v < 16; ++v) mx = fmaxf(mx, s[0][v]);
      // The reference point is the maximum over the whole tile, whose second unit is formed for it and again in its turn: where a row's
      // largest probability is 1 it is not rounded (with the first unit's maximum alone outputs lay 0.5 % further from float64; 0.3 us).
      if (both_units(w0)) {   // (wave-uniform)
#pragma unroll
        for (int i = 0; i < KS; ++i) qk_step(s[1], i);
        mask(s[1], w0, 1);
#pragma unroll
        for (int v = 0; v < 16; ++v) mx = fmaxf(mx, s[1][v]);
      }
      move_reference(s[0], mx);
    }
    stage_all(j++, yes{});
    for (; j + 1 < w1; ++j) {
      begin_step(j, no{});
      move_k(j);
      half_qk(yes{}, s[1], s[0], 0, staging);
      mask(s[1], j, 1);
      float mx = half_pv(yes{}, s[1], 0, staging);
      move_reference(s[1], mx);
      half_qk(yes{}, s[0], s[1], 1, nothing);
      move_v(j);
      mask(s[0], j + 1, 0);
      mx = half_pv(yes{}, s[0], 1, nothing);
      move_reference(s[0], mx);
    }
    begin_step(j, no{});
    stage_all(j, no{});
    if (both_units(j)) {
      half_qk(yes{}, s[1], s[0], 0, nothing);
      mask(s[1], j, 1);
      float mx = -INFINITY;
#pragma unroll
      for (int v = 0; v < 16; ++v) mx = fmaxf(mx, s[1][v]);
      half_pv(no{}, s[1], 0, nothing);
      move_reference(s[1], mx);
      if constexpr (!KSPLIT) {   // the second unit takes the first one's place
        s[0] = s[1];
#pragma unroll
        for (int c = 0; c < DB; ++c) va[c] += 32 * Cfg::ROW;   // (V's groups lie one behind the other)
      }
    }
    half_qk(no{}, s[0], s[KSPLIT ? 1 : 0], KSPLIT ? 1 : 0, nothing);
    half_pv(no{}, s[0], 0, nothing);
    ++j;
  }
  for (; j < t_end; ++j) {
    begin_step(j, no{});
    stage_all(j, no{});
  }
  if constexpr (DMA) wait_vmcnt<0>();   // nothing may land in LDS from here on

  // ---- merge of the two wave sets (SPLIT): set 1 hands (m, l, O) to set 0 through LDS ---------------------------
  if constexpr (SPLIT) {
    // (16 bytes a lane and access; m and l behind the rows)
    constexpr int REC = 64 * (DB * 16 + 2);   // floats of a slot: both sets' waves of a slot share rows
    float* mg = reinterpret_cast<float*>(smem) + (size_t)slot * REC;
    __syncthreads();   // all tiles consumed: the tile buffers may be reused
    if (set == 1) {
#pragma unroll
      for (int c = 0; c < DB; ++c)
#pragma unroll
        for (int v4 = 0; v4 < 4; ++v4)
          *reinterpret_cast<float4*>(mg + ((c * 4 + v4) * 64 + lane) * 4) =
              make_float4(o[c][4 * v4], o[c][4 * v4 + 1], o[c][4 * v4 + 2], o[c][4 * v4 + 3]);
      *reinterpret_cast<float2*>(mg + 64 * DB * 16 + 2 * lane) = make_float2(m_run, l_run);
    }
    __syncthreads();
    if (set == 1) return;
    const float2 ml1 = *reinterpret_cast<const float2*>(mg + 64 * DB * 16 + 2 * lane);
    const float m1 = ml1.x, l1 = ml1.y;
    const float m_new = fmaxf(m_run, m1);
    const float m_fin = (m_new == -INFINITY) ? 0.f : m_new;
    const float a0 = __builtin_amdgcn_exp2f(m_run - m_fin), a1 = __builtin_amdgcn_exp2f(m1 - m_fin);
    m_run = m_new;
    l_run = a0 * l_run + a1 * l1;
#pragma unroll
    for (int c = 0; c < DB; ++c)
#pragma unroll
      for (int v4 = 0; v4 < 4; ++v4) {
        const float4 t = *reinterpret_cast<const float4*>(mg + ((c * 4 + v4) * 64 + lane) * 4);
        o[c][4 * v4] = a0 * o[c][4 * v4] + a1 * t.x;
        o[c][4 * v4 + 1] = a0 * o[c][4 * v4 + 1] + a1 * t.y;
        o[c][4 * v4 + 2] = a0 * o[c][4 * v4 + 2] + a1 * t.z;
        o[c][4 * v4 + 3] = a0 * o[c][4 * v4 + 3] + a1 * t.w;
      }
  }

  // ---- epilogue -------------------------------------------------------------------------------
  const float l_tot = l_run + other_half(l_run);
  if constexpr (KSPLIT) {   // the partial goes out as the registers lie, 1 KiB per store
    if (!wave_on) return;
    float* rec = a.part + (((size_t)(b * dm.n_kv + kv) * (g * ((dm.C + 31) / 32)) + x) * a.n_splits + split) * Cfg::kRecFloats;
#pragma unroll
    for (int c = 0; c < DB; ++c)
#pragma unroll
      for (int v4 = 0; v4 < 4; ++v4)
        *reinterpret_cast<float4*>(rec + ((c * 4 + v4) * 64 + lane) * 4) =
            make_float4(o[c][4 * v4], o[c][4 * v4 + 1], o[c][4 * v4 + 2], o[c][4 * v4 + 3]);
    if (hf == 0) {
      rec[32 * D + li] = m_run;
      rec[32 * D + 32 + li] = l_tot;
    }
    return;
  }
  if constexpr (!WHOLE) {
    if (wave_on && tok < C) {
      const float inv = 1.0f / l_tot;
      uint16_t* orow = static_cast<uint16_t*>(a.out) + b * dm.os[0] + h * dm.os[1] + (size_t)tok * dm.os[2];
#pragma unroll
      for (int c = 0; c < DB; ++c)
#pragma unroll
        for (int v4 = 0; v4 < 4; ++v4) {   // registers 4*v4 .. 4*v4+3 are four consecutive dims
          *reinterpret_cast<uint2*>(orow + 32 * c + 8 * v4 + 4 * hf) =
              make_uint2(bf16_pair(o[c][4 * v4] * inv, o[c][4 * v4 + 1] * inv), bf16_pair(o[c][4 * v4 + 2] * inv, o[c][4 * v4 + 3] * inv));
        }
      if (a.lse != nullptr && hf == 0)
        a.lse[(size_t)(b * dm.n_q + h) * dm.C + tok] = (m_run + log2f(l_tot)) * 0.6931471805599453f;
    }
    return;
  }
  constexpr int OLD = D + 8;   // pitch (elements)
  // SPLIT: the piece is the one whose records this wave's lanes have just read, each its own; a lane's stores go to the
  // others' records, so the reads of all lanes come first.  (A wave's LDS accesses stay in the order they are issued in: the
  // fence orders the compiler and costs no instruction.)
  if constexpr (SPLIT) {
    wave_fence();
  } else {
    __syncthreads();   // all tiles consumed
  }
  uint16_t* ot = reinterpret_cast<uint16_t*>(smem) + (SPLIT ? (size_t)slot * 64 * (2 + DB * 16) * 2 : (size_t)slot * 32 * OLD);
  if (!wave_on) return;
  const float inv = 1.0f / l_tot;
#pragma unroll
  for (int c = 0; c < DB; ++c)
#pragma unroll
    for (int v4 = 0; v4 < 4; ++v4) {   // registers 4*v4 .. 4*v4+3 are four consecutive dims
      *reinterpret_cast<uint2*>(ot + li * OLD + 32 * c + 8 * v4 + 4 * hf) =
          make_uint2(bf16_pair(o[c][4 * v4] * inv, o[c][4 * v4 + 1] * inv), bf16_pair(o[c][4 * v4 + 2] * inv, o[c][4 * v4 + 3] * inv));
    }
  if (a.lse != nullptr && hf == 0 && tok < C)
    a.lse[(size_t)(b * dm.n_q + h) * dm.C + tok] = (m_run + log2f(l_tot)) * 0.6931471805599453f;
  wave_fence();   // (the rows are read back by other lanes)
  uint16_t* obase = static_cast<uint16_t*>(a.out) + b * dm.os[0] + h * dm.os[1] + (size_t)tok0 * dm.os[2] + (lane % CG) * 8;
  u32x4 rows_out[32 * CG / 64];   // all read before the first goes out
#pragma unroll
  for (int i = 0; i < 32 * CG / 64; ++i)
    rows_out[i] = *reinterpret_cast<const u32x4*>(ot + (i * (64 / CG) + lane / CG) * OLD + (lane % CG) * 8);
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int i = 0; i < 32 * CG / 64; ++i) {
    const int r = i * (64 / CG) + lane / CG;
    if (tok0 + r < C) *reinterpret_cast<u32x4*>(obase + (size_t)r * dm.os[2]) = rows_out[i];
  }
}

// Sum of the key splits' partials: a wave takes one dim block of a row block and up to kMergeRun neighbouring splits at a time, all of
// whose records are requested before the first is used, and the sums of the waves that share a dim block meet in LDS.  A block
// is all waves of a row block where those are at most eight, else those of a dim block (`dims` of a block).  The lane layout is
// the attention kernel's own, so the loads are whole kilobytes.  Everything is added in a fixed order.
// What bounds it is the chain of fetches, not the bytes: with one wave walking a dim block's splits two at a time the launch took
// 0.4 us a split (8 heads, d 64, 103 tokens, 32 splits 15.4 us, now 5.4; 2 heads of 7, d 128, 5 tokens 13.2, now 4.4; 4 heads
// of 3, d 128, 147 tokens 9.3, now 5.3).
constexpr int kMergeWaves = 8, kMergeRun = 4;
template <int D>
__global__ __launch_bounds__(64 * kMergeWaves) void attn_bf16_merge(Dims dm, AttnArgs a, int dims) {
  constexpr int REC = AttnCfg<D, true>::kRecFloats;
  __shared__ float2 ml[kMergeWaves][32];
  __shared__ float4 sum[kMergeWaves][4][64];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int w = wave / dims, nw = (int)(blockDim.x >> 6) / dims;   // of the dim block
  const int li = lane & 31, hf = lane >> 5;
  const int x = blockIdx.x, kv = blockIdx.y % dm.n_kv, b = blockIdx.y / dm.n_kv, c = (int)blockIdx.z * dims + wave % dims;
  const int C = dm.chunk(b);
  if (x >= dm.g * ((C + 31) / 32)) return;   // block-uniform
  const float* rec = a.part + ((size_t)blockIdx.y * gridDim.x + x) * a.n_splits * REC;
  const int s0 = a.n_splits * w / nw, s1 = a.n_splits * (w + 1) / nw;
  float m = -INFINITY, l = 0.f;
  float o[16];
#pragma unroll
  for (int v = 0; v < 16; ++v) o[v] = 0.f;
  for (int s = s0; s < s1; s += kMergeRun) {
    float ms[kMergeRun], ls[kMergeRun];
    float4 t[kMergeRun][4];
#pragma unroll
    for (int i = 0; i < kMergeRun; ++i) {
      if (s + i < s1) {   // (wave-uniform)
        const float* p = rec + (size_t)(s + i) * REC;
        ms[i] = p[32 * D + li];
        ls[i] = p[32 * D + 32 + li];
#pragma unroll
        for (int v4 = 0; v4 < 4; ++v4) t[i][v4] = *reinterpret_cast<const float4*>(p + ((c * 4 + v4) * 64 + lane) * 4);
      } else {   // adds zeros
        ms[i] = -INFINITY;
        ls[i] = 0.f;
#pragma unroll
        for (int v4 = 0; v4 < 4; ++v4) t[i][v4] = make_float4(0.f, 0.f, 0.f, 0.f);
      }
    }
    __builtin_amdgcn_sched_barrier(0);   // all of them in flight
    float m_new = m;
#pragma unroll
    for (int i = 0; i < kMergeRun; ++i) m_new = fmaxf(m_new, ms[i]);
    const float m_fin = m_new == -INFINITY ? 0.f : m_new;   // (a row that no split so far has seen a key for)
    const float alpha = __builtin_amdgcn_exp2f(m - m_fin);
    m = m_new;
    l *= alpha;
#pragma unroll
    for (int v = 0; v < 16; ++v) o[v] *= alpha;
#pragma unroll
    for (int i = 0; i < kMergeRun; ++i) {
      const float wgt = __builtin_amdgcn_exp2f(ms[i] - m_fin);
      l += wgt * ls[i];
#pragma unroll
      for (int v4 = 0; v4 < 4; ++v4) {
        o[4 * v4] += wgt * t[i][v4].x;
        o[4 * v4 + 1] += wgt * t[i][v4].y;
        o[4 * v4 + 2] += wgt * t[i][v4].z;
        o[4 * v4 + 3] += wgt * t[i][v4].w;
      }
    }
  }
  if (nw > 1) {
    if (hf == 0) ml[wave][li] = make_float2(m, l);
    if (w > 0) {
#pragma unroll
      for (int v4 = 0; v4 < 4; ++v4)
        sum[wave][v4][lane] = make_float4(o[4 * v4], o[4 * v4 + 1], o[4 * v4 + 2], o[4 * v4 + 3]);
    }
    __syncthreads();
    if (w > 0) return;
    float m_all = m;
    for (int i = 1; i < nw; ++i) m_all = fmaxf(m_all, ml[i * dims + wave][li].x);   // (w is 0: wave is the dim block's place)
    const float m_fin = m_all == -INFINITY ? 0.f : m_all;
    const float alpha = __builtin_amdgcn_exp2f(m - m_fin);
    m = m_all;
    l *= alpha;
#pragma unroll
    for (int v = 0; v < 16; ++v) o[v] *= alpha;
    for (int i = 1; i < nw; ++i) {
      const float wgt = __builtin_amdgcn_exp2f(ml[i * dims + wave][li].x - m_fin);
      l += wgt * ml[i * dims + wave][li].y;
#pragma unroll
      for (int v4 = 0; v4 < 4; ++v4) {
        const float4 t = sum[i * dims + wave][v4][lane];
        o[4 * v4] += wgt * t.x;
        o[4 * v4 + 1] += wgt * t.y;
        o[4 * v4 + 2] += wgt * t.z;
        o[4 * v4 + 3] += wgt * t.w;
      }
    }
  }
  const int tok = (x / dm.g) * 32 + li, h = kv * dm.g + x % dm.g;
  if (tok >= C) return;
  const float inv = 1.0f / l;
  uint16_t* orow = static_cast<uint16_t*>(a.out) + b * dm.os[0] + h * dm.os[1] + (size_t)tok * dm.os[2];
#pragma unroll
  for (int v4 = 0; v4 < 4; ++v4) {
    *reinterpret_cast<uint2*>(orow + 32 * c + 8 * v4 + 4 * hf) =
        make_uint2(bf16_pair(o[4 * v4] * inv, o[4 * v4 + 1] * inv), bf16_pair(o[4 * v4 + 2] * inv, o[4 * v4 + 3] * inv));
  }
  if (a.lse != nullptr && hf == 0 && c == 0)
    a.lse[(size_t)(b * dm.n_q + h) * dm.C + tok] = (m + log2f(l)) * 0.6931471805599453f;
}

template <int D, bool SPLIT, bool XS, bool KSPLIT, bool WHOLE>
static hipError_t launch_variant(const Dims& dm, const AttnArgs& a, hipStream_t st) {
  using Cfg = AttnCfg<D, SPLIT>;
  constexpr size_t lds = Cfg::kLdsBytes;
  static std::atomic<uint64_t> lds_done{0};
  const hipError_t e =
      ensure_dynamic_lds(reinterpret_cast<const void*>(&attn_bf16<D, SPLIT, XS, KSPLIT, WHOLE>), lds, lds_done);
  if (e != hipSuccess) return e;
  const int nrb = dm.g * ((dm.C + 31) / 32);
  const int half = (nrb + 1) / 2;
  dim3 grid(dm.n_kv, (half + Cfg::HW - 1) / Cfg::HW * a.n_splits, dm.b);
  AttnArgs aa = a;
  aa.inv_g = quotient_factor(dm.g);
  aa.inv_splits = quotient_factor(a.n_splits);
  // one block is resident per compute unit: from two rounds on, neighbouring row blocks and longest ranges first
  // (measured at 512 blocks, 4096-token chunk over 131072 cached tokens: 3.5 % faster than pairing; a launch of one
  // round needs the pairing, or its last block sets the time alone)
  aa.adjacent = (long long)grid.x * grid.y * grid.z >= 2 * kComputeUnits ? 1 : 0;
  hipLaunchKernelGGL((attn_bf16<D, SPLIT, XS, KSPLIT, WHOLE>), grid, dim3(2 * kSetThreads), lds, st, dm, aa);
  if (KSPLIT) {
    const int runs = (a.n_splits + kMergeRun - 1) / kMergeRun, waves = runs < kMergeWaves ? runs : kMergeWaves;
    const int dims = waves * (D / 32) <= kMergeWaves ? D / 32 : 1;
    hipLaunchKernelGGL((attn_bf16_merge<D>), dim3(nrb, dm.b * dm.n_kv, D / 32 / dims), dim3(64 * waves * dims), 0, st, dm, aa, dims);
  }
  return hipGetLastError();
}

template <int D, bool SPLIT, bool XS>
static hipError_t launch_dsx(const Dims& dm, const AttnArgs& a, hipStream_t st) {
  if (a.n_splits > 1) return launch_variant<D, SPLIT, XS, true, false>(dm, a, st);
  if constexpr (SPLIT) {
    if (dm.g * dm.C < 64) return launch_variant<D, SPLIT, XS, false, false>(dm, a, st);
  }
  return launch_variant<D, SPLIT, XS, false, SPLIT || D == 128>(dm, a, st);
}

template <int D, bool SPLIT>
static hipError_t launch_ds(const Dims& dm, const AttnArgs& a, hipStream_t st) {
  return dm.flags & QUOKA_ATTN_SCALE_F32 ? launch_dsx<D, SPLIT, true>(dm, a, st) : launch_dsx<D, SPLIT, false>(dm, a, st);
}

// ---- which variant: 8 row blocks per block or 4 (SPLIT), and over how many blocks the key list is split -----------

static int key_splits_limit(const Dims& dm, bool sparse, int keys_per_tile) {
  const long long tiles = ((long long)attended_cap(dm, sparse) + keys_per_tile - 1) / keys_per_tile +
                          (dm.C + keys_per_tile - 1) / keys_per_tile;
  return (int)(tiles < kMaxKeySplits ? tiles : kMaxKeySplits);
}

// Whole key lists of more than 1024 row blocks: eight row blocks per block, or four.
// A batch: eight where that gives every compute unit a block.  (The lengths may differ, which the host cannot know, and then
// smaller blocks fill up the second round where eight row blocks alone would be one.)
// One sequence, d 128: up to 256 groups of eight (one round) eight is the faster in all but one of 1050 measured calls (blocks of four
// take 0.99 - 1.36 of its time); above that blocks of four take three rounds where those of eight take two, up to 384 groups in
// less time (0.84 of it at 257 - 288 groups, 0.97 at 353 - 384); from there on those of eight, whose longest ranges come first, even
// the rounds out (four: 1.03 at 385 - 416 groups, 1.08 - 1.13 beyond).
// d 64: up to 256 groups it depends on how much of the list is the chunk's own, whose causal ranges blocks of four follow more closely; the
// bound is a fit of the two times' difference, in us, to half of 1040 measured calls (0 - 6000 keys; with it they take 0.1 % more than the
// better form, with eight throughout 2.8 %): 12/4 heads, 3203 tokens alone, eight 42.9, four 39.9; 32/8, 1064 tokens over 3000 keys 62 and
// 71.  Up to 384 groups four (0.74 - 0.88), up to 512 where the chunk is more than three fifths of the list (0.90 - 0.96; else 1.01 -
// 1.07), beyond that eight.
static bool eight_row_blocks(const Dims& dm, bool sparse, long long groups) {
  if (dm.b > 1) return groups >= kComputeUnits;
  const float c = (float)attended_cap(dm, sparse) / kSub, r = (float)dm.C / kSub;
  if (groups <= kComputeUnits) return dm.d == 128 || 4.35f + 0.103f * c - r * (0.078f + 9.0f / (float)groups) > 0.f;
  if (dm.d == 64 && 3.f * c < 2.f * r) return groups > 512;
  return groups > 384;
}

// Few row blocks leave compute units idle whatever the tile mode; their key lists are split over blocks instead.
// Measured (kernel and merge, unsplit -> split): 4 KV heads x 3 sequences, d 64, 333 tokens over 4999 keys (2 splits)
// 60 -> 38 us; one KV head of 16 q-heads x 8 sequences, d 64, 69 tokens over 13477 keys (5 splits) 138 -> 65 us.
// The cheapest variant by a model of the call in microseconds: a fixed part, the steps of the longest key list's share times the rounds of
// 256 resident blocks, a part for each further round, and for a split list one for each split, one for the partials' bytes and one where
// there are more than four, whose merge's waves hand their sums to each other.  The numbers are fits to half of 13300 measured calls (2 -
// 3000 tokens over 0 - 20000 keys, at most 1024 row blocks).  On the other half the plans are behind the best of the measured ones, on the
// mean, by 0.4 % (d 64) and 0.8 % (d 128) for 2 - 64 tokens, by 0.4 % for 33 - 3000 tokens and by 0.15 and 0.3 % for one sequence over few
// keys; 12 % for single ones.  (Without the part beyond four splits, fitted to 33 tokens and more: 0.6, 1.1, 0.6 and 0.6 %, 20 %.)  Whole
// lists may take blocks of eight only where ragged row blocks make more than 256 blocks of four: 13 x 4 heads of 3, d 128, 187 tokens over
// 454 keys 34.3 -> 24.8 us.  (Elsewhere they gain up to 5 % on the shortest lists and cost precision: in blocks of four each wave set takes
// its own reference point, so that two probabilities of a row are 1 and not rounded; 65 tokens over 130 keys lie 2.6 % further from float64
// in blocks of eight.)  And not in a batch with room for more than kRaggedKeys keys: its sequences may have fewer, and then the blocks
// beyond 256 are short ones that fill gaps (13 x 4 heads of 3, without and with whole lists in blocks of eight: d 64, 174 tokens over 512
// to 2616 keys 40 and 50 us, over 1868 each 43 and 40; d 128, 171 tokens over 586 to 4688 keys 66 and 105, over 4688 each 133 and 108).
constexpr int kRaggedKeys = 1024;
struct AttnPlan {
  bool split_tile;
  int n_splits;
};

static AttnPlan attn_plan(const Dims& dm, bool sparse) {
  const long long nrb = (long long)dm.g * ((dm.C + 31) / 32), heads = (long long)dm.n_kv * dm.b;
  if (heads * nrb * 2 > kMaxRecords) return AttnPlan{!eight_row_blocks(dm, sparse, heads * ((nrb + 7) / 8)), 1};
  struct Fit {
    float fixed, step, round, per_mb, per_split, beyond_four;   // a step is 8 row blocks x 64 keys or 4 x 128
  };
  constexpr Fit kWhole[2][2] = {{{6.6f, 0.91f, 3.4f, 0.f, 0.f, 0.f}, {4.7f, 0.955f, 6.1f, 0.f, 0.f, 0.f}},    // d 64: eight row blocks, four
                                {{6.9f, 1.14f, 2.f, 0.f, 0.f, 0.f}, {7.2f, 1.26f, 6.7f, 0.f, 0.f, 0.f}}};     // d 128
  constexpr Fit kSplit[2][2] = {{{9.3f, 0.83f, 1.1f, 0.59f, 0.067f, 0.42f}, {7.35f, 1.015f, 0.f, 0.65f, 0.009f, 0.48f}},
                                {{9.8f, 1.2f, 1.45f, 0.45f, 0.017f, 0.6f}, {9.8f, 1.48f, 0.85f, 0.51f, 0.01f, 1.1f}}};
  const int wide = dm.d == 128 ? 1 : 0;
  AttnPlan best{true, 1};
  float best_us = INFINITY;
  for (int mode = 1; mode >= 0; --mode) {
    const int kt = mode == 0 ? kSub : 2 * kSub, per_block = mode == 0 ? 8 : 4;
    const long long blocks = heads * ((nrb + per_block - 1) / per_block);
    const int limit = key_splits_limit(dm, sparse, kt);
    const long long tiles = ((long long)attended_cap(dm, sparse) + kt - 1) / kt + (dm.C + kt - 1) / kt;
    const bool whole = mode == 1 || (heads * ((nrb + 3) / 4) > kComputeUnits && (dm.b == 1 || attended_cap(dm, sparse) <= kRaggedKeys));
    for (int n = whole ? 1 : 2; n == 1 || (n <= limit && heads * nrb * n <= kMaxRecords); ++n) {
      const Fit& f = n == 1 ? kWhole[wide][mode] : kSplit[wide][mode];
      const long long rounds = (blocks * n + kComputeUnits - 1) / kComputeUnits, steps = (tiles + n - 1) / n;
      const float mb = (float)(heads * nrb * n) * (float)(dm.d + 2) * 128e-6f;
      const float us = f.fixed + f.step * (float)(rounds * steps) + f.round * (float)(rounds - 1) + f.per_mb * mb + f.per_split * (float)n +
                       (n > 4 ? f.beyond_four : 0.f);
      if (us < best_us) {
        best = AttnPlan{mode == 1, n};
        best_us = us;
      }
    }
  }
  return best;
}

// Both factors of the first bound grow with the chunk length, so shorter chunks of the same shape fit as well: a prompt's last
// chunk may be split where the others never are (heads * nrb beyond kMaxRecords / 2), with the same workspace.
size_t attn_bf16_ws_floats(const Dims& dm) {
  const long long nrb = (long long)dm.g * ((dm.C + 31) / 32), heads = (long long)dm.n_kv * dm.b;
  const long long most = heads * nrb * key_splits_limit(dm, false, kSub);
  return (size_t)(most < kMaxRecords ? most : kMaxRecords) * 32 * (dm.d + 2);
}

template <int D>
static hipError_t launch_d(const Dims& dm, const AttnArgs& a, hipStream_t st) {
  const AttnPlan p = attn_plan(dm, a.k_idx != nullptr);
  AttnArgs aa = a;
  aa.n_splits = p.n_splits;
  return p.split_tile ? launch_ds<D, true>(dm, aa, st) : launch_ds<D, false>(dm, aa, st);
}

void attn_bf16_plan(const Dims& dm, bool sparse, int32_t* row_blocks, int32_t* n_splits) {
  const AttnPlan p = attn_plan(dm, sparse);
  *row_blocks = p.split_tile ? 4 : 8;
  *n_splits = p.n_splits;
}

hipError_t launch_attn_bf16(const Dims& dm, const AttnArgs& a, float* part, hipStream_t st) {
  AttnArgs aa = a;
  aa.part = part;
  return dm.d == 64 ? launch_d<64>(dm, aa, st) : launch_d<128>(dm, aa, st);
}

}  // namespace quoka
