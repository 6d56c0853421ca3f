// C-ABI layer of libquoka: argument validation, workspace carving, kernel dispatch.
// Nothing here allocates or synchronises; the only state kept is the per-device address of the library-owned
// scratch array of quoka_topk_keys_noalloc.
#include <hip/hip_runtime.h>

#include <atomic>

#include "kernels.h"
#include "quoka.h"

namespace {

using quoka::Dims;

using quoka::kMaxChunk;
using quoka::kMaxGroup;
using quoka::kMaxKv;

constexpr int kMaxRetain = 128;
constexpr size_t kAlign = 256;

size_t round_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

struct WsLayout {
  size_t select_off, select_bytes;
  size_t topk_off, topk_bytes;
  size_t sel_off, sel_bytes;
  size_t part_off, part_bytes;
  size_t terms_off, terms_bytes;
  size_t total;
};

quoka_status check_shape(const quoka_shape* s, Dims* dm) {
  if (s == nullptr) return QUOKA_EINVAL;
  if (s->batch < 1 || s->n_q_heads < 1 || s->n_kv_heads < 1 || s->chunk_len < 1 || s->n_retain < 1 ||
      s->max_kv_len < 0 || s->max_budget < 0 || (s->score_flags & ~(QUOKA_SCORE_DOT | QUOKA_SCORE_MEAN | QUOKA_SELECT_UNIFORM | QUOKA_SCORE_QBAR_BF16 |
                          QUOKA_ATTN_SCALE_F32)) != 0)
    return QUOKA_EINVAL;
  if (s->n_q_heads % s->n_kv_heads != 0) return QUOKA_EINVAL;
  if (s->max_budget > s->max_kv_len) return QUOKA_EINVAL;
  if (s->dtype != QUOKA_F32 && s->dtype != QUOKA_BF16) return QUOKA_EUNSUPPORTED;
  if (s->head_dim != 64 && s->head_dim != 128) return QUOKA_EUNSUPPORTED;
  if (s->n_retain > kMaxRetain || s->chunk_len > kMaxChunk || s->max_kv_len >= kMaxKv) return QUOKA_EUNSUPPORTED;
  if (s->n_q_heads / s->n_kv_heads > kMaxGroup) return QUOKA_EUNSUPPORTED;
  if ((long long)s->batch * s->n_q_heads > 65535 || s->batch > 65535) return QUOKA_EUNSUPPORTED;
  const int64_t* strides[4] = {s->q_stride, s->kv_stride, s->ck_stride, s->o_stride};
  for (const int64_t* st : strides) {
    for (int i = 0; i < 3; ++i)
      if (st[i] < 0 || st[i] % 8 != 0) return QUOKA_EINVAL;
    if (st[2] < s->head_dim) return QUOKA_EINVAL;
  }
  // kernels address the rows of one (batch, KV head) slice with 32-bit byte offsets
  const int es = s->dtype == QUOKA_BF16 ? 2 : 4;
  if ((unsigned long long)s->max_kv_len * (unsigned long long)s->kv_stride[2] * es >= (1ull << 32) ||
      (unsigned long long)s->chunk_len * (unsigned long long)s->ck_stride[2] * es >= (1ull << 32))
    return QUOKA_EUNSUPPORTED;
  dm->b = s->batch;
  dm->n_q = s->n_q_heads;
  dm->n_kv = s->n_kv_heads;
  dm->g = s->n_q_heads / s->n_kv_heads;
  dm->d = s->head_dim;
  dm->C = s->chunk_len;
  dm->T_max = dm->T_cap = s->max_kv_len;
  dm->n_ret = s->n_retain;
  dm->B_max = s->max_budget;
  dm->flags = s->score_flags;
  dm->ls = 1;
  dm->prompt_chunks = 0;
  dm->C_last = dm->C;
  for (int i = 0; i < 3; ++i) {
    dm->qs[i] = s->q_stride[i];
    dm->kvs[i] = s->kv_stride[i];
    dm->cks[i] = s->ck_stride[i];
    dm->os[i] = s->o_stride[i];
  }
  return QUOKA_OK;
}

// (`part`: partials of the key-split attention kernels)
WsLayout layout(const Dims& dm, int dtype) {
  WsLayout l;
  l.select_off = 0;
  l.select_bytes = round_up(quoka::select_queries_ws_floats(dm) * sizeof(float), kAlign);
  l.topk_off = l.select_off + l.select_bytes;
  l.topk_bytes = round_up(quoka::topk_ws_words(dm) * sizeof(uint32_t), kAlign);
  l.sel_off = l.topk_off + l.topk_bytes;
  l.sel_bytes = round_up(quoka::select_keys_ws_words(dm) * sizeof(uint32_t), kAlign);
  l.part_off = l.sel_off + l.sel_bytes;
  size_t part_floats = quoka::attn_f32_ws_floats(dm);
  if (dtype == QUOKA_BF16) {   // (a prompt's last chunk may be decode-sized when the others are not)
    const size_t decode = quoka::attn_decode_ws_floats(dm), prefill = quoka::attn_bf16_ws_floats(dm);
    part_floats = decode > prefill ? decode : prefill;
  }
  l.part_bytes = round_up(part_floats * sizeof(float), kAlign);
  l.terms_off = l.part_off + l.part_bytes;
  l.terms_bytes = dtype == QUOKA_BF16 ? round_up(quoka::query_terms_bytes(dm), kAlign) : 0;
  l.total = l.terms_off + l.terms_bytes;
  if (l.total == 0) l.total = kAlign;
  return l;
}

quoka_status check_ws(const WsLayout& l, const void* ws, size_t bytes) {
  if (ws == nullptr) return QUOKA_EINVAL;
  if (reinterpret_cast<uintptr_t>(ws) % kAlign != 0) return QUOKA_EWORKSPACE;
  if (bytes < l.total) return QUOKA_EWORKSPACE;
  return QUOKA_OK;
}

bool aligned16(const void* p) { return reinterpret_cast<uintptr_t>(p) % 16 == 0; }

quoka_status from_hip(hipError_t e) { return e == hipSuccess ? QUOKA_OK : QUOKA_EHIP; }

// What a call knows beyond its shape.
struct CallInfo {
  int kv_cap = kMaxKv;   // no cache length of this call exceeds it
  int len_stride = 1;    // entries between the cache lengths (budgets) of neighbouring batch entries
  int last_len = 0;      // tokens of the last batch entry where it is shorter than the others
  bool prompt_chunks = false;   // the batch entries are chunks of one prompt
  bool of_prompt = false;       // a chunk of a prompt, by itself or among others: leaves the same `scores` either way
  void apply(Dims* dm) const {
    dm->T_cap = kv_cap < dm->T_max ? kv_cap : dm->T_max;
    dm->ls = len_stride;
    dm->prompt_chunks = prompt_chunks;
    if (last_len > 0) dm->C_last = last_len;
  }
};

// ---- chunks of one prompt as the batch of one call ---------------------------------------------------------------
// A prompt's queries, keys and values all exist when quoka_prefill_attn is called, so neither the selection nor the
// attention of a chunk waits for an earlier chunk: `n` consecutive chunks of one sequence run as one batched call whose
// batch strides are chunk steps.  The intermediates of the chunks lie at the front of the workspace.
constexpr int kMaxGroupChunks = 64;                     // (the attention kernels rank up to 64 batch entries by length)
constexpr size_t kGroupBytes = size_t{256} << 20;       // workspace bound: by then the launches are long

quoka_shape group_shape(const quoka_shape& s, int n) {
  quoka_shape sh = s;
  sh.batch = n;
  sh.q_stride[0] = s.chunk_len * s.q_stride[2];
  sh.o_stride[0] = s.chunk_len * s.o_stride[2];
  for (int a = 0; a < 3; ++a) sh.ck_stride[a] = s.kv_stride[a];
  sh.ck_stride[0] = s.chunk_len * s.kv_stride[2];
  sh.kv_stride[0] = 0;
  return sh;
}

struct GroupLayout {
  size_t q_idx, qbar, scores, k_idx, k_cnt, rest, total;
};
GroupLayout group_layout(const quoka_shape& s, Dims dm, int n) {   // dm: dimensions of one chunk
  dm.b = n;
  const size_t n_keep = dm.n_ret < dm.C ? dm.n_ret : dm.C, heads = (size_t)n * dm.n_kv;
  GroupLayout l;
  l.q_idx = 0;
  l.qbar = l.q_idx + round_up((size_t)n * dm.n_q * n_keep * 4, kAlign);
  l.scores = l.qbar + round_up(heads * n_keep * dm.d * 4, kAlign);
  l.k_idx = l.scores + round_up(heads * dm.T_max * 4, kAlign);
  l.k_cnt = l.k_idx + round_up(heads * dm.B_max * 4 + 4, kAlign);
  l.rest = l.k_cnt + round_up(heads * 4, kAlign);
  l.total = l.rest + layout(dm, s.dtype).total;
  return l;
}

// Chunks that fit one group within `bytes` of workspace (at most n).
int group_chunks(const quoka_shape& s, const Dims& dm, int n, size_t bytes) {
  n = n < kMaxGroupChunks ? n : kMaxGroupChunks;
  const int most = 65535 / s.n_q_heads;
  n = n < most ? n : most;
  while (n > 1 && group_layout(s, dm, n).total > bytes) --n;
  return n;
}

// The last chunk's intermediates to where the caller expects them (one sequence).
struct LastChunk {
  const int32_t* q_idx;
  const float *qbar, *scores;
  const int32_t *k_idx, *k_cnt;
  int32_t* q_idx_out;
  float *qbar_out, *scores_out;
  int32_t *k_idx_out, *k_cnt_out;
  int n_kv, n_qidx, n_qbar, T, T_max, B_max;
};
__global__ void copy_last_chunk(LastChunk p) {
  const int i0 = blockIdx.x * blockDim.x + threadIdx.x, step = gridDim.x * blockDim.x, kv = blockIdx.y;
  if (kv == 0) {
    for (int i = i0; i < p.n_qidx; i += step) p.q_idx_out[i] = p.q_idx[i];
    for (int i = i0; i < p.n_qbar; i += step) p.qbar_out[i] = p.qbar[i];
  }
  const int n = p.k_cnt[kv];
  if (i0 == 0) p.k_cnt_out[kv] = n;
  for (int i = i0; i < min(n, p.B_max); i += step) p.k_idx_out[(size_t)kv * p.B_max + i] = p.k_idx[(size_t)kv * p.B_max + i];
  for (int i = i0; i < p.T; i += step) p.scores_out[(size_t)kv * p.T_max + i] = p.scores[(size_t)kv * p.T_max + i];
}

}  // namespace

// ---- entry point for callers that cannot allocate ------------------------------------------------------------
// The multi-block top-k's histograms, cut steps and per-tile counts in an array the library owns.  `scratch` is the
// host-side handle of the device array; its device address differs per GPU and is looked up once per device with
// that device current.  Host code below only ever uses the looked-up pointer.
namespace {
constexpr size_t kScratchWords = QUOKA_NOALLOC_SCRATCH_BYTES / sizeof(uint32_t);
constexpr int kMaxDevices = 64;
}  // namespace
static __device__ __align__(256) uint32_t scratch[kScratchWords];
static std::atomic<uint32_t*> g_scratch_ptr[kMaxDevices];

static hipError_t scratch_address(uint32_t** out) {
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  uint32_t* p = g_scratch_ptr[dev].load(std::memory_order_acquire);
  if (p == nullptr) {
    void* sym = nullptr;
    e = hipGetSymbolAddress(&sym, HIP_SYMBOL(scratch));   // this device's copy of the array
    if (e != hipSuccess) return e;
    if (sym == nullptr) return hipErrorInvalidSymbol;
    p = static_cast<uint32_t*>(sym);
    g_scratch_ptr[dev].store(p, std::memory_order_release);   // (two threads racing here store the same address)
  }
  *out = p;
  return hipSuccess;
}

extern "C" {

quoka_status quoka_workspace_bytes(const quoka_shape* shape, size_t* out_bytes) {
  Dims dm;
  quoka_status st = check_shape(shape, &dm);
  if (st != QUOKA_OK) return st;
  if (out_bytes == nullptr) return QUOKA_EINVAL;
  *out_bytes = layout(dm, shape->dtype).total;
  return QUOKA_OK;
}

quoka_status quoka_prefill_workspace_bytes(const quoka_shape* shape, size_t* out_bytes) {
  Dims dm;
  quoka_status st = check_shape(shape, &dm);
  if (st != QUOKA_OK) return st;
  if (out_bytes == nullptr) return QUOKA_EINVAL;
  size_t total = layout(dm, shape->dtype).total;
  const int n_chunks = (dm.T_max + dm.C - 1) / dm.C;
  const int n = group_chunks(*shape, dm, n_chunks, kGroupBytes);
  if (n > 1) {
    const size_t group = group_layout(*shape, dm, n).total;
    total = group > total ? group : total;
  }
  *out_bytes = total;
  return QUOKA_OK;
}

quoka_status quoka_select_queries(const quoka_shape* shape, const void* q, int32_t* q_idx, float* qbar,
                                  void* workspace, size_t workspace_bytes, void* stream) {
  Dims dm;
  quoka_status st = check_shape(shape, &dm);
  if (st != QUOKA_OK) return st;
  if (q == nullptr || q_idx == nullptr || qbar == nullptr) return QUOKA_EINVAL;
  if (!aligned16(q) || !aligned16(qbar)) return QUOKA_EINVAL;
  const WsLayout l = layout(dm, shape->dtype);
  st = check_ws(l, workspace, workspace_bytes);
  if (st != QUOKA_OK) return st;
  float* ws = reinterpret_cast<float*>(static_cast<char*>(workspace) + l.select_off);
  return from_hip(quoka::launch_select_queries(dm, shape->dtype, q, q_idx, qbar, ws, static_cast<hipStream_t>(stream)));
}

quoka_status quoka_score_keys(const quoka_shape* shape, const float* qbar, const void* k_cache,
                              const int32_t* kv_lens, float* scores, void* workspace, size_t workspace_bytes,
                              void* stream) {
  Dims dm;
  quoka_status st = check_shape(shape, &dm);
  if (st != QUOKA_OK) return st;
  if (qbar == nullptr || kv_lens == nullptr) return QUOKA_EINVAL;
  if (dm.T_max > 0 && (k_cache == nullptr || scores == nullptr)) return QUOKA_EINVAL;
  if (!aligned16(qbar) || !aligned16(k_cache)) return QUOKA_EINVAL;
  st = check_ws(layout(dm, shape->dtype), workspace, workspace_bytes);
  if (st != QUOKA_OK) return st;
  return from_hip(
      quoka::launch_score_keys(dm, shape->dtype, qbar, k_cache, kv_lens, scores, static_cast<hipStream_t>(stream)));
}

quoka_status quoka_topk_keys(const quoka_shape* shape, const float* scores, const int32_t* kv_lens,
                             const int32_t* budgets, int32_t* k_idx, int32_t* k_cnt, void* workspace,
                             size_t workspace_bytes, void* stream) {
  Dims dm;
  quoka_status st = check_shape(shape, &dm);
  if (st != QUOKA_OK) return st;
  if (kv_lens == nullptr || budgets == nullptr || k_cnt == nullptr) return QUOKA_EINVAL;
  if (dm.T_max > 0 && scores == nullptr) return QUOKA_EINVAL;
  if (dm.B_max > 0 && k_idx == nullptr) return QUOKA_EINVAL;
  const WsLayout l = layout(dm, shape->dtype);
  st = check_ws(l, workspace, workspace_bytes);
  if (st != QUOKA_OK) return st;
  uint32_t* ws = reinterpret_cast<uint32_t*>(static_cast<char*>(workspace) + l.topk_off);
  return from_hip(
      quoka::launch_topk_keys(dm, scores, kv_lens, budgets, k_idx, k_cnt, ws, static_cast<hipStream_t>(stream)));
}

static quoka_status attn_common(const quoka_shape* shape, const CallInfo& info, const void* q, const void* k_cache,
                                const void* v_cache, const int32_t* k_idx, const int32_t* n_cache, bool sparse,
                                const void* k_chunk, const void* v_chunk, void* out, float* lse, void* workspace,
                                size_t workspace_bytes, void* stream) {
  Dims dm;
  quoka_status st = check_shape(shape, &dm);
  if (st != QUOKA_OK) return st;
  info.apply(&dm);
  if (q == nullptr || k_chunk == nullptr || v_chunk == nullptr || out == nullptr || n_cache == nullptr)
    return QUOKA_EINVAL;
  const bool has_cache = sparse ? dm.B_max > 0 : dm.T_max > 0;
  if (has_cache && (k_cache == nullptr || v_cache == nullptr)) return QUOKA_EINVAL;
  if (sparse && dm.B_max > 0 && k_idx == nullptr) return QUOKA_EINVAL;
  if (!aligned16(q) || !aligned16(k_cache) || !aligned16(v_cache) || !aligned16(k_chunk) || !aligned16(v_chunk) ||
      !aligned16(out))
    return QUOKA_EINVAL;
  const WsLayout l = layout(dm, shape->dtype);
  st = check_ws(l, workspace, workspace_bytes);
  if (st != QUOKA_OK) return st;
  quoka::AttnArgs a;
  a.q = q;
  a.k_cache = k_cache;
  a.v_cache = v_cache;
  a.k_chunk = k_chunk;
  a.v_chunk = v_chunk;
  if (!sparse) dm.T_max = dm.T_cap;   // what the kernels cut a cache length at: the launch is sized for that
  // A null k_idx selects the dense kernel path, so a sparse call with B_max == 0 still needs a non-null one: n_cache, not the
  // caller's pointer to an array without entries, because the kernels fetch entry 0 before they know a list's length (and do not use it).
  a.k_idx = !sparse ? nullptr : dm.B_max > 0 ? k_idx : n_cache;
  a.n_cache = n_cache;
  a.out = out;
  a.lse = lse;
  hipStream_t hs = static_cast<hipStream_t>(stream);
  float* part = reinterpret_cast<float*>(static_cast<char*>(workspace) + l.part_off);
  if (shape->dtype != QUOKA_BF16) return from_hip(quoka::launch_attn_f32(dm, a, part, hs));
  if (quoka::attn_decode_applies(dm)) return from_hip(quoka::launch_attn_decode_bf16(dm, a, part, hs));
  return from_hip(quoka::launch_attn_bf16(dm, a, part, hs));
}

quoka_status quoka_sparse_attn(const quoka_shape* shape, const void* q, const void* k_cache, const void* v_cache,
                               const int32_t* k_idx, const int32_t* k_cnt, const void* k_chunk,
                               const void* v_chunk, void* out, float* lse, void* workspace,
                               size_t workspace_bytes, void* stream) {
  return attn_common(shape, CallInfo{}, q, k_cache, v_cache, k_idx, k_cnt, true, k_chunk, v_chunk, out, lse, workspace,
                     workspace_bytes, stream);
}

quoka_status quoka_dense_attn(const quoka_shape* shape, const void* q, const void* k_cache, const void* v_cache,
                              const int32_t* kv_lens, const void* k_chunk, const void* v_chunk, void* out,
                              float* lse, void* workspace, size_t workspace_bytes, void* stream) {
  return attn_common(shape, CallInfo{}, q, k_cache, v_cache, nullptr, kv_lens, false, k_chunk, v_chunk, out, lse, workspace,
                     workspace_bytes, stream);
}

// Scoring and top-B of one chunk on `stream`: the two-pass stage where it applies, else the two separate launches
// (whose scoring launch clears the multi-block top-k's histograms).
static quoka_status select_keys_common(const Dims& dm, int dtype, const float* qbar, const void* k_cache,
                                       const int32_t* kv_lens, const int32_t* budgets, float* scores, int32_t* k_idx,
                                       int32_t* k_cnt, void* workspace, const WsLayout& l, hipStream_t hs,
                                       bool sel_ws_is_zero, const quoka::FusedQbar& fq = {},
                                       const uint16_t* terms = nullptr, bool exact = false) {
  if (dm.T_max > 0 && quoka::select_keys_two_pass_applies(dm, dtype)) {
    uint32_t* sel_ws = reinterpret_cast<uint32_t*>(static_cast<char*>(workspace) + l.sel_off);
    if (exact)
      return from_hip(quoka::launch_select_keys_exact(dm, qbar, k_cache, kv_lens, budgets, scores, k_idx, k_cnt, sel_ws, terms,
                                                      hs));
    return from_hip(quoka::launch_select_keys(dm, qbar, k_cache, kv_lens, budgets, scores, k_idx, k_cnt, sel_ws, hs,
                                              sel_ws_is_zero, terms));
  }
  uint32_t* topk_ws = reinterpret_cast<uint32_t*>(static_cast<char*>(workspace) + l.topk_off);
  const bool fuse_clear = quoka::topk_uses_ws(dm);
  const size_t topk_words = fuse_clear ? quoka::topk_ws_words(dm) : 0;
  quoka_status st = from_hip(quoka::launch_score_keys(dm, dtype, qbar, k_cache, kv_lens, scores, hs,
                                                      fuse_clear ? topk_ws : nullptr, topk_words, fq, terms));
  if (st != QUOKA_OK) return st;
  return from_hip(quoka::launch_topk_keys(dm, scores, kv_lens, budgets, k_idx, k_cnt, topk_ws, hs, fuse_clear));
}

quoka_status quoka_select_keys(const quoka_shape* shape, const float* qbar, const void* k_cache,
                               const int32_t* kv_lens, const int32_t* budgets, float* scores, int32_t* k_idx,
                               int32_t* k_cnt, void* workspace, size_t workspace_bytes, void* stream) {
  Dims dm;
  quoka_status st = check_shape(shape, &dm);
  if (st != QUOKA_OK) return st;
  if (qbar == nullptr || kv_lens == nullptr || budgets == nullptr || k_cnt == nullptr) return QUOKA_EINVAL;
  if (dm.T_max > 0 && (k_cache == nullptr || scores == nullptr)) return QUOKA_EINVAL;
  if (dm.B_max > 0 && k_idx == nullptr) return QUOKA_EINVAL;
  if (!aligned16(qbar) || !aligned16(k_cache)) return QUOKA_EINVAL;
  const WsLayout l = layout(dm, shape->dtype);
  st = check_ws(l, workspace, workspace_bytes);
  if (st != QUOKA_OK) return st;
  return select_keys_common(dm, shape->dtype, qbar, k_cache, kv_lens, budgets, scores, k_idx, k_cnt, workspace, l,
                            static_cast<hipStream_t>(stream), false);
}

static quoka_status chunk_common(const quoka_shape* shape, const CallInfo& info, const void* q, const void* k_cache,
                                 const void* v_cache, const int32_t* kv_lens, const int32_t* budgets,
                                 const void* k_chunk, const void* v_chunk, int32_t* q_idx, float* qbar, float* scores,
                                 int32_t* k_idx, int32_t* k_cnt, void* out, float* lse, void* workspace,
                                 size_t workspace_bytes, void* stream) {
  // The stages as in quoka_select_queries / quoka_select_keys (same checks), except that the last launch of the query
  // stage also clears the histograms and counters of the two-pass key selection, which saves that stage a launch.
  Dims dm;
  quoka_status st = check_shape(shape, &dm);
  if (st != QUOKA_OK) return st;
  info.apply(&dm);
  if (q == nullptr || q_idx == nullptr || qbar == nullptr) return QUOKA_EINVAL;
  if (kv_lens == nullptr || budgets == nullptr || k_cnt == nullptr) return QUOKA_EINVAL;
  if (dm.T_max > 0 && (k_cache == nullptr || scores == nullptr)) return QUOKA_EINVAL;
  if (dm.B_max > 0 && k_idx == nullptr) return QUOKA_EINVAL;
  if (!aligned16(q) || !aligned16(qbar) || !aligned16(k_cache)) return QUOKA_EINVAL;
  const WsLayout l = layout(dm, shape->dtype);
  st = check_ws(l, workspace, workspace_bytes);
  if (st != QUOKA_OK) return st;
  hipStream_t hs = static_cast<hipStream_t>(stream);
  const bool two_pass = dm.T_max > 0 && quoka::select_keys_two_pass_applies(dm, shape->dtype);
  // (the same lists, either way)
  const bool streams_exact = two_pass && !info.of_prompt && quoka::select_keys_streams_exact(dm, shape->dtype);
  const bool exact = two_pass && !info.of_prompt && !streams_exact && quoka::select_keys_exact_pays(dm, shape->dtype);
  uint32_t* sel_ws = reinterpret_cast<uint32_t*>(static_cast<char*>(workspace) + l.sel_off);
  float* sq_ws = reinterpret_cast<float*>(static_cast<char*>(workspace) + l.select_off);
  quoka::FusedQbar fq;
  uint16_t* terms = (!two_pass || exact || streams_exact) && quoka::score_reads_terms(dm, shape->dtype)
                        ? reinterpret_cast<uint16_t*>(static_cast<char*>(workspace) + l.terms_off)
                        : nullptr;
  if (!two_pass && quoka::score_forms_qbar(dm, shape->dtype)) {   // a few tokens: one launch less
    fq = quoka::FusedQbar{q, q_idx, qbar};
  } else {
    st = from_hip(quoka::launch_select_queries(dm, shape->dtype, q, q_idx, qbar, sq_ws, hs, two_pass ? sel_ws : nullptr,
                                               two_pass ? quoka::select_keys_zero_words(dm, exact) : 0, terms));
    if (st != QUOKA_OK) return st;
  }
  st = select_keys_common(dm, shape->dtype, qbar, k_cache, kv_lens, budgets, scores, k_idx, k_cnt, workspace, l, hs,
                          two_pass, fq, terms, exact);
  if (st != QUOKA_OK) return st;
  return attn_common(shape, info, q, k_cache, v_cache, k_idx, k_cnt, true, k_chunk, v_chunk, out, lse, workspace,
                     workspace_bytes, stream);
}

quoka_status quoka_chunk_attn(const quoka_shape* shape, const void* q, const void* k_cache, const void* v_cache,
                              const int32_t* kv_lens, const int32_t* budgets, const void* k_chunk,
                              const void* v_chunk, int32_t* q_idx, float* qbar, float* scores, int32_t* k_idx,
                              int32_t* k_cnt, void* out, float* lse, void* workspace, size_t workspace_bytes,
                              void* stream) {
  return chunk_common(shape, CallInfo{}, q, k_cache, v_cache, kv_lens, budgets, k_chunk, v_chunk, q_idx, qbar, scores, k_idx,
                      k_cnt, out, lse, workspace, workspace_bytes, stream);
}

quoka_status quoka_prefill_attn(const quoka_shape* shape, int sparse, const void* q, const void* k, const void* v,
                                const int32_t* kv_lens_all, const int32_t* budgets_all, int32_t* q_idx, float* qbar,
                                float* scores, int32_t* k_idx, int32_t* k_cnt, void* out, void* workspace,
                                size_t workspace_bytes, void* stream) {
  Dims dm;
  quoka_status st = check_shape(shape, &dm);
  if (st != QUOKA_OK) return st;
  if (q == nullptr || k == nullptr || v == nullptr || out == nullptr || kv_lens_all == nullptr) return QUOKA_EINVAL;
  if (sparse) {   // what the first chunk does not need but a later one does
    if (budgets_all == nullptr || q_idx == nullptr || qbar == nullptr || scores == nullptr || k_cnt == nullptr)
      return QUOKA_EINVAL;
    if ((dm.B_max > 0 && k_idx == nullptr) || !aligned16(qbar)) return QUOKA_EINVAL;
  }
  const int L = shape->max_kv_len, C = shape->chunk_len;
  if (L < 1) return QUOKA_EINVAL;
  const size_t es = shape->dtype == QUOKA_BF16 ? 2 : 4;
  const int n_chunks = (L + C - 1) / C;

  // Groups of chunks per sequence, where that takes at most three quarters (dense: three fifths) of the calls of chunk after
  // chunk of the whole batch: beyond, the batch fills a launch as well, with chunks of one length.  (Grouped against chunk
  // after chunk, 8 sequences of 5000 in chunks of 500, 32/8 heads, d 64, sparse 707 / 621 us; 8 of 3214 in chunks of 333,
  // 8/8 heads, dense 458 / 357.  220 measured batches: 0.6 of the time and less up to a third of the calls, 0.8 up to three
  // fifths, 0.85 up to three quarters, 0.99 above.)
  // 32/8 heads, d 128, 16000 tokens in chunks of 1024: 106 launches, 1197 us -> 8 launches, 573 us: the short launches
  // of the selection run once, and the attention blocks of all chunks fill the chip together.  (Batches: 2 sequences of
  // 16000 1777 -> 1099 us, 8 of them 5125 -> 4389, 8 of 20000 in chunks of 500, 8/2 heads 3844 -> 2104.)  A short last chunk goes
  // along where it selects as many queries as the others (up to n_retain tokens it keeps all, in position order) and its results do not
  // depend on that: a decode-sized one is attended by attn_decode_bf16, which rounds Q no second time, and the query stage's
  // form for batches rounds the mean differently.  (Its one-block form for short chunks forms the tiled kernels' very sums.)
  const int last_len = L - (n_chunks - 1) * C;
  Dims last = dm;   // the last chunk by itself
  last.C = last.C_last = last_len;
  const int keep = dm.n_ret < C ? dm.n_ret : C;
  const bool last_along =
      last_len == C || (shape->dtype == QUOKA_BF16 && !quoka::attn_decode_applies(last) && last_len > dm.n_ret &&
                        quoka::select_queries_one_block(last) == quoka::select_queries_one_block(dm));
  const int n_grouped = last_along ? n_chunks : n_chunks - 1;
  const int most = group_chunks(*shape, dm, n_grouped, workspace_bytes);
  const int n_groups = n_grouped > 0 ? (n_grouped + most - 1) / most : 0;
  int done = 0;   // chunks enqueued
  if (workspace != nullptr && reinterpret_cast<uintptr_t>(workspace) % kAlign == 0 && most > 1 &&
      (sparse ? 4LL : 5LL) * n_groups * shape->batch <= 3LL * n_grouped) {
    const int per_group = (n_grouped + n_groups - 1) / n_groups;
    char* ws = static_cast<char*>(workspace);
    for (int s = 0; s < shape->batch; ++s) {
      for (int i0 = 0; i0 < n_grouped; i0 += per_group) {
        const int n = i0 + per_group < n_grouped ? per_group : n_grouped - i0;
        const quoka_shape sh = group_shape(*shape, n);
        const GroupLayout gl = group_layout(*shape, dm, n);
        CallInfo info;
        info.kv_cap = (i0 + n - 1) * C;
        info.len_stride = shape->batch;
        info.prompt_chunks = info.of_prompt = true;
        const bool holds_last = i0 + n == n_chunks;
        if (holds_last) info.last_len = last_len;
        const size_t first = (size_t)i0 * C;
        const char* qi = static_cast<const char*>(q) + (s * shape->q_stride[0] + first * shape->q_stride[2]) * es;
        const char* kc = static_cast<const char*>(k) + s * shape->kv_stride[0] * es;
        const char* vc = static_cast<const char*>(v) + s * shape->kv_stride[0] * es;
        const char* ki = kc + first * shape->kv_stride[2] * es;
        const char* vi = vc + first * shape->kv_stride[2] * es;
        char* oi = static_cast<char*>(out) + (s * shape->o_stride[0] + first * shape->o_stride[2]) * es;
        const int32_t* lens = kv_lens_all + first / C * shape->batch + s;
        char* rest = ws + gl.rest;
        const size_t rest_bytes = workspace_bytes - gl.rest;
        if (!sparse) {
          st = attn_common(&sh, info, qi, kc, vc, nullptr, lens, false, ki, vi, oi, nullptr, rest, rest_bytes, stream);
          if (st != QUOKA_OK) return st;
          continue;
        }
        int32_t *g_q_idx = reinterpret_cast<int32_t*>(ws + gl.q_idx), *g_k_idx = reinterpret_cast<int32_t*>(ws + gl.k_idx),
                *g_k_cnt = reinterpret_cast<int32_t*>(ws + gl.k_cnt);
        float *g_qbar = reinterpret_cast<float*>(ws + gl.qbar), *g_scores = reinterpret_cast<float*>(ws + gl.scores);
        st = chunk_common(&sh, info, qi, kc, vc, lens, budgets_all + first / C * shape->batch + s, ki, vi, g_q_idx,
                          g_qbar, g_scores, g_k_idx, g_k_cnt, oi, nullptr, rest, rest_bytes, stream);
        if (st != QUOKA_OK) return st;
        if (holds_last) {
          LastChunk p;
          const size_t at = n - 1, heads = at * dm.n_kv, heads_out = (size_t)s * dm.n_kv;
          p.n_kv = dm.n_kv;
          p.n_qidx = dm.n_q * keep;
          p.n_qbar = dm.n_kv * keep * dm.d;
          p.T = info.kv_cap;
          p.T_max = dm.T_max;
          p.B_max = dm.B_max;
          p.q_idx = g_q_idx + at * p.n_qidx;
          p.q_idx_out = q_idx + (size_t)s * p.n_qidx;
          p.qbar = g_qbar + at * p.n_qbar;
          p.qbar_out = qbar + (size_t)s * p.n_qbar;
          p.scores = g_scores + heads * dm.T_max;
          p.scores_out = scores + heads_out * dm.T_max;
          p.k_idx = g_k_idx + heads * dm.B_max;
          p.k_idx_out = k_idx + heads_out * dm.B_max;
          p.k_cnt = g_k_cnt + heads;
          p.k_cnt_out = k_cnt + heads_out;
          hipLaunchKernelGGL(copy_last_chunk, dim3(32, dm.n_kv), dim3(256), 0, static_cast<hipStream_t>(stream), p);
          st = from_hip(hipGetLastError());
          if (st != QUOKA_OK) return st;
        }
      }
    }
    done = n_grouped;
  }

  for (int i = done; i < n_chunks; ++i) {
    quoka_shape sh = *shape;
    sh.chunk_len = (i + 1) * C <= L ? C : L - i * C;   // the last chunk may be short
    for (int a = 0; a < 3; ++a) sh.ck_stride[a] = shape->kv_stride[a];
    const size_t tok = (size_t)i * C;
    const char* qi = static_cast<const char*>(q) + tok * shape->q_stride[2] * es;
    const char* ki = static_cast<const char*>(k) + tok * shape->kv_stride[2] * es;
    const char* vi = static_cast<const char*>(v) + tok * shape->kv_stride[2] * es;
    char* oi = static_cast<char*>(out) + tok * shape->o_stride[2] * es;
    const int32_t* lens = kv_lens_all + (size_t)i * shape->batch;
    // Chunk i's cache holds i * C rows: launches are sized for that, not for the prompt (16 chunks of 1024: 1307 ->
    // 1222 us).  The first chunk has no cache to select from, and only the last chunk's intermediates are the caller's.
    CallInfo info;
    info.kv_cap = i * C;
    info.of_prompt = true;
    if (sparse && (i > 0 || n_chunks == 1)) {
      st = chunk_common(&sh, info, qi, k, v, lens, budgets_all + (size_t)i * shape->batch, ki, vi, q_idx, qbar, scores,
                        k_idx, k_cnt, oi, nullptr, workspace, workspace_bytes, stream);
    } else {
      st = attn_common(&sh, info, qi, k, v, nullptr, lens, false, ki, vi, oi, nullptr, workspace, workspace_bytes, stream);
    }
    if (st != QUOKA_OK) return st;
  }
  return QUOKA_OK;
}

quoka_status quoka_topk_keys_noalloc(const quoka_shape* shape, const float* scores, const int32_t* kv_lens,
                                     const int32_t* budgets, int32_t* k_idx, int32_t* k_cnt, void* stream) {
  Dims dm;
  quoka_status st = check_shape(shape, &dm);
  if (st != QUOKA_OK) return st;
  if (kv_lens == nullptr || budgets == nullptr || k_cnt == nullptr) return QUOKA_EINVAL;
  if (dm.T_max > 0 && scores == nullptr) return QUOKA_EINVAL;
  if (dm.B_max > 0 && k_idx == nullptr) return QUOKA_EINVAL;
  if (quoka::topk_ws_words(dm) > kScratchWords) return QUOKA_EWORKSPACE;
  uint32_t* ws = nullptr;
  if (scratch_address(&ws) != hipSuccess) return QUOKA_EHIP;
  // the launcher clears the words it uses with a fill kernel of its own (no memset node, nothing allocated)
  return from_hip(
      quoka::launch_topk_keys(dm, scores, kv_lens, budgets, k_idx, k_cnt, ws, static_cast<hipStream_t>(stream)));
}

quoka_status quoka_probe_mfma(int blocks, int iters, float* sink, void* stream) {
  if (blocks < 1 || blocks > 65535 || iters < 1 || sink == nullptr) return QUOKA_EINVAL;
  return from_hip(quoka::launch_probe_mfma(blocks, iters, sink, static_cast<hipStream_t>(stream)));
}

quoka_status quoka_probe_attn_plan(const quoka_shape* shape, int sparse, int32_t* row_blocks, int32_t* n_splits) {
  Dims dm;
  const quoka_status st = check_shape(shape, &dm);
  if (st != QUOKA_OK) return st;
  if (row_blocks == nullptr || n_splits == nullptr) return QUOKA_EINVAL;
  *row_blocks = *n_splits = 0;
  if (shape->dtype == QUOKA_BF16 && !quoka::attn_decode_applies(dm)) quoka::attn_bf16_plan(dm, sparse != 0, row_blocks, n_splits);
  return QUOKA_OK;
}

quoka_status quoka_probe_attn_mix(int blocks, int steps, float* sink, void* stream) {
  if (blocks < 1 || blocks > 65535 || steps < 1 || sink == nullptr) return QUOKA_EINVAL;
  return from_hip(quoka::launch_probe_attn_mix(blocks, steps, sink, static_cast<hipStream_t>(stream)));
}

quoka_status quoka_probe_read(const void* src, size_t bytes, float* sink, void* stream) {
  if (src == nullptr || sink == nullptr || bytes == 0 || bytes % 16 != 0 || !aligned16(src)) return QUOKA_EINVAL;
  return from_hip(quoka::launch_probe_read(src, bytes, sink, static_cast<hipStream_t>(stream)));
}

const char* quoka_status_string(quoka_status status) {
  switch (status) {
    case QUOKA_OK: return "ok";
    case QUOKA_EINVAL: return "invalid argument";
    case QUOKA_EUNSUPPORTED: return "unsupported shape or dtype";
    case QUOKA_EWORKSPACE: return "workspace too small or misaligned";
    case QUOKA_EHIP: return "HIP launch failed";
  }
  return "unknown status";
}

int quoka_version(void) { return 100; }

}  // extern "C"
