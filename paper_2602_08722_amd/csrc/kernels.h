// Internal launcher interface between the C-ABI layer (api.hip) and the kernel translation units.
#pragma once
#include <atomic>
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "common.hip.h"

namespace quoka {

// Sizes that every call is checked against, and that kernels count on
constexpr int kMaxGroup = 16;   // q-heads per KV head
constexpr int kMaxChunk = 8192;
constexpr int kMaxKv = 1 << 24;   // (cache lengths are below it)

// x / n as x * quotient_factor(n) >> 16.  The product is x / n + x * (n * factor - 2^16) / (n * 2^16) before the shift, so the quotient is
// right as long as x * (n * factor - 2^16) < 2^16, and the product fits 32 bits for x <= 2^16 - 1.
constexpr uint32_t quotient_factor(uint32_t n) { return (65536u + n - 1) / n; }
constexpr bool quotients_hold(uint32_t n_most, uint32_t x_most) {   // for every n up to n_most and x up to x_most
  for (uint32_t n = 1; n <= n_most; ++n)
    if (x_most * (n * quotient_factor(n) - 65536u) >= 65536u) return false;
  return x_most < 65536u;
}

// Kernels that use more than 64 KiB of dynamic LDS need the limit raised once per function and device.  `done` is a
// per-function bit mask over device ordinals (a function-local static of the caller); the attribute call is
// idempotent, so two threads racing through it are harmless, and the mask itself is atomic.
inline hipError_t ensure_dynamic_lds(const void* func, size_t bytes, std::atomic<uint64_t>& done) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  const uint64_t bit = dev >= 0 && dev < 64 ? (uint64_t{1} << dev) : 0;   // ordinals beyond 63: set it every time
  if (bit != 0 && (done.load(std::memory_order_acquire) & bit) != 0) return hipSuccess;
  e = hipFuncSetAttribute(func, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
  if (e != hipSuccess) return e;
  done.fetch_or(bit, std::memory_order_release);
  return hipSuccess;
}

// --- query sub-selection (select_queries.hip) -------------------------------------------------
size_t select_queries_ws_floats(const Dims& dm);
// `zero` / `zero_words`: optional side job for the fused call -- the last launch clears that many 32-bit words (what
// the key-selection stage that follows needs cleared).
hipError_t launch_select_queries(const Dims& dm, int dtype, const void* q, int32_t* q_idx, float* qbar, float* ws,
                                 hipStream_t st, uint32_t* zero = nullptr, size_t zero_words = 0,
                                 uint16_t* terms = nullptr);
// (`terms`: the last launch also leaves Qbar as the exact scorer's operands, TermsLayout of score_tile.hip.h; bf16)
size_t query_terms_bytes(const Dims& dm);
bool select_queries_one_block(const Dims& dm);   // which of its two routes (C > n_ret) the launch takes

// --- key scoring (score_keys.hip) ---------------------------------------------------------------
// `zero` / `zero_words`: optional side job for the fused call -- the scoring blocks clear that many 32-bit words (the
// histograms the multi-block top-k that follows would otherwise clear with a launch of its own).
// `fq` (where score_forms_qbar): the query stage has not run; the launch forms Qbar and q_idx itself.
struct FusedQbar {
  const void* q = nullptr;
  int32_t* q_idx = nullptr;
  float* qbar = nullptr;
};
bool score_forms_qbar(const Dims& dm, int dtype);
hipError_t launch_score_keys(const Dims& dm, int dtype, const float* qbar, const void* k_cache, const int32_t* kv_lens,
                             float* scores, hipStream_t st, uint32_t* zero = nullptr, size_t zero_words = 0,
                             const FusedQbar& fq = {}, const uint16_t* terms = nullptr);
bool score_reads_terms(const Dims& dm, int dtype);   // whether the launch would rather have `terms` than Qbar

// --- top-B key selection (topk_keys.hip) ----------------------------------------------------------
size_t topk_ws_words(const Dims& dm);
bool topk_uses_ws(const Dims& dm);   // whether a launch with these sizes takes the multi-block path
// `ws_is_zero`: the workspace words (topk_ws_words) have already been cleared on this stream.
hipError_t launch_topk_keys(const Dims& dm, const float* scores, const int32_t* kv_lens, const int32_t* budgets,
                            int32_t* k_idx, int32_t* k_cnt, uint32_t* ws, hipStream_t st, bool ws_is_zero = false);

// --- scoring + top-B as one stage for long caches (select_keys.hip) --------------------------------
// Provisional one-term scores, exact re-scoring of the keys near the cut, ordered emission: the same index lists as
// launch_score_keys followed by launch_topk_keys.  `ws_is_zero`: the first select_keys_zero_words words of the
// workspace have already been cleared on this stream.
hipError_t launch_score_stream(const Dims& dm, const float* qbar, const uint16_t* terms, const void* k_cache,
                               const int32_t* kv_lens, float* scores, uint32_t* hist_ws, hipStream_t st);
bool select_keys_two_pass_applies(const Dims& dm, int dtype);
// The same lists from exact scores and their histogram (launch_score_hist), which is the faster up to a size; `terms` as
// launch_select_queries leaves them, the workspace cleared as for launch_select_keys.
bool select_keys_exact_pays(const Dims& dm, int dtype);
hipError_t launch_score_hist(const Dims& dm, const float* qbar, const void* k_cache, const int32_t* kv_lens, float* scores,
                             hipStream_t st, const uint16_t* terms, uint32_t* hist_ws);
hipError_t launch_select_keys_exact(const Dims& dm, const float* qbar, const void* k_cache, const int32_t* kv_lens,
                                    const int32_t* budgets, float* scores, int32_t* k_idx, int32_t* k_cnt, uint32_t* ws,
                                    const uint16_t* terms, hipStream_t st);
size_t select_keys_ws_words(const Dims& dm);
size_t select_keys_zero_words(const Dims& dm, bool exact);   // (`exact`: for launch_select_keys_exact)
hipError_t launch_select_keys(const Dims& dm, const float* qbar, const void* k_cache, const int32_t* kv_lens,
                              const int32_t* budgets, float* scores, int32_t* k_idx, int32_t* k_cnt, uint32_t* ws,
                              hipStream_t st, bool ws_is_zero = false, const uint16_t* terms = nullptr);
// (`terms`, where select_keys_streams_exact: the streaming launch leaves exact scores and no key is scored again)
bool select_keys_streams_exact(const Dims& dm, int dtype);

// --- attention (attn_mfma.hip for bf16, attn_f32.hip for float32) ---------------------------------
// Cache rows attended: sparse (k_idx != nullptr): k_idx[b,kv,0..k_cnt[b,kv]); dense: 0..kv_lens[b].  The kernels cut
// the list at B_max (in a prompt the top-B launch has cut it at T_cap) and the length at T_max, which a dense launch has set
// to the T_cap that it is sized for: a merge adds up only partials that some block has written.
struct AttnArgs {
  const void *q, *k_cache, *v_cache, *k_chunk, *v_chunk;
  const int32_t* k_idx;    // nullptr for dense
  const int32_t* n_cache;  // k_cnt [b,n_kv] (sparse) or kv_lens [b] (dense)
  void* out;
  float* lse;              // may be nullptr
  // set by the launcher of the bf16 kernel:
  int adjacent = 0;        // row-block assignment (paired or adjacent)
  int n_splits = 1;        // blocks that share a row block's key list
  // quotient_factor of g and of n_splits
  uint32_t inv_g = 0, inv_splits = 0;
  float* part = nullptr;   // their partial results
};
// the most cache rows any sequence of the call attends
inline int attended_cap(const Dims& dm, bool sparse) { return sparse && dm.B_max < dm.T_cap ? dm.B_max : dm.T_cap; }
size_t attn_bf16_ws_floats(const Dims& dm);
hipError_t launch_attn_bf16(const Dims& dm, const AttnArgs& a, float* part, hipStream_t st);
void attn_bf16_plan(const Dims& dm, bool sparse, int32_t* row_blocks, int32_t* n_splits);   // what that launch would choose
// decode-sized chunks (g * C <= 32 query rows per KV head): split-KV kernel + merge, partials in `part`
bool attn_decode_applies(const Dims& dm);
size_t attn_decode_ws_floats(const Dims& dm);
hipError_t launch_attn_decode_bf16(const Dims& dm, const AttnArgs& a, float* part, hipStream_t st);
// (float32: partials of key-split blocks in `part`)
size_t attn_f32_ws_floats(const Dims& dm);
hipError_t launch_attn_f32(const Dims& dm, const AttnArgs& a, float* part, hipStream_t st);

// --- measurement aids (probes.hip) ------------------------------------------------------------------
hipError_t launch_probe_mfma(int blocks, int iters, float* sink, hipStream_t st);
hipError_t launch_probe_attn_mix(int blocks, int steps, float* sink, hipStream_t st);
hipError_t launch_probe_read(const void* src, size_t bytes, float* sink, hipStream_t st);

}  // namespace quoka
