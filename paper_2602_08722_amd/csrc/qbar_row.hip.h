// One row of Qbar (Alg. 1 normalise and reshape / mean; Sec. 3.3), worked out by one wave: the r-th retained query of each
// head of the group, unit-normalised, and averaged.  Lanes own D/64 consecutive elements each.  The group's rows are all
// requested before any is used, so this pays one index latency and one row latency, not g of each.
#pragma once
#include <type_traits>

#include "common.hip.h"

namespace quoka {

// RULE: where the retained positions come from.  kFromIndex: q_idx as written by the selection kernel.  The other two
// are known in closed form, so q_idx is written here (`write_idx`) and no separate launch is needed: kIdentity keeps
// every query (C <= N_Q), kUniform takes the even stride floor(r * C / N') of the query-sampling baseline of Sec. 4.
// GU: heads requested at a time.  SIDE: their norms form side by side, without a branch a head, which is the faster as long as the chip is
// not full (query stage of one KV head of 16, d 128, 600 tokens 18.6 -> 15.8 us); in the scoring launch that forms Qbar itself, whose every
// block does this, groups of more than four go one head after the other (24 x 8 KV heads of 7, d 64, 8 tokens over 1500 keys, whole
// calls 36.2 / 37.4 us; one sequence 19.2 / 18.9).  The same bits.
enum { kFromIndex = 0, kIdentity = 1, kUniform = 2 };
// `first` (bf16): the rows of the group's first eight heads, as the caller has requested them.  A smaller group's last row is requested
// again for the places beyond it: a choice by the group's size stands ahead of the first fetch and costs more than the fetches (scoring
// launch of 8 heads of 4, 8192 keys, 1 token 9.3 -> 9.9 us; asked for a wave's later rows only, 1 token 9.25 -> 9.4, 13 x 8 heads, 8 tokens
// over 1500 keys 14.0 -> 13.7).
template <int D>
struct QbarRows {
  typedef typename std::conditional<D == 128, uint32_t, uint16_t>::type elems;   // a lane's D / 64 elements
  elems v[8];
  __device__ __forceinline__ void load(const Dims& dm, const uint16_t* q, int tok, int kv, int b, int lane) {
#pragma unroll
    for (int j = 0; j < 8; ++j)
      v[j] = *reinterpret_cast<const elems*>(q + b * dm.qs[0] + (size_t)(kv * dm.g + min(j, dm.g - 1)) * dm.qs[1] +
                                             (size_t)tok * dm.qs[2] + lane * (D / 64));
  }
  __device__ __forceinline__ float at(int j, int e) const {
    return __uint_as_float(e == 0 ? (uint32_t)v[j] << 16 : (uint32_t)v[j] & 0xFFFF0000u);
  }
};
template <typename T, int D, int RULE, int GU, bool SIDE>
__device__ __forceinline__ void qbar_row(const Dims& dm, const T* __restrict__ q, int32_t* __restrict__ q_idx, int n_keep,
                                         int r, int kv, int b, int lane, bool write_idx, float (&row)[D / 64],
                                         const QbarRows<D>* first = nullptr) {
  constexpr int EPL = D / 64;
  float acc[EPL];
#pragma unroll
  for (int e = 0; e < EPL; ++e) acc[e] = 0.f;
  // kFromIndex: lane j has the position in head j of the group (at most 16), in one vector load: as scalar loads they would be waited
  // for one by one
  int32_t* slot = q_idx + (size_t)(b * dm.n_q + kv * dm.g + min(lane, dm.g - 1)) * n_keep + r;
  int my_tok = RULE == kIdentity ? r : (int)(((int64_t)r * dm.chunk(b)) / n_keep);
  if constexpr (RULE == kFromIndex) {
    my_tok = *slot;
  } else {
    if (write_idx && lane < dm.g) *slot = my_tok;
  }
  for (int j0 = 0; j0 < dm.g; j0 += GU) {
    float v[GU][EPL], ss[GU];
#pragma unroll
    for (int jj = 0; jj < GU; ++jj) {
      const int j = min(j0 + jj, dm.g - 1);
      const int tok = RULE == kFromIndex ? __builtin_amdgcn_readlane(my_tok, j) : my_tok;
      const T* src = q + b * dm.qs[0] + (size_t)(kv * dm.g + j) * dm.qs[1] + (size_t)tok * dm.qs[2];
#pragma unroll
      for (int e = 0; e < EPL; ++e) {
        if (GU <= 8 && first != nullptr && j0 == 0) v[jj][e] = first->at(jj % 8, e);
        else v[jj][e] = Elem<T>::load1(src + lane * EPL + e);
      }
    }
    if constexpr (SIDE) {
      // (a row beyond the group is made zero, and adds zero; without normalisation (dot-product ablation) every norm is made one)
#pragma unroll
      for (int jj = 0; jj < GU; ++jj) {
        ss[jj] = 0.f;
#pragma unroll
        for (int e = 0; e < EPL; ++e) {
          v[jj][e] = j0 + jj < dm.g ? v[jj][e] : 0.f;
          ss[jj] += v[jj][e] * v[jj][e];
        }
      }
#pragma unroll
      for (int jj = 0; jj < GU; ++jj) ss[jj] = wave64_sum(ss[jj]);
#pragma unroll
      for (int jj = 0; jj < GU; ++jj) {
        const float nrm = fmaxf(sqrtf((dm.flags & 1) ? 1.0f : ss[jj]), kNormEps);
#pragma unroll
        for (int e = 0; e < EPL; ++e) acc[e] += v[jj][e] / nrm;   // heads are accumulated in ascending order
      }
    } else {
#pragma unroll
      for (int jj = 0; jj < GU; ++jj) {
        ss[jj] = 0.f;
#pragma unroll
        for (int e = 0; e < EPL; ++e) ss[jj] += v[jj][e] * v[jj][e];
        ss[jj] = wave64_sum(ss[jj]);
        const float nrm = (dm.flags & 1) ? 1.0f : fmaxf(sqrtf(ss[jj]), kNormEps);
        if (j0 + jj < dm.g) {   // wave-uniform
#pragma unroll
          for (int e = 0; e < EPL; ++e) acc[e] += v[jj][e] / nrm;
        }
      }
    }
  }
#pragma unroll
  for (int e = 0; e < EPL; ++e) row[e] = acc[e] / (float)dm.g;
}

}  // namespace quoka
