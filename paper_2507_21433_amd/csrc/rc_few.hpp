// Search of a small problem with few queries: the plan, and the two launches that carry it out (rc_few.hip).
#pragma once
#include <cstddef>
#include <cstdint>

#include "rc.h"

namespace rc {

constexpr int kFewRows = 64;      // pool blocks of a workgroup
constexpr int kFewQueries = 64;   // most query blocks

// Shares per tile of 64 pool blocks (half of them on the K tensor, half on V), 0 = not a problem for these kernels.
int few_shares(bool layer_mean, int64_t L, int64_t P, int64_t Q, int T, int H);

// workspace of S shares: a row of floats per share and query
inline size_t few_bytes(int S, int64_t L, int64_t P, int64_t Q) {
  return (size_t)L * (size_t)S * (size_t)Q * (size_t)((P + kFewRows - 1) / kFewRows * kFewRows) * sizeof(float);
}

struct FewArgs {
  const rc_kv_desc *qdesc, *pdesc;
  const void *kq, *vq, *kp, *vp;
  int64_t Q, P;
  const float *q_ksq, *q_vsq, *p_ksq, *p_vsq;
  const uint8_t* live;   // [L][P], or [P] for the layer mean
  float threshold;       // tau, or the largest distance that matches
  int32_t* best_idx;
  float* best_value;
  int32_t* match_idx;
  float* second_value;
  void* workspace;
  void* hip_stream;
};
// layer_mean: the layer-mean distance and one decision per query, else the cosine per layer
rc_status few_search(const FewArgs& a, int S, bool layer_mean, const char* who);

// The per-head score (one share per head): whether a call comes here, and the call.
bool few_heads(int64_t L, int64_t P, int64_t Q, int T, int H);
rc_status few_search_heads(const FewArgs& a, const char* who);

}  // namespace rc
