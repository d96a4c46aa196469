// Top-2 selection shared by the search kernels: the best value with its pool index and the runner-up's value.
#pragma once
#include <hip/hip_runtime.h>

namespace rc {
namespace {

__device__ __forceinline__ void top2_push(float v, int i, float& best, int& bidx, float& second) {
  const bool gt = v > best;
  second = gt ? best : fmaxf(second, v);
  bidx = gt ? i : bidx;
  best = gt ? v : best;
}

// Merge (b2, i2, s2) into (best, bidx, second): higher score wins, equal scores go to the lower index.
__device__ __forceinline__ void top2_merge(float& best, int& bidx, float& second, float b2, int i2, float s2) {
  const bool take = (b2 > best) || (b2 == best && (unsigned)i2 < (unsigned)bidx);
  const float loser = take ? best : b2;
  const float wsec = take ? s2 : second;
  bidx = take ? i2 : bidx;
  best = take ? b2 : best;
  second = fmaxf(wsec, loser);
}

}  // namespace
}  // namespace rc
