// How the workgroups of a layer share its table and its reference counts.  Plain C++, so that the arithmetic can be
// checked where there is no GPU.
#pragma once
#include <cstdint>

namespace rc {

constexpr int kGatherThreads = 1024;
constexpr int kGatherPerThread = 16;                                  // entries a thread keeps in flight
constexpr int kGatherBatch = kGatherThreads * kGatherPerThread;       // entries per batch of a workgroup

// Workgroups per layer.  One (which then also finalizes its layer) when the layers alone fill the chip or the
// layer's table is small; otherwise as many as keep the launch at one workgroup per compute unit, of at least
// a quarter batch each: a single compute unit takes longer to stream a large layer (with a launch that adds the
// workgroups' histograms, at 64 layers of 49 664 entries and 50 176 reference counts: 40 us with one workgroup per layer,
// 30 with 3, 26 with 4, 33 with 8).
inline int64_t chunks_per_layer(int64_t RE, int64_t L) {
  if (L >= 128) return 1;
  int64_t g = 256 / (L > 0 ? L : 1);
  const int64_t most = RE / (kGatherBatch / 4);
  if (g > most) g = most;
  if (g < 1) g = 1;
  if (g > 65535) g = 65535;
  return g;
}

// Items of a share where G workgroups share n of them, in fours (16 bytes).
inline int64_t share_length(int64_t n, int64_t G) { return ((n + G - 1) / G + 3) / 4 * 4; }

// Items of the share that starts at `first`, of n in all; none where it starts past the last one, which the rounding
// to fours does to the last workgroups of a long table over few blocks.
constexpr int share_items(int n, int first, int length) {
  return first >= n ? 0 : n - first < length ? n - first : length;
}

}  // namespace rc
