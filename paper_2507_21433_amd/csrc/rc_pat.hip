// rc_pat_threshold, rc_apply_threshold: percentile-based adaptive thresholding (ReasonCache
// Sec. IV-A, PAT).  The threshold is the nearest-rank p-th percentile of the distances collected
// during warm-up: an exact order statistic, found by a radix select over the bit patterns, most
// significant bits first (three passes of 11, 11 and 10 bits; four of 8 in a workspace of 4 KB or
// for few samples).  Each pass histograms the next bits of the keys that still match the prefix
// chosen so far; the next pass derives that prefix again from the histograms (every workgroup
// repeats the short scan), so no pass needs a launch of its own for the scan.  Integer counts only: the result is the same on every run.
#include <hip/hip_runtime.h>

#include "rc_common.hpp"

namespace rc {
namespace {

constexpr int kPatThreads = 256;

struct PatState {
  unsigned int hist[4][256];
  unsigned int nonfinite;
  unsigned int pad[3];
};

// Order-preserving map float -> unsigned; every non-finite value becomes the largest key.
__device__ __forceinline__ unsigned int key_of(float x) {
  const unsigned int b = __float_as_uint(x);
  const bool finite = (b & 0x7f800000u) != 0x7f800000u;
  const unsigned int k = (b & 0x80000000u) ? ~b : (b | 0x80000000u);
  return finite ? k : 0xffffffffu;
}

__device__ __forceinline__ float value_of(unsigned int k) {
  return __uint_as_float((k & 0x80000000u) ? (k & 0x7fffffffu) : ~k);
}

__global__ __launch_bounds__(kPatThreads) void pat_clear_kernel(PatState* st) {
  unsigned int* w = reinterpret_cast<unsigned int*>(st);
  for (int i = threadIdx.x; i < (int)(sizeof(PatState) / 4); i += kPatThreads) w[i] = 0u;
}

// Rank of the percentile among the n_f finite samples: ceil(p/100 * n_f) in double, within [1, n_f].
__device__ __forceinline__ long long pat_rank(double p, long long n_f) {
  long long k = (long long)ceil(p * (double)n_f / 100.0);
  if (k < 1) k = 1;
  if (k > n_f) k = n_f;
  return k;
}

// Exclusive prefix sum of one value per thread over the 256 threads of the workgroup.
__device__ __forceinline__ long long scan256(long long v, long long* s_wave /* [4] */) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  long long incl = v;
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const long long n = __shfl_up(incl, off);
    if (lane >= off) incl += n;
  }
  __syncthreads();  // s_wave may still be read from the previous call
  if (lane == 63) s_wave[wave] = incl;
  __syncthreads();
  long long before = 0;
#pragma unroll
  for (int w = 0; w < 4; ++w) before += (w < wave) ? s_wave[w] : 0;
  return before + incl - v;
}

// The bytes fixed by passes 0 .. npass-1 (s_h holds their histograms): in every pass the digit
// whose bin contains rank k, found by all 256 threads together (thread d owns bin d).
// Returns the prefix to every thread.  s_sel: two words of scratch.
__device__ __forceinline__ unsigned int pat_prefix(const unsigned int (*s_h)[256], int npass, long long k,
                                                   long long* s_wave, long long* s_sel) {
  unsigned int prefix = 0;
  for (int j = 0; j < npass; ++j) {
    const long long c = s_h[j][threadIdx.x];
    const long long before = scan256(c, s_wave);
    if (threadIdx.x == 0) s_sel[0] = -1;
    __syncthreads();
    if (c > 0 && before < k && k <= before + c) {  // exactly one bin, if k is within the total
      s_sel[0] = threadIdx.x;
      s_sel[1] = before;
    }
    __syncthreads();
    const long long digit = s_sel[0] < 0 ? 255 : s_sel[0];
    k -= s_sel[0] < 0 ? 0 : s_sel[1];
    prefix |= (unsigned int)digit << (24 - 8 * j);
    __syncthreads();
  }
  return prefix;
}

// One more key in bin `bin` (-1: none of this lane's).  Distances come in a cluster or two, so most lanes of a wave
// hit one or two bins, and LDS adds to one word are done one after the other: the bins of the first two lanes
// that are left go out as one add each, the rest as they are.
__device__ __forceinline__ void count_bin(unsigned int* h, int bin) {
#pragma unroll
  for (int round = 0; round < 2; ++round) {
    const unsigned long long active = __ballot(bin >= 0);
    if (active == 0) return;  // the same for the whole wave
    const int leader = __ffsll((long long)active) - 1;
    const int theirs = __shfl(bin, leader);
    const unsigned long long same = __ballot(bin == theirs);
    if ((int)(threadIdx.x & 63) == leader) atomicAdd(&h[theirs], (unsigned int)__popcll(same));
    if (bin == theirs) bin = -1;
  }
  if (bin >= 0) atomicAdd(&h[bin], 1u);
}

// Few samples: one workgroup keeps their keys in registers and does all four passes; one launch instead of six
// (3 to 6 us each).  2000 samples 23 -> 8.5 us, 8000 32 -> 16; at 32 768 one workgroup would take 47 us, the six launches 35.
constexpr int kPatSmallThreads = 1024, kPatSmallKeys = 16;
constexpr int kPatFew = 11264;  // above, the launches of pat_wide_kernel take less (clustered samples, us, one workgroup and they: 9000 16.8 and 18.8, 11 264 19.1 and 19.1, 16 384 24.4 and 19.5)
__global__ __launch_bounds__(kPatSmallThreads) void pat_small_kernel(const float* __restrict__ s, int n, double p,
                                                                     float* __restrict__ threshold,
                                                                     long long* __restrict__ n_finite) {
  __shared__ unsigned int s_h[256];
  __shared__ unsigned int s_bad, s_digit, s_before;
  const int tid = threadIdx.x, lane = tid & 63;
  if (tid == 0) s_bad = 0u;
  unsigned int key[kPatSmallKeys];
#pragma unroll
  for (int u = 0; u < kPatSmallKeys; ++u) {
    const int i = u * kPatSmallThreads + tid;
    key[u] = i < n ? key_of(s[i]) : 0u;
  }
  __syncthreads();
  unsigned int bad = 0;
#pragma unroll
  for (int u = 0; u < kPatSmallKeys; ++u) bad += (unsigned int)__popcll(__ballot(key[u] == 0xffffffffu));
  if (lane == 0 && bad) atomicAdd(&s_bad, bad);
  __syncthreads();
  const long long n_f = (long long)n - (long long)s_bad;
  if (tid == 0 && n_finite) *n_finite = n_f;
  if (n_f <= 0) {
    if (tid == 0) *threshold = -INFINITY;
    return;
  }
  long long k = pat_rank(p, n_f);
  unsigned int prefix = 0;
  for (int pass = 0; pass < 4; ++pass) {
    const int shift = 24 - 8 * pass;
    const unsigned int mask = pass == 0 ? 0u : 0xffffffffu << (32 - 8 * pass);
    if (tid < 256) s_h[tid] = 0u;
    __syncthreads();
#pragma unroll
    for (int u = 0; u < kPatSmallKeys; ++u) {
      if (u * kPatSmallThreads >= n) break;  // the same for the whole workgroup
      const bool in = u * kPatSmallThreads + tid < n && (key[u] & mask) == prefix;
      count_bin(s_h, in ? (int)((key[u] >> shift) & 255u) : -1);
    }
    __syncthreads();
    if (tid < 64) {  // four bins per lane: the bin that holds rank k
      unsigned int c[4], sum = 0;
#pragma unroll
      for (int b = 0; b < 4; ++b) {
        c[b] = s_h[4 * lane + b];
        sum += c[b];
      }
      unsigned int incl = sum;
#pragma unroll
      for (int off = 1; off < 64; off <<= 1) {
        const unsigned int v = __shfl_up(incl, off);
        if (lane >= off) incl += v;
      }
      unsigned int before = incl - sum;
#pragma unroll
      for (int b = 0; b < 4; ++b) {
        if ((long long)before < k && k <= (long long)before + c[b]) {  // exactly one bin of one lane
          s_digit = 4 * lane + b;
          s_before = before;
        }
        before += c[b];
      }
    }
    __syncthreads();
    prefix |= s_digit << shift;
    k -= s_before;
    __syncthreads();
  }
  if (tid == 0) *threshold = value_of(prefix);
}

__global__ __launch_bounds__(kPatThreads) void pat_hist_kernel(const float* __restrict__ s, long long n, double p,
                                                               PatState* st, int pass) {
  __shared__ unsigned int s_h[3][256];
  __shared__ unsigned int s_local[256];
  __shared__ long long s_wave[4], s_sel[2];
  __shared__ unsigned int s_bad;
  const int tid = threadIdx.x;
  s_local[tid] = 0u;
  if (tid == 0) s_bad = 0u;
  for (int j = 0; j < pass; ++j) s_h[j][tid] = st->hist[j][tid];
  __syncthreads();
  const long long n_f = n - (long long)st->nonfinite;  // final once pass 0 is complete
  const unsigned int prefix = (pass > 0 && n_f > 0) ? pat_prefix(s_h, pass, pat_rank(p, n_f), s_wave, s_sel) : 0u;
  const unsigned int mask = pass == 0 ? 0u : 0xffffffffu << (32 - 8 * pass);
  const int shift = 24 - 8 * pass;
  unsigned int bad = 0;
  for (long long i = (long long)blockIdx.x * kPatThreads + tid; i < n; i += (long long)gridDim.x * kPatThreads) {
    const unsigned int k = key_of(s[i]);
    if ((k & mask) == prefix) atomicAdd(&s_local[(k >> shift) & 255u], 1u);
    bad += (k == 0xffffffffu);
  }
  if (pass == 0 && bad) atomicAdd(&s_bad, bad);
  __syncthreads();
  if (s_local[tid]) atomicAdd(&st->hist[pass][tid], s_local[tid]);
  if (pass == 0 && tid == 0 && s_bad) atomicAdd(&st->nonfinite, s_bad);
}

__global__ __launch_bounds__(kPatThreads) void pat_final_kernel(long long n, double p, const PatState* st,
                                                                float* __restrict__ threshold,
                                                                long long* __restrict__ n_finite) {
  __shared__ unsigned int s_h[4][256];
  __shared__ long long s_wave[4], s_sel[2];
  const int tid = threadIdx.x;
  for (int j = 0; j < 4; ++j) s_h[j][tid] = st->hist[j][tid];
  __syncthreads();
  const long long n_f = n - (long long)st->nonfinite;
  const unsigned int key = n_f > 0 ? pat_prefix(s_h, 4, pat_rank(p, n_f), s_wave, s_sel) : 0u;
  if (tid == 0) {
    *threshold = n_f > 0 ? value_of(key) : -INFINITY;
    if (n_finite) *n_finite = n_f;
  }
}

// Many samples in three passes of 11, 11 and 10 bits instead of four of 8, the last workgroup to arrive in the third one
// finishing the job: four launches instead of six, for a larger state.  What bounds it is launches and the chain inside each
// (state, prefix, samples, counts out), not the samples.  Six launches -> these, us: 30 000 samples 29 -> 17, 1 million 40 -> 27,
// 4 million 77 -> 38.  Samples that are not finite (lists without a candidate) are counted but not binned: their adds would all
// go to one address, one lane after the other (4 million of nothing else 68 us, 26 so; 43 in six launches).
constexpr int kWideThreads = 1024, kWideBins = 2048, kWideUnroll = 4;
struct PatWideState {
  unsigned int hist[3][kWideBins];
  unsigned int nonfinite, arrived;
  unsigned int pad[2];
};

__global__ __launch_bounds__(kWideThreads) void pat_wide_clear_kernel(PatWideState* st) {
  unsigned int* w = reinterpret_cast<unsigned int*>(st);
  for (int i = threadIdx.x; i < (int)(sizeof(PatWideState) / 4); i += kWideThreads) w[i] = 0u;
}

// The bin of `hist` that holds rank k, to every thread; k becomes the rank within it.  FRESH: the counts were added by other
// workgroups of this launch, so the loads go to where their atomic adds went.
template <bool FRESH>
__device__ __forceinline__ unsigned int pat_wide_digit(unsigned int* hist, long long& k, unsigned int* s_wave, long long* s_sel) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  unsigned int c[2];
#pragma unroll
  for (int b = 0; b < 2; ++b)
    c[b] = FRESH ? __hip_atomic_load(&hist[2 * tid + b], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : hist[2 * tid + b];
  unsigned int incl = c[0] + c[1];
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const unsigned int v = __shfl_up(incl, off);
    if (lane >= off) incl += v;
  }
  if (lane == 63) s_wave[wave] = incl;
  if (tid == 0) {
    s_sel[0] = kWideBins - 1;
    s_sel[1] = 0;
  }
  __syncthreads();
  unsigned int before = incl - c[0] - c[1];
#pragma unroll
  for (int w = 0; w < kWideThreads / 64; ++w) before += w < wave ? s_wave[w] : 0u;
#pragma unroll
  for (int b = 0; b < 2; ++b) {
    if ((long long)before < k && k <= (long long)before + c[b]) {  // exactly one bin, if k is within the total
      s_sel[0] = 2 * tid + b;
      s_sel[1] = before;
    }
    before += c[b];
  }
  __syncthreads();
  const unsigned int digit = (unsigned int)s_sel[0];
  k -= s_sel[1];
  __syncthreads();  // the two are rewritten by the next call
  return digit;
}

template <int PASS>
__global__ __launch_bounds__(kWideThreads) void pat_wide_kernel(const float* __restrict__ s, long long n, double p, PatWideState* st,
                                                                float* __restrict__ threshold, long long* __restrict__ n_finite) {
  constexpr int kShift = PASS == 0 ? 21 : PASS == 1 ? 10 : 0;
  constexpr unsigned int kBins = PASS == 2 ? 1024u : 2048u;
  __shared__ unsigned int s_local[kWideBins];
  __shared__ unsigned int s_wave[kWideThreads / 64], s_bad;
  __shared__ long long s_sel[2];
  const int tid = threadIdx.x;
  const long long stride = (long long)gridDim.x * kWideThreads;
  // the first samples are on their way while the prefix is worked out
  float x[kWideUnroll];
  auto load = [&](long long i0) {
#pragma unroll
    for (int u = 0; u < kWideUnroll; ++u) {
      const long long i = i0 + u * stride;
      x[u] = i < n ? s[i] : 0.f;
    }
  };
  long long i0 = (long long)blockIdx.x * kWideThreads + tid;
  load(i0);
  s_local[tid] = 0u;
  s_local[tid + kWideThreads] = 0u;
  if (tid == 0) s_bad = 0u;
  long long k = 0;
  unsigned int prefix = 0;
  bool any = true;
  if (PASS > 0) {
    const long long n_f = n - (long long)st->nonfinite;
    any = n_f > 0;
    k = any ? pat_rank(p, n_f) : 1;
    prefix = pat_wide_digit<false>(st->hist[0], k, s_wave, s_sel);
    if (PASS > 1) prefix = prefix << 11 | pat_wide_digit<false>(st->hist[1], k, s_wave, s_sel);
  }
  __syncthreads();
  unsigned int bad = 0;
  for (; any && i0 - tid < n; i0 += kWideUnroll * stride) {  // the same for the whole workgroup
    unsigned int key[kWideUnroll];
#pragma unroll
    for (int u = 0; u < kWideUnroll; ++u) key[u] = key_of(x[u]);
    const long long here = i0;
    load(i0 + kWideUnroll * stride);
#pragma unroll
    for (int u = 0; u < kWideUnroll; ++u) {
      if (here + u * stride >= n) break;
      const bool finite = key[u] != 0xffffffffu;
      if (PASS == 0) bad += !finite;
      if (PASS == 0 ? finite : (key[u] >> (PASS == 1 ? 21 : 10)) == prefix) atomicAdd(&s_local[(key[u] >> kShift) & (kBins - 1u)], 1u);
    }
  }
  if (PASS == 0 && bad) atomicAdd(&s_bad, bad);
  __syncthreads();
  for (unsigned int b = tid; b < kBins; b += kWideThreads)
    if (s_local[b]) __hip_atomic_fetch_add(&st->hist[PASS][b], s_local[b], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  if (PASS == 0 && tid == 0 && s_bad) __hip_atomic_fetch_add(&st->nonfinite, s_bad, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  if (PASS < 2) return;
  // the last workgroup to arrive has everyone's counts: its own have reached memory before it says so, and so had the others'
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  if (tid == 0) s_bad = __hip_atomic_fetch_add(&st->arrived, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  __syncthreads();
  if (s_bad != gridDim.x - 1) return;
  const unsigned int low = pat_wide_digit<true>(st->hist[2], k, s_wave, s_sel);
  if (tid == 0) {
    *threshold = any ? value_of(prefix << 10 | low) : -INFINITY;
    if (n_finite) *n_finite = n - (long long)st->nonfinite;
  }
}

__global__ __launch_bounds__(256) void apply_threshold_kernel(const int32_t* __restrict__ best_idx,
                                                              const float* __restrict__ best_dist, long long n,
                                                              const float* __restrict__ threshold,
                                                              int32_t* __restrict__ match_idx) {
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const float thr = *threshold;
  const int idx = best_idx[i];
  match_idx[i] = (idx >= 0 && best_dist[i] <= thr) ? idx : -1;
}

}  // namespace
}  // namespace rc

extern "C" size_t rc_pat_workspace_size(void) { return sizeof(rc::PatWideState); }

extern "C" rc_status rc_pat_threshold(const float* samples, int64_t n, double p, float* threshold, int64_t* n_finite,
                                      void* workspace, size_t workspace_bytes, void* hip_stream) {
  using namespace rc;
  clear_error();
  if (n < 0 || n > 0x7fffffffLL) return fail(RC_ERR_INVALID_ARG, "rc_pat_threshold: n = %lld outside [0, 2^31)", (long long)n);
  if (!(p >= 0.0 && p <= 100.0)) return fail(RC_ERR_INVALID_ARG, "rc_pat_threshold: p = %g outside [0, 100]", p);
  if (!threshold || (n > 0 && !samples)) return fail(RC_ERR_INVALID_ARG, "rc_pat_threshold: NULL samples or threshold");
  if (!workspace || workspace_bytes < sizeof(PatState) || !aligned16(workspace))
    return fail(RC_ERR_WORKSPACE, "rc_pat_threshold: workspace of %zu bytes needed (16-byte aligned), got %zu",
                sizeof(PatState), workspace_bytes);
  hipStream_t st = static_cast<hipStream_t>(hip_stream);
  const bool wide = workspace_bytes >= sizeof(PatWideState);
  if (n <= (wide ? kPatFew : kPatSmallThreads * kPatSmallKeys)) {
    pat_small_kernel<<<1, kPatSmallThreads, 0, st>>>(samples, (int)n, p, threshold, reinterpret_cast<long long*>(n_finite));
    return check_launch("rc_pat_threshold(few samples)");
  }
  if (wide) {
    PatWideState* state = static_cast<PatWideState*>(workspace);
    pat_wide_clear_kernel<<<1, kWideThreads, 0, st>>>(state);
    if (rc_status s = check_launch("rc_pat_threshold(clear)")) return s;
    long long wgs = (n + kWideThreads * kWideUnroll - 1) / (kWideThreads * kWideUnroll);
    if (wgs > 256) wgs = 256;  // one per compute unit; 512: 3 million samples 42 us, 256: 34
    long long* nf = reinterpret_cast<long long*>(n_finite);
    pat_wide_kernel<0><<<(unsigned)wgs, kWideThreads, 0, st>>>(samples, (long long)n, p, state, threshold, nf);
    pat_wide_kernel<1><<<(unsigned)wgs, kWideThreads, 0, st>>>(samples, (long long)n, p, state, threshold, nf);
    pat_wide_kernel<2><<<(unsigned)wgs, kWideThreads, 0, st>>>(samples, (long long)n, p, state, threshold, nf);
    return check_launch("rc_pat_threshold(histograms)");
  }
  PatState* state = static_cast<PatState*>(workspace);
  pat_clear_kernel<<<1, kPatThreads, 0, st>>>(state);
  if (rc_status s = check_launch("rc_pat_threshold(clear)")) return s;
  long long wgs = (n + kPatThreads * 16 - 1) / (kPatThreads * 16);  // about 16 samples per thread
  if (wgs > 2048) wgs = 2048;
  for (int pass = 0; pass < 4; ++pass) {
    pat_hist_kernel<<<(unsigned)wgs, kPatThreads, 0, st>>>(samples, (long long)n, p, state, pass);
    if (rc_status s = check_launch("rc_pat_threshold(histogram)")) return s;
  }
  pat_final_kernel<<<1, kPatThreads, 0, st>>>((long long)n, p, state, threshold,
                                              reinterpret_cast<long long*>(n_finite));
  return check_launch("rc_pat_threshold(final)");
}

extern "C" rc_status rc_apply_threshold(const int32_t* best_idx, const float* best_dist, int64_t n,
                                        const float* threshold, int32_t* match_idx, void* hip_stream) {
  using namespace rc;
  clear_error();
  if (n < 0) return fail(RC_ERR_INVALID_ARG, "rc_apply_threshold: negative n");
  if (n == 0) return RC_OK;
  if (!best_idx || !best_dist || !threshold || !match_idx)
    return fail(RC_ERR_INVALID_ARG, "rc_apply_threshold: NULL pointer");
  if (n > 0x7fffffffLL * 256) return fail(RC_ERR_UNSUPPORTED, "rc_apply_threshold: n beyond the grid limits");
  apply_threshold_kernel<<<(unsigned)((n + 255) / 256), 256, 0, static_cast<hipStream_t>(hip_stream)>>>(
      best_idx, best_dist, (long long)n, threshold, match_idx);
  return check_launch("rc_apply_threshold");
}
