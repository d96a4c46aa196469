// rc_score_candidates: Stage 2 restricted to listed candidates (ReasonCache Sec. IV-A: only the
// blocks of the steps flagged by Stage 1 are compared).  HBM-bound gather: the pool blocks' K and V
// tensors are streamed against the query block, the dot products accumulated in fp32 and normalised
// with the cached squared norms.  A workgroup takes 16 or 4 candidates of a list, or, where lists are
// many and share blocks, a wave takes a list; a small kernel (or the wave) picks the best candidate.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "rc_common.hpp"
#include "rc_lists_plan.hpp"

namespace rc {
namespace {

constexpr int kCandThreads = 256;

typedef _Float16 half2_t __attribute__((ext_vector_type(2)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

// <x, y> of the 8 fp16 / bf16 values packed in two 16-byte words, accumulated in fp32.
template <bool BF16>
__device__ __forceinline__ float dot8(u32x4 x, u32x4 y, float acc) {
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const unsigned int xi = x[i], yi = y[i];  // copies: a bit_cast applied to the vector element itself reads lane 0
    if (BF16) {
      acc = fmaf(__uint_as_float(xi << 16), __uint_as_float(yi << 16), acc);
      acc = fmaf(__uint_as_float(xi & 0xffff0000u), __uint_as_float(yi & 0xffff0000u), acc);
    } else {
      acc = __builtin_amdgcn_fdot2(__builtin_bit_cast(half2_t, xi), __builtin_bit_cast(half2_t, yi), acc, false);
    }
  }
  return acc;
}

struct CandParams {
  const char *kq, *vq, *kp, *vp;
  const float *q_ksq, *q_vsq, *p_ksq, *p_vsq;
  const uint8_t* live;
  const int32_t* cand;
  float* scores;
  long long q_lstride_b, p_lstride_b;
  int Q, P, C;
  int block_bytes;  // one K (or V) tensor of a block
  int heads;        // 1 in block mode, H in per-head-all mode
};

// grid = (ceil(C / kCandPerWg), Q, L).  A workgroup scores kCandPerWg candidates of one query: the query
// chunk a thread holds is used against all of them, which divides the query traffic from the L2.
// Thread t takes the 16-byte chunks t, t+256, ...; 16 consecutive chunks are one head of one
// token, so with 16*heads dividing 256 a thread stays in one head: head = (t/16) % heads.
// ANYH (per-head mode with a head count that does not divide 16, e.g. 10 KV heads): the head of a
// thread's chunk changes from one trip to the next, so every trip ends with the sum over the 16
// lanes of a (token, head) group, added by the group's first lane to its own slot
// hpart[candidate][K or V][head][group]: no two groups share a slot, so plain LDS updates do.
// Few pairs: kCandFew candidates per workgroup, so that a call of a few queries has workgroups for more of the
// chip and a thread more of its slices in flight (rule and measurements at cand_per_wg).
constexpr int kCandFew = 4;

template <bool BF16, bool ANYH, int PER>
__global__ __launch_bounds__(kCandThreads) void candidates_kernel(const CandParams p) {
  __shared__ float part[PER][2][kCandThreads / 16];
  __shared__ float head_score[PER][16];
  __shared__ float hpart[ANYH ? PER : 1][2][ANYH ? 16 : 1][ANYH ? kCandThreads / 16 : 1];
  const int c0 = blockIdx.x * PER, q = blockIdx.y, tid = threadIdx.x;
  const long long l = blockIdx.z;
  const long long slot0 = (l * p.Q + q) * p.C + c0;
  int pidx[PER];
  bool valid[PER];
  const u32x4* xp_k[PER];
  const u32x4* xp_v[PER];
  bool any = false;
#pragma unroll
  for (int c = 0; c < PER; ++c) {  // the same for the whole workgroup
    pidx[c] = (c0 + c < p.C) ? p.cand[slot0 + c] : -1;
    valid[c] = pidx[c] >= 0 && pidx[c] < p.P && (!p.live || p.live[l * p.P + pidx[c]]);
    const long long off = l * p.p_lstride_b + (long long)(valid[c] ? pidx[c] : 0) * p.block_bytes;
    xp_k[c] = reinterpret_cast<const u32x4*>(p.kp + off);
    xp_v[c] = reinterpret_cast<const u32x4*>(p.vp + off);
    any = any || valid[c];
    if (!valid[c] && tid == 0 && c0 + c < p.C) p.scores[slot0 + c] = -INFINITY;
  }
  if (!any) return;
  if (ANYH) {
    float* z = &hpart[0][0][0][0];
    for (int i = tid; i < PER * 2 * 16 * (kCandThreads / 16); i += kCandThreads) z[i] = 0.f;
    __syncthreads();
  }
  const u32x4* xq_k = reinterpret_cast<const u32x4*>(p.kq + l * p.q_lstride_b + (long long)q * p.block_bytes);
  const u32x4* xq_v = reinterpret_cast<const u32x4*>(p.vq + l * p.q_lstride_b + (long long)q * p.block_bytes);
  const int chunks = p.block_bytes / 16;
  float dk[PER], dv[PER];
#pragma unroll
  for (int c = 0; c < PER; ++c) dk[c] = dv[c] = 0.f;
  auto trip = [&](int i) {
    const u32x4 qk = xq_k[i], qv = xq_v[i];
    u32x4 pk[PER], pv[PER];
#pragma unroll
    for (int c = 0; c < PER; ++c)
      if (valid[c]) {
        pk[c] = __builtin_nontemporal_load(xp_k[c] + i);
        pv[c] = __builtin_nontemporal_load(xp_v[c] + i);
      }
#pragma unroll
    for (int c = 0; c < PER; ++c)
      if (valid[c]) {
        dk[c] = dot8<BF16>(qk, pk[c], dk[c]);
        dv[c] = dot8<BF16>(qv, pv[c], dv[c]);
      }
    if (ANYH) {
      const int head = (i >> 4) % p.heads;
#pragma unroll
      for (int c = 0; c < PER; ++c)
        if (valid[c]) {  // the same for the whole workgroup
#pragma unroll
          for (int off = 8; off > 0; off >>= 1) {
            dk[c] += __shfl_xor(dk[c], off);
            dv[c] += __shfl_xor(dv[c], off);
          }
          if ((tid & 15) == 0) {
            hpart[c][0][head][tid >> 4] += dk[c];
            hpart[c][1][head][tid >> 4] += dv[c];
          }
          dk[c] = dv[c] = 0.f;
        }
    }
  };
  // chunks = 16*T*H is a multiple of 256
  if (ANYH) {
    for (int i = tid; i < chunks; i += kCandThreads) trip(i);
  } else {
    constexpr int TRIPS = PER <= 4 ? 4 : 2;
#pragma unroll TRIPS
    for (int i = tid; i < chunks; i += kCandThreads) trip(i);
  }
  // sum over the 16 lanes that share a (token, head) group, then over the groups of a head
#pragma unroll
  for (int c = 0; c < PER; ++c) {
#pragma unroll
    for (int off = 8; off > 0; off >>= 1) {
      dk[c] += __shfl_xor(dk[c], off);
      dv[c] += __shfl_xor(dv[c], off);
    }
    if ((tid & 15) == 0) {
      part[c][0][tid >> 4] = dk[c];
      part[c][1][tid >> 4] = dv[c];
    }
  }
  __syncthreads();
  const int c = tid >> 4, h = tid & 15;  // one thread per (candidate, head)
  if (c < PER && h < p.heads && valid[c]) {
    float sk = 0.f, sv = 0.f;
    if (ANYH) {
      for (int g = 0; g < kCandThreads / 16; ++g) {
        sk += hpart[c][0][h][g];
        sv += hpart[c][1][h][g];
      }
    } else {
      for (int g = h; g < kCandThreads / 16; g += p.heads) {
        sk += part[c][0][g];
        sv += part[c][1][g];
      }
    }
    const long long oq = (l * p.Q + q) * p.heads + h, op = (l * p.P + pidx[c]) * p.heads + h;
    const float nkq = p.q_ksq[oq], nvq = p.q_vsq[oq], nkp = p.p_ksq[op], nvp = p.p_vsq[op];
    const float ck = (nkq > 0.f && nkp > 0.f) ? sk * __builtin_amdgcn_rsqf(nkq) * __builtin_amdgcn_rsqf(nkp) : 0.f;
    const float cv = (nvq > 0.f && nvp > 0.f) ? sv * __builtin_amdgcn_rsqf(nvq) * __builtin_amdgcn_rsqf(nvp) : 0.f;
    head_score[c][h] = 0.5f * (ck + cv);
  }
  __syncthreads();
  if (tid < PER && valid[tid]) {
    float s = head_score[tid][0];
    for (int hh = 1; hh < p.heads; ++hh) s = fminf(s, head_score[tid][hh]);
    p.scores[slot0 + tid] = s;
  }
}

// One thread per (layer, query): best of its list, equal scores to the lowest pool index.
__global__ __launch_bounds__(256) void candidates_select_kernel(const float* __restrict__ scores,
                                                                const int32_t* __restrict__ cand, long long LQ, int C,
                                                                float tau, int32_t* __restrict__ best_idx,
                                                                float* __restrict__ best_score,
                                                                int32_t* __restrict__ match_idx) {
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= LQ) return;
  float best = -INFINITY;
  int bidx = -1;
  for (int c = 0; c < C; ++c) {
    const float s = scores[i * C + c];
    const int pi = cand[i * C + c];
    if (s == -INFINITY) continue;  // empty, out of range or dead
    if (s > best || (s == best && pi < bidx) || bidx < 0) {
      best = s;
      bidx = pi;
    }
  }
  best_idx[i] = bidx;
  best_score[i] = best;
  match_idx[i] = (bidx >= 0 && best >= tau) ? bidx : -1;
}

// ---- layer-mean Euclidean distance of listed pairs (Stage 2 exactly as Sec. IV-A runs it)

typedef float float2_t __attribute__((ext_vector_type(2)));

// sum of (x - y)^2 over the 8 fp16 / bf16 values of two 16-byte words, in fp32 (differences of
// 16-bit values are exact in fp32, so only the squares and the sum round).
template <bool BF16>
__device__ __forceinline__ float sqdiff8(u32x4 x, u32x4 y, float acc) {
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const unsigned int xi = x[i], yi = y[i];
    float a0, a1, b0, b1;
    if (BF16) {
      a0 = __uint_as_float(xi << 16);
      a1 = __uint_as_float(xi & 0xffff0000u);
      b0 = __uint_as_float(yi << 16);
      b1 = __uint_as_float(yi & 0xffff0000u);
    } else {
      const float2_t a = __builtin_convertvector(__builtin_bit_cast(half2_t, xi), float2_t);
      const float2_t b = __builtin_convertvector(__builtin_bit_cast(half2_t, yi), float2_t);
      a0 = a[0];
      a1 = a[1];
      b0 = b[0];
      b1 = b[1];
    }
    const float d0 = a0 - b0, d1 = a1 - b1;
    acc = fmaf(d0, d0, acc);
    acc = fmaf(d1, d1, acc);
  }
  return acc;
}

struct CandDistParams {
  const char *kq, *vq, *kp, *vp;
  const uint8_t* live;   // [P] or null
  const int32_t* cand;   // [Q][C]
  float* part;           // [groups][Q][C]: sum over the group's layers of |Kq-Kp| + |Vq-Vp|
  long long q_lstride_b, p_lstride_b;
  int Q, P, C, L, G;     // G = layers per group
  int block_bytes;
};

// grid = (ceil(C / kCandPerWg), Q, layer groups).  The workgroup walks the layers of its group; per
// layer it streams the listed pool blocks against the query chunk held in registers, reduces the
// squared differences over the workgroup and adds the two square roots to the running sum that
// thread c keeps for candidate c.
template <bool BF16, int PER>
__global__ __launch_bounds__(kCandThreads) void candidate_distances_kernel(const CandDistParams p) {
  __shared__ float s_red[kCandThreads / 64][PER][2];
  const int c0 = blockIdx.x * PER, q = blockIdx.y, tid = threadIdx.x;
  const int l0 = blockIdx.z * p.G, nl = min(p.G, p.L - l0);
  int pidx[PER];
  bool valid[PER];
  bool any = false;
#pragma unroll
  for (int c = 0; c < PER; ++c) {  // the same for the whole workgroup
    pidx[c] = (c0 + c < p.C) ? p.cand[(long long)q * p.C + c0 + c] : -1;
    valid[c] = pidx[c] >= 0 && pidx[c] < p.P && (!p.live || p.live[pidx[c]]);
    any = any || valid[c];
  }
  if (!any) return;  // the selection kernel derives validity itself and never reads these sums
  const int chunks = p.block_bytes / 16;
  float total = 0.f;
  for (int li = 0; li < nl; ++li) {
    const long long l = l0 + li;
    const u32x4* xq_k = reinterpret_cast<const u32x4*>(p.kq + l * p.q_lstride_b + (long long)q * p.block_bytes);
    const u32x4* xq_v = reinterpret_cast<const u32x4*>(p.vq + l * p.q_lstride_b + (long long)q * p.block_bytes);
    float dk[PER], dv[PER];
#pragma unroll
    for (int c = 0; c < PER; ++c) dk[c] = dv[c] = 0.f;
    constexpr int TRIPS = PER <= 4 ? 4 : 1;
#pragma unroll TRIPS
    for (int i = tid; i < chunks; i += kCandThreads) {
      const u32x4 qk = xq_k[i], qv = xq_v[i];
      u32x4 pk[PER], pv[PER];
#pragma unroll
      for (int c = 0; c < PER; ++c)
        if (valid[c]) {
          const long long off = l * p.p_lstride_b + (long long)pidx[c] * p.block_bytes;
          pk[c] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(p.kp + off) + i);
          pv[c] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(p.vp + off) + i);
        }
#pragma unroll
      for (int c = 0; c < PER; ++c)
        if (valid[c]) {
          dk[c] = sqdiff8<BF16>(qk, pk[c], dk[c]);
          dv[c] = sqdiff8<BF16>(qv, pv[c], dv[c]);
        }
    }
#pragma unroll
    for (int c = 0; c < PER; ++c) {
#pragma unroll
      for (int off = 32; off > 0; off >>= 1) {
        dk[c] += __shfl_xor(dk[c], off);
        dv[c] += __shfl_xor(dv[c], off);
      }
      if ((tid & 63) == 0) {
        s_red[tid >> 6][c][0] = dk[c];
        s_red[tid >> 6][c][1] = dv[c];
      }
    }
    __syncthreads();
    if (tid < PER) {
      float sk = 0.f, sv = 0.f;
#pragma unroll
      for (int w = 0; w < kCandThreads / 64; ++w) {
        sk += s_red[w][tid][0];
        sv += s_red[w][tid][1];
      }
      total += __builtin_amdgcn_sqrtf(sk) + __builtin_amdgcn_sqrtf(sv);
    }
    __syncthreads();  // s_red is rewritten by the next layer
  }
  if (tid < PER && c0 + tid < p.C)
    p.part[((long long)blockIdx.z * p.Q + q) * p.C + c0 + tid] = total;
}

// ---- many lists: a wave per list

// Up to 2 * SLOTS candidates of one query and a wave for all of them: lanes 0..31 and 32..63 hold the same 512 bytes of
// the query against two candidates at a time, K first, then V, with no LDS and no barrier.  The waves of a launch start
// together and advance at the same rate, so the lists of a layer read the same 512-byte window of their blocks at about the
// same time, and a block that several lists name comes from the L2 (neighbouring lists are dealt to one XCD) or the
// memory-side cache when the second of them asks for it.  A workgroup per list (above) keeps the lists on a chip apart by up
// to a whole block each.  The waves of a compute unit are served oldest first and drift apart; where there are enough of them
// eight are a workgroup that meets every two windows, elsewhere a wave is a workgroup of its own, so that few lists spread over
// all compute units (wide_plan).  What bounds it: the stream of blocks, less what lists share (64 x 4096 x 256 lists of 16,
// 32-KB tensors: 2120 us = 8.6 TB/s of listed blocks and queries, 7.0 of them from memory; 2431 with waves alone, 2591 in
// workgroups of a list; 36 x 150 x 65 x 17: 250 -> 84).
// Lists are as long as their fullest one and many are partly or wholly empty.  The valid candidates of a wave move to its first
// slots; it walks 2 or 4 of the SLOTS where they fit, none where there is none, and a workgroup that is nearly empty throughout
// keeps no step.  (64 x 4096 x 256 x 16 with a part of the entries empty, workgroup per list -> every slot walked -> this, us:
// a half 1403 -> 1425 -> 1420, three quarters 836 -> 1188 -> 879, nine tenths 554 -> 1034 -> 472, all 60 -> 889 -> 22;
// 0 to 16 valid, evenly 1415 -> 1531 -> 1511.  37 x 1823 x 795 x 19, three quarters 2627 -> 2412 -> 1600.  With a slot
// count for every second number of candidates a group of waves falls out of step where a quarter is empty: 44 x 257 x 110 x 11
// 565 -> 600, as it is 562.)
struct WideParams {
  const char *kq, *vq, *kp, *vp;
  const float *q_ksq, *q_vsq, *p_ksq, *p_vsq;
  const uint8_t* live;   // [L][P]; distances: [P]
  const int32_t* cand;   // [L][Q][C]; distances: [Q][C]
  float* out;            // scores [L][Q][C]; distances: sums [groups of layers][Q][C]
  int32_t* best_idx;
  float* best_score;
  int32_t* match_idx;
  long long q_lstride_b, p_lstride_b;
  int Q, P, C;
  int L, G;              // distances: layers, layers of a group
  int per, parts;        // candidates of a wave, waves per list
  int block_bytes;
  int waves;             // of a workgroup, at most kWideWaves
  long long wgs_z;       // workgroups of a layer, or of a group of layers
  long long items;       // workgroups
  long long per_xcd;     // workgroups of an XCD's run; 0: they are dealt out one after the other
  float tau;
};
constexpr int kWindow = 512;   // bytes of a block per step

template <bool BF16, int SLOTS, bool DIST>
__global__ __launch_bounds__(64 * kWideWaves, SLOTS == 8 ? 3 : 4) void candidates_wide_kernel(const WideParams p) {
  __shared__ int s_valid[kWideWaves];
  const int lane = threadIdx.x & 63, half = lane >> 5;
  const long long item = p.per_xcd ? (blockIdx.x & 7) * p.per_xcd + (blockIdx.x >> 3) : blockIdx.x;
  if (item >= p.items) return;
  const long long z = item / p.wgs_z;  // layer or group of layers
  const long long w = item % p.wgs_z * p.waves + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const bool idle = w >= (long long)p.Q * p.parts;  // a list of none
  const long long q = idle ? 0 : w / p.parts, list = z * p.Q + q;
  const int c0 = idle ? 0 : (int)(w % p.parts) * p.per, n = idle ? 0 : min(p.per, p.C - c0);
  const long long l0 = DIST ? z * p.G : z;
  const int nl = DIST ? (int)min((long long)p.G, p.L - l0) : 1;
  const long long slot0 = list * p.C + c0, cand0 = (DIST ? q : list) * p.C + c0;
  // lane s + 32 * half keeps candidate 2 * s + half
  const int mine = 2 * (lane & 31) + half;
  const bool listed = (lane & 31) < SLOTS && mine < n;
  const int pidx = listed ? p.cand[cand0 + mine] : -1;
  const bool valid = pidx >= 0 && pidx < p.P && (!p.live || p.live[(DIST ? 0 : l0 * p.P) + pidx]);
  constexpr int kNowhere = (int)0x80000000u;  // past the end of the pool's descriptor: reads as zero, no traffic
  // the valid candidates move to the front: candidate of rank r to slot r / 2, half r % 2, the others behind them
  const unsigned long long valids = __ballot(valid);
  const int n_valid = __popcll(valids);
  auto seat_of = [&](int at) {
    const int below = __popcll(valids & ((1ull << at) - 1ull)), rank = valids >> at & 1 ? below : n_valid + at - below;
    return (rank >> 1) + 32 * (rank & 1);
  };
  const int moff = __builtin_amdgcn_ds_permute(seat_of(lane) * 4, valid ? pidx * p.block_bytes : kNowhere);
  const int qoff = (lane & 31) * 16;
  const int pool_bytes = (int)((long long)p.P * p.block_bytes);  // below 2^31: a condition of this kernel
  const int steps = p.block_bytes / kWindow;                     // a multiple of 8
  struct Source {
    __amdgpu_buffer_rsrc_t q, p;
  };
  auto source = [&](int li, bool v) __attribute__((always_inline)) {
    const long long l = l0 + li;
    Source r;
    r.q = __builtin_amdgcn_make_buffer_rsrc((void*)((v ? p.vq : p.kq) + l * p.q_lstride_b + q * p.block_bytes), 0, p.block_bytes, 0x00020000);
    r.p = __builtin_amdgcn_make_buffer_rsrc((void*)((v ? p.vp : p.kp) + l * p.p_lstride_b), 0, pool_bytes, 0x00020000);
    return r;
  };
  // the waves of a workgroup meet where one of them at least has more than half of its slots to read
  bool together = false;
  if (p.waves > 1) {
    if (lane == 0) s_valid[threadIdx.x >> 6] = n_valid;
    __syncthreads();
    int most = 0;
#pragma unroll
    for (int i = 0; i < kWideWaves; ++i) most = max(most, s_valid[i]);
    together = __builtin_amdgcn_readfirstlane(most) > SLOTS;
  }
  float total = 0.f, sk = 0.f, sv = 0.f;
  // all layers with the first N slots; the sum of a candidate ends in the lane of its seat
  auto score_slots = [&](auto n_slots) __attribute__((always_inline)) {
    constexpr int N = decltype(n_slots)::value;
    int off[N];
#pragma unroll
    for (int s = 0; s < N; ++s) off[s] = __shfl(moff, s + 32 * half) + (lane & 31) * 16;
    u32x4 x[2][N], y[2];
    auto load = [&](int buf, const Source& src, int step) __attribute__((always_inline)) {
      y[buf] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(src.q, qoff, step * kWindow, 0));
#pragma unroll
      for (int s = 0; s < N; ++s) x[buf][s] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(src.p, off[s], step * kWindow, 0));
    };
    float run[N];
    auto add = [&](int buf) __attribute__((always_inline)) {
#pragma unroll
      for (int s = 0; s < N; ++s) run[s] = DIST ? sqdiff8<BF16>(y[buf], x[buf][s], run[s]) : dot8<BF16>(y[buf], x[buf][s], run[s]);
    };
    auto walk = [&](const Source& src, const Source& next, bool more) __attribute__((always_inline)) {  // one tensor
      float d[N];
#pragma unroll
      for (int s = 0; s < N; ++s) d[s] = 0.f;
      // short chains of fp32 adds join the running sums, so that the error stays that of 256 lanes per block: squares, all of one
      // sign, lose most in long chains (8 steps, blocks of 12 KB: 1.3 times), products of both signs in the running sums (2 steps,
      // blocks of 64 KB: 1.25 times)
      constexpr int kFold = DIST ? 2 : 8;  // steps; a block has a multiple of 8
#pragma unroll 1
      for (int t0 = 0; t0 < steps; t0 += kFold) {
#pragma unroll
        for (int s = 0; s < N; ++s) run[s] = 0.f;
#pragma unroll 1
        for (int t = t0; t < t0 + kFold; t += 2) {
          if (together) __builtin_amdgcn_s_barrier();
          load(1, src, t + 1);
          __builtin_amdgcn_sched_barrier(0);
          add(0);
          __builtin_amdgcn_sched_barrier(0);
          if (t + 2 < steps)
            load(0, src, t + 2);
          else if (more)
            load(0, next, 0);
          __builtin_amdgcn_sched_barrier(0);
          add(1);
          __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int s = 0; s < N; ++s) d[s] += run[s];
      }
      float sum = 0.f;
#pragma unroll
      for (int s = 0; s < N; ++s) {
#pragma unroll
        for (int o = 16; o > 0; o >>= 1) d[s] += __shfl_xor(d[s], o);
        if ((lane & 31) == s) sum = d[s];
      }
      return sum;
    };
    load(0, source(0, false), 0);
    for (int li = 0; li < nl; ++li) {
      sk = walk(source(li, false), source(li, true), true);
      sv = walk(source(li, true), source(min(li + 1, nl - 1), false), li + 1 < nl);
      if (DIST) total += __builtin_amdgcn_sqrtf(sk) + __builtin_amdgcn_sqrtf(sv);
    }
  };
  if (n_valid == 0) {
    if (together)
      for (int t = 0; t < nl * steps; ++t) __builtin_amdgcn_s_barrier();  // one per two steps of each of the two tensors
  } else if (SLOTS > 2 && n_valid <= 4) {
    score_slots(std::integral_constant<int, 2>());
  } else if (SLOTS == 8 && n_valid <= 8) {
    score_slots(std::integral_constant<int, 4>());
  } else {
    score_slots(std::integral_constant<int, SLOTS>());
  }
  if (idle) return;
  int lane_again = lane;
  asm volatile("" : "+v"(lane_again));  // the seat is worked out again: kept, it costs a register that the loops need
  const int seat = seat_of(lane_again);
  if (DIST) {
    total = __shfl(total, seat);
    if (valid) p.out[slot0 + mine] = total;  // the selection kernel derives validity itself
    return;
  }
  sk = __shfl(sk, seat);
  sv = __shfl(sv, seat);
  float score = -INFINITY;
  if (valid) {
    const long long oq = list, op = l0 * p.P + pidx;
    const float nkq = p.q_ksq[oq], nvq = p.q_vsq[oq], nkp = p.p_ksq[op], nvp = p.p_vsq[op];
    const float ck = (nkq > 0.f && nkp > 0.f) ? sk * __builtin_amdgcn_rsqf(nkq) * __builtin_amdgcn_rsqf(nkp) : 0.f;
    const float cv = (nvq > 0.f && nvp > 0.f) ? sv * __builtin_amdgcn_rsqf(nvq) * __builtin_amdgcn_rsqf(nvp) : 0.f;
    score = 0.5f * (ck + cv);
  }
  if (listed) p.out[slot0 + mine] = score;
  if (p.parts > 1) return;  // the selection kernel picks
  float best = -INFINITY;
  int bidx = -1;
#pragma unroll
  for (int c = 0; c < 2 * SLOTS; ++c) {  // in list order, as the selection kernel does; an entry that was not scored is -inf
    const float sc = __shfl(score, (c >> 1) + 32 * (c & 1));
    const int pi = __shfl(pidx, (c >> 1) + 32 * (c & 1));
    if (c >= n || sc == -INFINITY) continue;
    if (sc > best || (sc == best && pi < bidx) || bidx < 0) {
      best = sc;
      bidx = pi;
    }
  }
  if (lane != 0) return;
  p.best_idx[list] = bidx;
  p.best_score[list] = best;
  p.match_idx[list] = (bidx >= 0 && best >= p.tau) ? bidx : -1;
}

// One wave per query, a candidate per lane: layer groups added in order (8 asked for at once), scaled, validity
// re-derived, nearest candidate.  One thread per query walked all its candidates' groups one load at a time: 96
// queries x 12 candidates x 24 groups 48 -> 5.6 us.
__global__ __launch_bounds__(256) void candidate_distances_select_kernel(const float* __restrict__ part, int groups,
                                                                        const int32_t* __restrict__ cand,
                                                                        const uint8_t* __restrict__ live, int Q, int P,
                                                                        int C, float scale, float thr,
                                                                        float* __restrict__ dist,
                                                                        int32_t* __restrict__ best_idx,
                                                                        float* __restrict__ best_dist,
                                                                        int32_t* __restrict__ match_idx) {
  const int q = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (q >= Q) return;
  float best = INFINITY;
  int bidx = -1;
  for (long long c = lane; c < C; c += 64) {
    const int pi = cand[(long long)q * C + c];
    float d = INFINITY;
    if (pi >= 0 && pi < P && (!live || live[pi])) {
      const float* src = part + (long long)q * C + c;
      const long long gstride = (long long)Q * C;
      float sum = 0.f;
      for (int g = 0; g < groups; g += 8) {
        float v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] = g + u < groups ? src[(g + u) * gstride] : 0.f;
#pragma unroll
        for (int u = 0; u < 8; ++u)
          if (g + u < groups) sum += v[u];
      }
      d = sum * scale;
      if (d < best || (d == best && pi < bidx)) {
        best = d;
        bidx = pi;
      }
    }
    dist[(long long)q * C + c] = d;
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    const float d = __shfl_xor(best, off);
    const int i = __shfl_xor(bidx, off);
    if (d < best || (d == best && i >= 0 && i < bidx)) {
      best = d;
      bidx = i;
    }
  }
  if (lane != 0) return;
  best_idx[q] = bidx;
  best_dist[q] = best;
  match_idx[q] = (bidx >= 0 && best <= thr) ? bidx : -1;
}

// layers per group: enough workgroups to fill the chip, as few groups as that allows
inline int cand_layers_per_group(int L, int64_t Q, int64_t C) {
  const int64_t wgs = Q * ((C + kCandPerWg - 1) / kCandPerWg);
  int64_t groups = (4096 + wgs - 1) / (wgs > 0 ? wgs : 1);
  if (groups < 1) groups = 1;
  if (groups > L) groups = L;
  return (int)((L + groups - 1) / groups);
}

// Candidates per workgroup of a launch over `lists` lists of C (`lists` x layer groups for the distances): 4 or 16.
// Four times the workgroups pay while the chip has idle compute units, and cost the query once more per workgroup,
// most where ceil(C / 4) workgroups are badly filled (C = 5).  The time of both goes in steps, at every 256 workgroups
// (one per compute unit), so the lines are at multiples of 256 of either count: up to 256 of 4 always; up to 512, where the
// second round is well filled or a block is small; again where 16 per workgroup are just over 256.  two_trips is false
// for the kernels that have one trip's loads in flight with 16 candidates (the distances, heads that do not divide 16):
// four pay longer there.  The lines are drawn through 5800 measured points (C = 1 to 64, 32 to 511 lists, blocks of 4 to
// 128 KB per tensor): of those that take 4, all but one (7 %) are at most 4 % slower with 4 than with 16.  Some, us, 16 -> 4:
//   block score, 32 KB   C = 5   120 lists 22 -> 17   400 33 -> 41 (takes 16)   C = 8   64 25 -> 17   288 41 -> 38   400 46 -> 48 (16)
//                        C = 16  64 37 -> 20   120 39 -> 32   200 46 -> 51 (16)   264 72 -> 63
//                128 KB  C = 5   120 55 -> 41   160 57 -> 66 (16)   400 100 -> 138 (16)   C = 16  120 115 -> 96   288 252 -> 222
//   distances,    64 KB  C = 8   200 54 -> 45   C = 12  160 68 -> 51   360 110 -> 111 (16)
inline int cand_per_wg(int64_t lists, int64_t C, int block_bytes, bool two_trips) {
  const int64_t n16 = lists * ((C + kCandPerWg - 1) / kCandPerWg), n4 = lists * ((C + kCandFew - 1) / kCandFew);
  const int kb = block_bytes / 1024;
  const bool small = kb <= 16;
  auto few = [&]() {
    if (n16 >= 512) return false;
    if (C <= 4) return C < 4 || kb <= 80 || n16 <= 256 || !two_trips;   // the same workgroups, with fewer registers each
    if (C > 16 && C <= 24) return C <= 23 || n4 <= 1280;                // 16 per workgroup leave a second one almost empty
    if (kb <= 8) return n16 <= 400;
    if (n16 > 256) return (C >= 7 || small) && n4 <= (C <= 8 ? 768 : C <= 12 ? 1024 : 1280);
    if (C > 24) return n4 <= (small || !two_trips ? 768 : 512);
    if (!two_trips) return kb <= 80 || n4 <= (C == 5 ? 384 : C <= 12 ? 512 : 768);
    if (small) return C <= 12 || n4 <= 768;
    if (C <= 8) return n4 <= (kb > 40 ? 256 : C == 5 ? 352 : 448);
    return n4 <= (kb > 80 && C <= 12 ? 448 : 512);
  };
  return few() ? kCandFew : kCandPerWg;
}

template <bool BF16>
void launch_candidates(bool any_h, int per, dim3 grid, const CandParams& cp, hipStream_t st) {
  if (per == kCandFew) {
    if (any_h)
      candidates_kernel<BF16, true, kCandFew><<<grid, kCandThreads, 0, st>>>(cp);
    else
      candidates_kernel<BF16, false, kCandFew><<<grid, kCandThreads, 0, st>>>(cp);
  } else {
    if (any_h)
      candidates_kernel<BF16, true, kCandPerWg><<<grid, kCandThreads, 0, st>>>(cp);
    else
      candidates_kernel<BF16, false, kCandPerWg><<<grid, kCandThreads, 0, st>>>(cp);
  }
}

inline void set_plan(WideParams& wp, const WidePlan& plan) {
  wp.parts = plan.lists.parts;
  wp.per = plan.lists.per;
  wp.waves = plan.waves;
  wp.wgs_z = plan.wgs_z;
  wp.items = plan.items;
  wp.per_xcd = plan.per_xcd;
}

template <bool BF16, bool DIST>
void launch_wide(const WideParams& wp, hipStream_t st) {
  const unsigned grid = (unsigned)wide_grid(wp.items, wp.per_xcd);
  if (wp.per <= 4)
    candidates_wide_kernel<BF16, 2, DIST><<<grid, 64 * wp.waves, 0, st>>>(wp);
  else if (wp.per <= 8)
    candidates_wide_kernel<BF16, 4, DIST><<<grid, 64 * wp.waves, 0, st>>>(wp);
  else if (wp.per <= 12)
    candidates_wide_kernel<BF16, 6, DIST><<<grid, 64 * wp.waves, 0, st>>>(wp);
  else
    candidates_wide_kernel<BF16, 8, DIST><<<grid, 64 * wp.waves, 0, st>>>(wp);
}

// z: layers, or groups of layers; alike: all groups have as many layers.
}  // namespace
}  // namespace rc

extern "C" rc_status rc_score_candidates(const rc_kv_desc* qdesc, const rc_kv_desc* pdesc, int32_t mode,
                                         const void* kq, const void* vq, int64_t Q, const float* q_ksq,
                                         const float* q_vsq, const void* kp, const void* vp, int64_t P,
                                         const float* p_ksq, const float* p_vsq, const uint8_t* pool_live,
                                         const int32_t* cand, int64_t C, float tau, float* scores, int32_t* best_idx,
                                         float* best_score, int32_t* match_idx, void* hip_stream) {
  using namespace rc;
  clear_error();
  if (rc_status s = check_desc(qdesc, Q, "rc_score_candidates(query)")) return s;
  if (rc_status s = check_desc(pdesc, P, "rc_score_candidates(pool)")) return s;
  if (mode != RC_SCORE_BLOCK && mode != RC_SCORE_PER_HEAD_ALL)
    return fail(RC_ERR_UNSUPPORTED, "rc_score_candidates: mode %d", mode);
  if (qdesc->n_layers != pdesc->n_layers || qdesc->block_tokens != pdesc->block_tokens ||
      qdesc->n_kv_heads != pdesc->n_kv_heads || qdesc->head_dim != pdesc->head_dim || qdesc->dtype != pdesc->dtype)
    return fail(RC_ERR_INVALID_ARG, "rc_score_candidates: query and pool descriptors differ in more than layer_stride");
  if (C < 0) return fail(RC_ERR_INVALID_ARG, "rc_score_candidates: negative C");
  if (!(tau == tau)) return fail(RC_ERR_INVALID_ARG, "rc_score_candidates: tau is NaN");
  const int H = qdesc->n_kv_heads;
  const int L = qdesc->n_layers;
  if (L == 0 || Q == 0) return RC_OK;
  if (!kq || !vq || !q_ksq || !q_vsq || !best_idx || !best_score || !match_idx)
    return fail(RC_ERR_INVALID_ARG, "rc_score_candidates: NULL query or output pointer");
  if (C > 0 && (!cand || !scores)) return fail(RC_ERR_INVALID_ARG, "rc_score_candidates: NULL cand or scores");
  if (C > 0 && P > 0 && (!kp || !vp || !p_ksq || !p_vsq))
    return fail(RC_ERR_INVALID_ARG, "rc_score_candidates: NULL pool pointer");
  if (!aligned16(kq) || !aligned16(vq) || !aligned16(kp) || !aligned16(vp))
    return fail(RC_ERR_INVALID_ARG, "rc_score_candidates: KV pointer not 16-byte aligned");
  if (C > 0x7fffffffLL || Q > 65535 || L > 65535 || P > 0x7fffffffLL)
    return fail(RC_ERR_UNSUPPORTED, "rc_score_candidates: C, Q or L beyond the grid limits");
  hipStream_t st = static_cast<hipStream_t>(hip_stream);
  const int block_bytes = qdesc->block_tokens * H * qdesc->head_dim * 2;
  if (mode == RC_SCORE_BLOCK && wide_wins((int64_t)L * Q, Q, C, P, block_bytes)) {
    WideParams wp;
    wp.kq = static_cast<const char*>(kq);
    wp.vq = static_cast<const char*>(vq);
    wp.kp = static_cast<const char*>(kp);
    wp.vp = static_cast<const char*>(vp);
    wp.q_ksq = q_ksq;
    wp.q_vsq = q_vsq;
    wp.p_ksq = p_ksq;
    wp.p_vsq = p_vsq;
    wp.live = pool_live;
    wp.cand = cand;
    wp.out = scores;
    wp.best_idx = best_idx;
    wp.best_score = best_score;
    wp.match_idx = match_idx;
    wp.q_lstride_b = qdesc->layer_stride * 2;
    wp.p_lstride_b = pdesc->layer_stride * 2;
    wp.Q = (int)Q;
    wp.P = (int)P;
    wp.C = (int)C;
    wp.L = L;
    wp.G = 1;
    wp.block_bytes = block_bytes;
    set_plan(wp, wide_plan(Q, C, P, L, true));
    wp.tau = tau;
    if (qdesc->dtype == RC_BF16)
      launch_wide<true, false>(wp, st);
    else
      launch_wide<false, false>(wp, st);
    if (rc_status s = check_launch("rc_score_candidates(lists)")) return s;
    if (wp.parts == 1) return RC_OK;
  } else if (C > 0) {
    CandParams cp;
    cp.kq = static_cast<const char*>(kq);
    cp.vq = static_cast<const char*>(vq);
    cp.kp = static_cast<const char*>(kp);
    cp.vp = static_cast<const char*>(vp);
    cp.q_ksq = q_ksq;
    cp.q_vsq = q_vsq;
    cp.p_ksq = p_ksq;
    cp.p_vsq = p_vsq;
    cp.live = pool_live;
    cp.cand = cand;
    cp.scores = scores;
    cp.q_lstride_b = qdesc->layer_stride * 2;
    cp.p_lstride_b = pdesc->layer_stride * 2;
    cp.Q = (int)Q;
    cp.P = (int)P;
    cp.C = (int)C;
    cp.block_bytes = block_bytes;  // T >= 16, Dh = 128: a multiple of 16 KB / 4
    cp.heads = (mode == RC_SCORE_BLOCK) ? 1 : H;
    const bool any_h = mode == RC_SCORE_PER_HEAD_ALL && (16 % H) != 0;  // a thread's chunks wander over the heads
    const int per = cand_per_wg((int64_t)L * Q, C, cp.block_bytes, !any_h);
    const dim3 grid((unsigned)((C + per - 1) / per), (unsigned)Q, (unsigned)L);
    if (qdesc->dtype == RC_BF16)
      launch_candidates<true>(any_h, per, grid, cp, st);
    else
      launch_candidates<false>(any_h, per, grid, cp, st);
    if (rc_status s = check_launch("rc_score_candidates(score)")) return s;
  }
  const long long LQ = (long long)L * Q;
  candidates_select_kernel<<<(unsigned)((LQ + 255) / 256), 256, 0, st>>>(scores, cand, LQ, (int)C, tau, best_idx,
                                                                         best_score, match_idx);
  return check_launch("rc_score_candidates(select)");
}

extern "C" size_t rc_candidate_distances_workspace_size(const rc_kv_desc* qdesc, int64_t Q, int64_t C) {
  using namespace rc;
  if (!qdesc || Q < 0 || C < 0 || qdesc->n_layers <= 0) return 0;
  const int G = cand_layers_per_group(qdesc->n_layers, Q, C);
  const int64_t groups = (qdesc->n_layers + G - 1) / G;
  const int64_t n = groups * Q * C;
  return (size_t)(n > 0 ? n : 1) * sizeof(float);
}

extern "C" rc_status rc_candidate_distances(const rc_kv_desc* qdesc, const rc_kv_desc* pdesc, const void* kq,
                                            const void* vq, int64_t Q, const void* kp, const void* vp, int64_t P,
                                            const uint8_t* pool_live, const int32_t* cand, int64_t C, float threshold,
                                            float* dist, int32_t* best_idx, float* best_dist, int32_t* match_idx,
                                            void* workspace, size_t workspace_bytes, void* hip_stream) {
  using namespace rc;
  clear_error();
  if (rc_status s = check_desc(qdesc, Q, "rc_candidate_distances(query)")) return s;
  if (rc_status s = check_desc(pdesc, P, "rc_candidate_distances(pool)")) return s;
  if (qdesc->n_layers != pdesc->n_layers || qdesc->block_tokens != pdesc->block_tokens ||
      qdesc->n_kv_heads != pdesc->n_kv_heads || qdesc->head_dim != pdesc->head_dim || qdesc->dtype != pdesc->dtype)
    return fail(RC_ERR_INVALID_ARG, "rc_candidate_distances: query and pool descriptors differ in more than layer_stride");
  if (C < 0) return fail(RC_ERR_INVALID_ARG, "rc_candidate_distances: negative C");
  if (!(threshold == threshold)) return fail(RC_ERR_INVALID_ARG, "rc_candidate_distances: threshold is NaN");
  const int L = qdesc->n_layers;
  if (L <= 0) return fail(RC_ERR_INVALID_ARG, "rc_candidate_distances: a mean over %d layers is undefined", L);
  if (Q == 0) return RC_OK;
  if (!kq || !vq || !best_idx || !best_dist || !match_idx)
    return fail(RC_ERR_INVALID_ARG, "rc_candidate_distances: NULL query or output pointer");
  if (C > 0 && (!cand || !dist)) return fail(RC_ERR_INVALID_ARG, "rc_candidate_distances: NULL cand or dist");
  if (C > 0 && P > 0 && (!kp || !vp)) return fail(RC_ERR_INVALID_ARG, "rc_candidate_distances: NULL pool pointer");
  if (!aligned16(kq) || !aligned16(vq) || !aligned16(kp) || !aligned16(vp))
    return fail(RC_ERR_INVALID_ARG, "rc_candidate_distances: KV pointer not 16-byte aligned");
  if (C > 0x7fffffffLL || Q > 65535 || P > 0x7fffffffLL || L > 65535)
    return fail(RC_ERR_UNSUPPORTED, "rc_candidate_distances: C, Q, P or L beyond the grid limits");
  const size_t need = rc_candidate_distances_workspace_size(qdesc, Q, C);
  if (!workspace || workspace_bytes < need || !aligned16(workspace))
    return fail(RC_ERR_WORKSPACE, "rc_candidate_distances: workspace of %zu bytes needed (16-byte aligned), got %zu", need,
                workspace_bytes);
  hipStream_t st = static_cast<hipStream_t>(hip_stream);
  const int G = cand_layers_per_group(L, Q, C);
  const int groups = (L + G - 1) / G;
  float* part = static_cast<float*>(workspace);
  const int block_bytes = qdesc->block_tokens * qdesc->n_kv_heads * qdesc->head_dim * 2;
  if (wide_wins((int64_t)groups * Q, Q, C, P, block_bytes)) {
    WideParams wp = {};
    wp.kq = static_cast<const char*>(kq);
    wp.vq = static_cast<const char*>(vq);
    wp.kp = static_cast<const char*>(kp);
    wp.vp = static_cast<const char*>(vp);
    wp.live = pool_live;
    wp.cand = cand;
    wp.out = part;
    wp.q_lstride_b = qdesc->layer_stride * 2;
    wp.p_lstride_b = pdesc->layer_stride * 2;
    wp.Q = (int)Q;
    wp.P = (int)P;
    wp.C = (int)C;
    wp.L = L;
    wp.G = G;
    wp.block_bytes = block_bytes;
    set_plan(wp, wide_plan(Q, C, P, groups, L % G == 0));
    if (qdesc->dtype == RC_BF16)
      launch_wide<true, true>(wp, st);
    else
      launch_wide<false, true>(wp, st);
    if (rc_status s = check_launch("rc_candidate_distances(lists)")) return s;
  } else if (C > 0 && P > 0) {
    CandDistParams cp;
    cp.kq = static_cast<const char*>(kq);
    cp.vq = static_cast<const char*>(vq);
    cp.kp = static_cast<const char*>(kp);
    cp.vp = static_cast<const char*>(vp);
    cp.live = pool_live;
    cp.cand = cand;
    cp.part = part;
    cp.q_lstride_b = qdesc->layer_stride * 2;
    cp.p_lstride_b = pdesc->layer_stride * 2;
    cp.Q = (int)Q;
    cp.P = (int)P;
    cp.C = (int)C;
    cp.L = L;
    cp.G = G;
    cp.block_bytes = qdesc->block_tokens * qdesc->n_kv_heads * qdesc->head_dim * 2;
    const int per = cand_per_wg((int64_t)groups * Q, C, cp.block_bytes, false);
    const dim3 grid((unsigned)((C + per - 1) / per), (unsigned)Q, (unsigned)groups);
    if (per == kCandFew) {
      if (qdesc->dtype == RC_BF16)
        candidate_distances_kernel<true, kCandFew><<<grid, kCandThreads, 0, st>>>(cp);
      else
        candidate_distances_kernel<false, kCandFew><<<grid, kCandThreads, 0, st>>>(cp);
    } else {
      if (qdesc->dtype == RC_BF16)
        candidate_distances_kernel<true, kCandPerWg><<<grid, kCandThreads, 0, st>>>(cp);
      else
        candidate_distances_kernel<false, kCandPerWg><<<grid, kCandThreads, 0, st>>>(cp);
    }
    if (rc_status s = check_launch("rc_candidate_distances(distances)")) return s;
  }
  const float scale = 1.0f / ((float)L * 2.0f * (float)qdesc->block_tokens * (float)qdesc->n_kv_heads);
  candidate_distances_select_kernel<<<(unsigned)((Q + 3) / 4), 256, 0, st>>>(part, groups, cand, pool_live, (int)Q, (int)P,
                                                                             (int)C, scale, threshold, dist, best_idx,
                                                                             best_dist, match_idx);
  return check_launch("rc_candidate_distances(select)");
}
