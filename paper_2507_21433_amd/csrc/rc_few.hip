// Search of a small problem with few queries (a decoding step of a few requests, a call for one layer): two launches.
// few_shares_kernel multiplies, few_select_kernel adds the shares, forms the scores and selects, with no pass over
// partial results after it.
#include <hip/hip_runtime.h>

#include "rc_common.hpp"
#include "rc_few.hpp"
#include "rc_select.hpp"
#include "rc_tile.hpp"

namespace rc {
namespace {

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

constexpr int kWaves = 4;
constexpr int kRotation = 10;  // slices
constexpr int kRowTiles = kFewRows / 16;  // column tiles of the matrix instruction: 16 pool blocks each
constexpr int kPadRow = kFewRows + 4;     // floats of a query's row in LDS: the four lane groups of a store hit other banks

struct FewParams {
  const char *kq, *vq, *kp, *vp;
  float* dpart;  // [L][S][Q][npt * 64] bare partial dot products
  long long q_lstride_b, p_lstride_b;
  int Q, P, S, npt;
  int row_b;   // bytes of one tensor of a block
  int slices;  // 128-byte slices of a wave, a multiple of the template's U
};

template <bool BF16>
__device__ __forceinline__ f32x4 mfma16(u32x4 a, u32x4 b, f32x4 c) {
  if (BF16)
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
  else
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), c, 0, 0, 0);
}

// A workgroup multiplies 64 pool blocks with all queries over one share of the reduction: half of the shares on the K
// tensor, half on V.  Its four waves take consecutive parts of the share, each straight from memory into registers (lane i
// reads 16 bytes of row i % 16), so that a wave's first loads go out at once and no barrier stands in its way; their sums
// meet in LDS and the share is stored as [query][pool block] floats.  U slices of 128 bytes are loaded while U are
// multiplied.  What bounds it: for a few MB the latency of the loads (so many small workgroups), for more the rate at which
// a compute unit's half-line requests are served; both halves of a line are asked for one after the other and without the
// non-temporal hint (1 x 4096 blocks x 16 queries 76 us with the halves apart, 60 together, 56 without the hint).
// One sequence of instructions per score, whatever the tile: identical pool blocks get identical scores.
template <bool BF16, int TM, int U>
__global__ __launch_bounds__(64 * kWaves, 2) void few_shares_kernel(const FewParams p) {
  __shared__ __attribute__((aligned(16))) float s_red[kWaves][TM * 16][kPadRow];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int share = blockIdx.x % p.S, pt = blockIdx.x / p.S % p.npt;
  const long long l = blockIdx.x / p.S / p.npt;
  const int half = p.S / 2, p0 = pt * kFewRows;
  const bool on_v = share >= half;
  const int part = (on_v ? share - half : share) * kWaves + wave, first = part * p.slices;
  const char* pool = (on_v ? p.vp : p.kp) + l * p.p_lstride_b + (long long)p0 * p.row_b;
  const char* query = (on_v ? p.vq : p.kq) + l * p.q_lstride_b;
  // rows past the last block fall outside the descriptors and read as zeros
  const __amdgpu_buffer_rsrc_t rp = __builtin_amdgcn_make_buffer_rsrc((void*)pool, 0, min(kFewRows, p.P - p0) * p.row_b, 0x00020000);
  const __amdgpu_buffer_rsrc_t rq = __builtin_amdgcn_make_buffer_rsrc((void*)query, 0, p.Q * p.row_b, 0x00020000);
  const int voff = (lane & 15) * p.row_b + (lane >> 4) * 16;

  u32x4 a[2][U][2][TM], b[2][U][2][kRowTiles];
  auto load = [&](int buf, int slice) __attribute__((always_inline)) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
#pragma unroll
      for (int t = 0; t < kRowTiles; ++t)
#pragma unroll
        for (int h = 0; h < 2; ++h)
          b[buf][u][h][t] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(rp, voff + u * 128 + h * 64, slice * 128 + t * 16 * p.row_b, 0));
#pragma unroll
      for (int m = 0; m < TM; ++m)
#pragma unroll
        for (int h = 0; h < 2; ++h)
          a[buf][u][h][m] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(rq, voff + u * 128 + h * 64, slice * 128 + m * 16 * p.row_b, 0));
    }
  };
  f32x4 acc[TM][kRowTiles];
#pragma unroll
  for (int m = 0; m < TM; ++m)
#pragma unroll
    for (int t = 0; t < kRowTiles; ++t) acc[m][t] = {0.f, 0.f, 0.f, 0.f};
  auto multiply = [&](int buf) __attribute__((always_inline)) {
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int t = 0; t < kRowTiles; ++t)
#pragma unroll
          for (int m = 0; m < TM; ++m) acc[m][t] = mfma16<BF16>(a[buf][u][h][m], b[buf][u][h][t], acc[m][t]);
  };
  // A wave walks its slices from here on and around, the same for every tile: the waves' parts are a power of two of KB
  // apart, and started at their first slices they would all ask the same memory channels at the same time (10 x 754 blocks
  // of 32 KB, 3 queries, 2 shares: 62 -> 53 us).
  int at = part * kRotation % p.slices / U * U;
  auto load_next = [&](int buf) __attribute__((always_inline)) {
    load(buf, first + at);
    at = at + U == p.slices ? 0 : at + U;
  };
  load_next(0);
  int s = U;
  for (; s + U < p.slices; s += 2 * U) {
    load_next(1);
    __builtin_amdgcn_sched_barrier(0);
    multiply(0);
    __builtin_amdgcn_sched_barrier(0);
    load_next(0);
    __builtin_amdgcn_sched_barrier(0);
    multiply(1);
    __builtin_amdgcn_sched_barrier(0);
  }
  if (s < p.slices) {
    load_next(1);
    __builtin_amdgcn_sched_barrier(0);
    multiply(0);
    multiply(1);
  } else {
    multiply(0);
  }

  // the four waves' parts, added in wave order
#pragma unroll
  for (int m = 0; m < TM; ++m)
#pragma unroll
    for (int t = 0; t < kRowTiles; ++t)
#pragma unroll
      for (int r = 0; r < 4; ++r) s_red[wave][m * 16 + 4 * (lane >> 4) + r][t * 16 + (lane & 15)] = acc[m][t][r];
  __syncthreads();
  float* out = p.dpart + ((l * p.S + share) * p.Q * p.npt + pt) * (long long)kFewRows;
#pragma unroll
  for (int i = tid; i < TM * 16 * kFewRows / 4; i += 64 * kWaves) {
    const int q = i / (kFewRows / 4), c = i % (kFewRows / 4) * 4;
    if (q >= p.Q) break;
    f32x4 sum = *reinterpret_cast<const f32x4*>(&s_red[0][q][c]);
#pragma unroll
    for (int w = 1; w < kWaves; ++w) sum += *reinterpret_cast<const f32x4*>(&s_red[w][q][c]);
    *reinterpret_cast<f32x4*>(out + (long long)q * p.npt * kFewRows + c) = sum;
  }
}

// ---- per-head score

// A workgroup scores 64 pool blocks against up to 32 queries on one head: K, rescale, V, one chain of the
// matrix instructions of the tile kernels in their order, so that a pair reports the same bits here and there.  What a small
// call waits for is the length of that chain, a step of 64 elements after the other, and the instructions a wave has to issue
// per step: two waves only load (straight to LDS, eight rows of a 128-byte line at a time, rows XOR-swizzled as in the tile
// kernels), two only read fragments and multiply (2 x 361 blocks of 8 heads, 3 queries: 22 us, 24 with every wave doing both;
// 61 x 690 x 2 514 and 536).  Six stages of 12 KB, two workgroups per compute unit: four stages and three 519, seven and one
// 564.
constexpr int kHeadThreads = 256, kHeadQueries = 32, kHeadLoaders = 128, kHeadStages = 6;
struct HeadParams {
  const char *kq, *vq, *kp, *vp;
  const float *q_ksq, *q_vsq, *p_ksq, *p_vsq;
  float* dpart;  // [L][H][Q][npt * 64] scores of a head
  long long q_lstride_b, p_lstride_b;
  int Q, P, T, H, npt;
};

template <bool BF16>
__global__ __launch_bounds__(kHeadThreads, 1) void head_shares_kernel(const HeadParams p) {
#if defined(__HIP_DEVICE_COMPILE__)  // the host pass only needs the launch stub
  constexpr int kRows = kFewRows + kHeadQueries, kStage = kRows * kRowBytes;
  constexpr int kLoadsA = kFewRows * 8 / kHeadLoaders, kLoadsB = kHeadQueries * 8 / kHeadLoaders, kLoads = kLoadsA + kLoadsB;
  constexpr int kInFlight = kHeadStages - 1;  // steps
  static_assert(kLoads * kInFlight <= 63 && kInFlight <= 32, "the counter of outstanding loads has six bits; a tensor has 32 steps at least");
  __shared__ __attribute__((aligned(1024))) char s_ring[kHeadStages * kStage];
  const uint32_t ring = lds_offset(s_ring);
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int head = blockIdx.x % p.H, pt = blockIdx.x / p.H % p.npt;
  const long long l = blockIdx.x / p.H / p.npt;
  const int p0 = pt * kFewRows;
  const int row_b = p.T * p.H * 256, tok = p.H * 256;

  const int sps = p.T * 2;  // steps of a tensor: two lines per token
  if (wave >= 2) {
    // ---- the loading waves.  Rows past the last block fall outside the descriptors and read as zeros.
    const int lt = tid - kHeadLoaders;
    const long long poff = l * p.p_lstride_b + (long long)p0 * row_b, qoff = l * p.q_lstride_b;
    const uint32_t prange = (uint32_t)(min(kFewRows, p.P - p0) * row_b), qrange = (uint32_t)(p.Q * row_b);
    const uint32_t voff = (uint32_t)(lt >> 3) * (uint32_t)row_b + (uint32_t)(((lt & 7) ^ ((lt >> 3) & 7)) * 16);
    const uint32_t first_dst = ring + (uint32_t)((wave - 2) * 1024);
    uint32_t dst = first_dst;
    auto load = [&](const i32x4& srdA, const i32x4& srdB, int u) __attribute__((always_inline)) {
      const uint32_t src = (uint32_t)(head * 256 + (u >> 1) * tok + (u & 1) * 128);
#pragma unroll
      for (int j = 0; j < kLoadsB; ++j) dma16<false>(srdB, voff, src + (uint32_t)(j * 16 * row_b), dst + (uint32_t)((kLoadsA + j) * kHeadLoaders * 16));
#pragma unroll
      for (int j = 0; j < kLoadsA; ++j) dma16<true>(srdA, voff, src + (uint32_t)(j * 16 * row_b), dst + (uint32_t)(j * kHeadLoaders * 16));
      dst = dst + kStage == first_dst + kHeadStages * kStage ? first_dst : dst + kStage;
    };
    // a step's loads go out when every wave has met at the step kInFlight before it: the stage it overwrites has been read
    auto step = [&](const i32x4& srdA, const i32x4& srdB, int u) __attribute__((always_inline)) {
      asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"(kLoads * (kInFlight - 1)) : "memory");
      load(srdA, srdB, u);
    };
    {
      const i32x4 srdA = make_srd(p.kp + poff, prange), srdB = make_srd(p.kq + qoff, qrange);
#pragma unroll
      for (int u = 0; u < kInFlight; ++u) load(srdA, srdB, u);
      for (int u = kInFlight; u < sps; ++u) step(srdA, srdB, u);
    }
    {
      const i32x4 srdA = make_srd(p.vp + poff, prange), srdB = make_srd(p.vq + qoff, qrange);
      for (int u = 0; u < sps; ++u) step(srdA, srdB, u);
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
#pragma unroll
    for (int i = 0; i < kInFlight; ++i) __builtin_amdgcn_s_barrier();
    return;
  }

  // ---- the multiplying waves, 32 pool blocks each
  const int col = p0 + wave * 32 + (lane & 31);
  float rp, fp, rq[16], fq[16];
  {
    const long long o = (l * p.P + min(col, p.P - 1)) * p.H + head;
    norm_factors(p.p_ksq[o], p.p_vsq[o], rp, fp);
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int q = min(8 * (r >> 2) + 4 * (lane >> 5) + (r & 3), p.Q - 1);
      const long long oq = (l * p.Q + q) * p.H + head;
      float av;
      norm_factors(p.q_ksq[oq], p.q_vsq[oq], rq[r], av);
      fq[r] = 0.5f * av;
    }
  }
  f32x16 acc;
#pragma unroll
  for (int r = 0; r < 16; ++r) acc[r] = 0.f;
  // fragment reads: row lane % 32 of the queries (rows of the matrix instruction) and of the wave's pool blocks (its columns),
  // logical chunk 2 * kk + lane / 32
  uint32_t frag[4];
#pragma unroll
  for (int kk = 0; kk < 4; ++kk)
    frag[kk] = (uint32_t)(lane & 31) * kRowBytes + ((((uint32_t)(2 * kk) + (uint32_t)(lane >> 5)) ^ (uint32_t)(lane & 7)) * 16);
  const char* stage = s_ring;
  uint4 a[2][4], b[2][4];  // fragments of a step, read while the step before is multiplied
  auto multiply = [&](int buf) __attribute__((always_inline)) {
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) acc = mfma<BF16>(a[buf][kk], b[buf][kk], acc);
    __builtin_amdgcn_sched_barrier(0);
  };
  auto step = [&](int buf) __attribute__((always_inline)) {
    // the fragments of the step before are in registers: its stage may be overwritten
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) {
      a[buf][kk] = *reinterpret_cast<const uint4*>(stage + kFewRows * kRowBytes + frag[kk]);
      b[buf][kk] = *reinterpret_cast<const uint4*>(stage + wave * 32 * kRowBytes + frag[kk]);
    }
    stage = stage + kStage == s_ring + kHeadStages * kStage ? s_ring : stage + kStage;
    __builtin_amdgcn_sched_barrier(0);
    multiply(buf ^ 1);
  };
  auto tensor = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) a[1][kk] = b[1][kk] = make_uint4(0, 0, 0, 0);  // nothing to multiply in the first step
    for (int u = 0; u < sps; u += 2) {  // an even number
      step(0);
      step(1);
    }
    multiply(1);
  };
  tensor();
#pragma unroll
  for (int r = 0; r < 16; ++r) acc[r] *= rq[r] * rp;
  tensor();
  const int width = p.npt * kFewRows;
  float* out = p.dpart + (l * p.H + head) * p.Q * (long long)width + col;
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const int q = 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
    if (q < p.Q) out[(long long)q * width] = acc[r] * (fq[r] * fp);
  }
#endif
}

constexpr int kSelWaves = 16;

// One workgroup per query (and layer, unless MEAN) adds the shares in a fixed order, forms the cosine or the distance from
// the cached norms, masks dead blocks and selects; no partial results go through memory.  Bound by round trips: a query's
// shares of 256 blocks are 64 KB at most.  `pw` waves stand side by side along the pool (256 blocks each), the
// other factor of the 16 takes turns with the shares (MEAN: with the 2 L distances of a pair, layer by layer, K before V).
// HEADS: the shares are the scores of the S heads, each put on the grid of 1/32767 and the least of them taken, as the
// selection of the tile kernels' shares does.
enum class Few { kCosine, kMean, kHeads };
template <Few MODE>
__global__ __launch_bounds__(64 * kSelWaves) void few_select_kernel(
    const float* __restrict__ dpart, int S, int L, int Q, int P, int npt, int pw, float scale, const float* __restrict__ q_ksq,
    const float* __restrict__ q_vsq, const float* __restrict__ p_ksq, const float* __restrict__ p_vsq,
    const uint8_t* __restrict__ live, float threshold, int32_t* __restrict__ best_idx, float* __restrict__ best_value,
    int32_t* __restrict__ match_idx, float* __restrict__ second_value) {
  constexpr bool MEAN = MODE == Few::kMean, HEADS = MODE == Few::kHeads, TWO = MODE == Few::kCosine;
  __shared__ f32x4 s_sum[TWO ? 2 : 1][kSelWaves][64];
  __shared__ float s_best[kSelWaves], s_second[kSelWaves];
  __shared__ int s_idx[kSelWaves];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int along = wave % pw, turn = wave / pw, turns = kSelWaves / pw;
  const int q = blockIdx.x;
  const long long l0 = MEAN ? 0 : blockIdx.y;
  const int half = S / 2, width = npt * kFewRows;
  const long long share_stride = (long long)Q * width;
  const float* src0 = dpart + (l0 * S * Q + q) * (long long)width;
  if (live) live += l0 * P;
  float best = -INFINITY, second = -INFINITY;
  int bidx = -1;
  for (int base = 0; base < P; base += 256 * pw) {
    const int pp = base + along * 256 + lane * 4;
    f32x4 sk = {0.f, 0.f, 0.f, 0.f}, sv = {0.f, 0.f, 0.f, 0.f};
    f32x4 nk = {0.f, 0.f, 0.f, 0.f}, nv = {0.f, 0.f, 0.f, 0.f};
    i32x4 least = {32767, 32767, 32767, 32767};
    unsigned alive = 0;
    if (pp < width) {
      if (turn == 0) {  // what the selection needs is on its way while the shares are added
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int pe = min(pp + e, P - 1);
          if (TWO) {
            nk[e] = p_ksq[l0 * P + pe];
            nv[e] = p_vsq[l0 * P + pe];
          }
          alive |= (unsigned)(pp + e < P && (!live || live[pe])) << e;
        }
      }
      if (HEADS) {
#pragma unroll 4
        for (int s = turn; s < S; s += turns) {
          const f32x4 v = __builtin_nontemporal_load(reinterpret_cast<const f32x4*>(src0 + s * share_stride + pp));
#pragma unroll
          for (int e = 0; e < 4; e += 2) {
            const i16x2 g = quantise_pair(v[e], v[e + 1]);
            least[e] = min(least[e], (int)g[0]);
            least[e + 1] = min(least[e + 1], (int)g[1]);
          }
        }
      } else if (!MEAN) {
#pragma unroll 4
        for (int s = turn; s < half; s += turns) {
          sk += __builtin_nontemporal_load(reinterpret_cast<const f32x4*>(src0 + s * share_stride + pp));
          sv += __builtin_nontemporal_load(reinterpret_cast<const f32x4*>(src0 + (half + s) * share_stride + pp));
        }
      } else {
        const int i0 = (int)(2LL * L * turn / turns), i1 = (int)(2LL * L * (turn + 1) / turns);
        for (int i = i0; i < i1; ++i) {
          const long long l = i >> 1;
          const int v = i & 1;
          const float* src = src0 + (l * S + v * half) * share_stride + pp;
          const float nq = (v ? q_vsq : q_ksq)[l * Q + q];
          const float* np = (v ? p_vsq : p_ksq) + l * P;
          f32x4 n, dot = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
          for (int e = 0; e < 4; ++e) n[e] = nq + np[min(pp + e, P - 1)];
#pragma unroll 8
          for (int s = 0; s < half; ++s) dot += __builtin_nontemporal_load(reinterpret_cast<const f32x4*>(src + s * share_stride));
#pragma unroll
          for (int e = 0; e < 4; ++e) sk[e] += __builtin_amdgcn_sqrtf(fmaxf(fmaf(-2.f, dot[e], n[e]), 0.f));
        }
      }
    }
    if (turns > 1) {
      s_sum[0][wave][lane] = HEADS ? __builtin_bit_cast(f32x4, least) : sk;
      if (TWO) s_sum[TWO ? 1 : 0][wave][lane] = sv;
      __syncthreads();
      if (turn == 0)
        for (int t = 1; t < turns; ++t) {
          if (HEADS) {
            const i32x4 other = __builtin_bit_cast(i32x4, s_sum[0][t * pw + along][lane]);
#pragma unroll
            for (int e = 0; e < 4; ++e) least[e] = min(least[e], other[e]);
          } else {
            sk += s_sum[0][t * pw + along][lane];
          }
          if (TWO) sv += s_sum[TWO ? 1 : 0][t * pw + along][lane];
        }
    }
    if (turn == 0 && pp < width) {
      float aq = 0.f, vq = 0.f;
      if (TWO) {
        const float ksq = q_ksq[l0 * Q + q], vsq = q_vsq[l0 * Q + q];
        aq = ksq > 0.f ? 0.5f * __builtin_amdgcn_rsqf(ksq) : 0.f;  // a zero norm: cosine 0
        vq = vsq > 0.f ? 0.5f * __builtin_amdgcn_rsqf(vsq) : 0.f;
      }
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        float v;
        if (HEADS) {
          v = (float)least[e] / 32767.f;
        } else if (MEAN) {
          v = -(sk[e] * scale);
        } else {
          const float ap = nk[e] > 0.f ? __builtin_amdgcn_rsqf(nk[e]) : 0.f, vp = nv[e] > 0.f ? __builtin_amdgcn_rsqf(nv[e]) : 0.f;
          v = sk[e] * (aq * ap) + sv[e] * (vq * vp);
        }
        if (alive >> e & 1) top2_push(v, pp + e, best, bidx, second);
      }
    }
    if (turns > 1) __syncthreads();  // the sums are read before the next round writes them
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1)
    top2_merge(best, bidx, second, __shfl_xor(best, off), __shfl_xor(bidx, off), __shfl_xor(second, off));
  if (lane == 0) {
    s_best[wave] = best;
    s_idx[wave] = bidx;
    s_second[wave] = second;
  }
  __syncthreads();
  if (threadIdx.x != 0) return;
  for (int w = 1; w < pw; ++w) top2_merge(best, bidx, second, s_best[w], s_idx[w], s_second[w]);
  const long long o = l0 * Q + q;
  const float value = MEAN ? -best : best;
  best_idx[o] = bidx;
  best_value[o] = value;
  match_idx[o] = (bidx >= 0 && (MEAN ? value <= threshold : value >= threshold)) ? bidx : -1;
  if (second_value) second_value[o] = MEAN ? -second : second;
}

// waves of the selection side by side along the pool
inline int select_waves(int64_t P) {
  int pw = 1;
  while (pw < kSelWaves && pw * 256 < P) pw *= 2;
  return pw;
}

template <bool BF16, int U>
void launch_shares(const FewParams& fp, unsigned wgs, hipStream_t st) {
  if (fp.Q <= 16)
    few_shares_kernel<BF16, 1, U><<<wgs, 64 * kWaves, 0, st>>>(fp);
  else if (fp.Q <= 32)
    few_shares_kernel<BF16, 2, U><<<wgs, 64 * kWaves, 0, st>>>(fp);
  else
    few_shares_kernel<BF16, 4, 1><<<wgs, 64 * kWaves, 0, st>>>(fp);
}

}  // namespace

// Which calls come here, and how many shares they take.  These kernels have less than half the fixed time of the ring
// pipeline (a wave's first loads are its own, nothing waits for a barrier) but ask for a block's line in two halves, and
// reach 5.3 TB/s where the ring reaches 6.8; and the selection takes a workgroup per row of shares, of each query and layer
// (block score), or walks all layers of a query (layer mean).  So the lines are drawn by the size of the pool's blocks, in
// bytes, by query count, and by what makes the other side slow: few rows to select from, or, for the layer mean, a pool of so few
// tiles of 256 blocks per layer that the ring shares them out.  Measured over 2858 shapes, ring pipeline -> these kernels, us per call:
//   block score  1 x 256 x 32 queries 30 -> 12, 3 x 659 x 3 47 -> 31, 1 x 4096 x 16 (268 MB) 61 -> 58, 1 x 8192 x 16 98 -> 107;
//                7 x 310 x 24 (142 MB) 45 -> 37, 16 x 1000 x 24 (1.0 GB) 176 -> 198;
//                2 x 1015 x 57 (133 MB) 47 -> 40, 14 x 208 x 44 (239 MB) 65 -> 82
//                layers x queries: 32 x 190 x 16 35 -> 30, 64 x 95 x 16 36 -> 43; 32 x 190 x 20 35 -> 34, 32 x 190 x 32 37 -> 40;
//                16 x 94 x 34 51 -> 46, 32 x 114 x 34 31 -> 39, 64 x 95 x 64 43 -> 100
//   layer mean   6 x 148 x 3 44 -> 15, 47 x 215 x 1 (331 MB) 208 -> 71, 16 x 934 x 6 (980 MB) 222 -> 188; of longer pools
//                2 x 2670 x 16 (350 MB) 90 -> 85, 2 x 3814 x 6 (500 MB) 109 -> 116, 16 x 7476 x 16 (980 MB) 196 -> 245;
//                33 x 132 x 21 (357 MB) 178 -> 104, 2 x 15258 x 32 (500 MB) 110 -> 127, 3 x 10303 x 24 (1.0 GB) 195 -> 206;
//                46 x 167 x 37 (503 MB) 200 -> 144, 2 x 7476 x 64 (490 MB) 107 -> 147
// Of the 2402 shapes that come here, 33 are more than 3 % slower than with the ring pipeline, by 6 % on average.
// Shares: the number with the lowest estimate in us, rounds of one workgroup per compute unit (an MI355X has 256) times
// the slices of a share times the time of a slice, and 3 ns per workgroup for storing and adding its share.  Within 2 % of
// the best number on average over those shapes.
int few_shares(bool layer_mean, int64_t L, int64_t P, int64_t Q, int T, int H) {
  if (L < 1 || L > 65535 || P < 1 || Q < 1 || Q > kFewQueries) return 0;
  const double mb = (double)L * (double)P * (double)(T * H) * 512e-6;
  const int by_queries = Q <= 16 ? 0 : Q <= 32 ? 1 : 2;
  constexpr double most_mb[2][3] = {{256.0, 200.0, 150.0}, {1000.0, 600.0, 500.0}};
  if (mb > most_mb[layer_mean][by_queries]) return 0;
  if (layer_mean) {
    constexpr double any_mb[3] = {400.0, 350.0, 200.0};
    constexpr int64_t most_blocks[3] = {2048, 1024, 512};
    if (mb > any_mb[by_queries] && (P > most_blocks[by_queries] || L * ((P + 255) / 256) > 160)) return 0;
  } else if (L * Q > (by_queries < 2 ? 768 : 640)) {
    return 0;
  }
  constexpr double slice_us[3] = {0.21, 0.27, 0.42};
  const int64_t tiles = L * ((P + kFewRows - 1) / kFewRows);
  const int units = T * H * 2 / kWaves;  // slices of a tensor that a wave of a single share walks
  int best = 0;
  double best_us = 0.0;
  for (int half = 1; half <= units; ++half) {
    if (units % half != 0) continue;
    const int64_t wgs = tiles * 2 * half;
    if (half > 1 && wgs > 16384) break;
    const double us = (double)((wgs + 255) / 256) * (double)(kWaves * units / half) * slice_us[by_queries] + 0.003 * (double)wgs;
    if (best == 0 || us < best_us) {
      best = 2 * half;
      best_us = us;
    }
  }
  return best;
}

rc_status few_search(const FewArgs& a, int S, bool layer_mean, const char* who) {
  hipStream_t st = static_cast<hipStream_t>(a.hip_stream);
  const int L = a.qdesc->n_layers, T = a.qdesc->block_tokens, H = a.qdesc->n_kv_heads;
  FewParams fp;
  fp.kq = static_cast<const char*>(a.kq);
  fp.vq = static_cast<const char*>(a.vq);
  fp.kp = static_cast<const char*>(a.kp);
  fp.vp = static_cast<const char*>(a.vp);
  fp.dpart = static_cast<float*>(a.workspace);
  fp.q_lstride_b = a.qdesc->layer_stride * 2;
  fp.p_lstride_b = a.pdesc->layer_stride * 2;
  fp.Q = (int)a.Q;
  fp.P = (int)a.P;
  fp.S = S;
  fp.npt = (int)((a.P + kFewRows - 1) / kFewRows);
  fp.row_b = T * H * 256;
  fp.slices = T * H * 2 / (S / 2) / kWaves;
  const unsigned wgs = (unsigned)(L * fp.npt * S);
  const bool bf = a.qdesc->dtype == RC_BF16;
  if (fp.slices % 2 == 0) {
    if (bf) launch_shares<true, 2>(fp, wgs, st); else launch_shares<false, 2>(fp, wgs, st);
  } else {
    if (bf) launch_shares<true, 1>(fp, wgs, st); else launch_shares<false, 1>(fp, wgs, st);
  }
  if (rc_status s = check_launch(who)) return s;
  const int pw = select_waves(a.P);
  if (layer_mean) {
    const float scale = 1.0f / ((float)L * 2.0f * (float)T * (float)H);
    few_select_kernel<Few::kMean><<<dim3((unsigned)a.Q), 64 * kSelWaves, 0, st>>>(
        fp.dpart, S, L, fp.Q, fp.P, fp.npt, pw, scale, a.q_ksq, a.q_vsq, a.p_ksq, a.p_vsq, a.live, a.threshold, a.best_idx,
        a.best_value, a.match_idx, a.second_value);
  } else {
    few_select_kernel<Few::kCosine><<<dim3((unsigned)a.Q, (unsigned)L), 64 * kSelWaves, 0, st>>>(
        fp.dpart, S, L, fp.Q, fp.P, fp.npt, pw, 1.0f, a.q_ksq, a.q_vsq, a.p_ksq, a.p_vsq, a.live, a.threshold, a.best_idx,
        a.best_value, a.match_idx, a.second_value);
  }
  return check_launch(who);
}

// Which per-head calls come here.  A share per head and tile of 64 blocks, not of 256, spreads over the chip where the tile
// kernels' shares do not; more queries are loaded by more workgroups, and a round of the tile kernels that is nearly full
// leaves nothing to gain.  Measured over 130 shapes (us per call, tile kernels -> these; the scores' bits are the same):
//   up to 3 queries    2 x 361 blocks x 3 71 -> 22, 47 x 293 x 2 217 -> 149, 62 x 1066 x 2 (5.4 GB) 989 -> 799
//   up to 8 queries    55 x 258 x 5 (128-KB tensors) 917 -> 606, 4 x 3583 x 7 246 -> 188, 50 x 2269 x 4 (7.4 GB) 1189 -> 1165
//   up to 16 queries   20 x 260 x 12 244 -> 136, 12 x 1851 x 8 335 -> 289, 15 x 1288 x 9 (2.5 GB) 509 -> 419, 8 x 8093 x 15 (4.2 GB) 630 -> 736
//   up to 32 queries   1 x 577 x 30 (80 workgroups) 71 -> 26, 14 x 208 x 23 (560) 75 -> 66, 30 x 700 x 30 (2640) 271 -> 286
//   209 to 256 shares of the tile kernels: 62 x 130 x 4, 4 heads 107 -> 115, 62 x 70 x 16 51 -> 58;  145 and more, from 17 queries
//   on: 46 x 83 x 29, 4 heads (184) 87 -> 112, 48 x 121 x 32 (192) 62 -> 75 - but 48 x 57 x 32 (192), where three quarters of
//   a share are padding 83 -> 71
//   blocks of 32 tokens of two heads (rows of 16 KB, a head every 512 bytes): 1 x 9155 x 12 (300 MB) 1.29 times as fast, 1 x 18 310 x 12
//   (600 MB) 0.93, 1 x 51 879 x 10 (1.7 GB) 290 -> 360; with 1, 3, 4, 6 and 8 heads 1.05 to 1.22 there
bool few_heads(int64_t L, int64_t P, int64_t Q, int T, int H) {
  if (L < 1 || L > 65535 || P < 1 || Q < 1 || Q > kHeadQueries) return false;
  const double mb = (double)L * (double)P * (double)(T * H) * 512e-6;
  if (mb > 6000.0 || few_bytes(H, L, P, Q) > ((size_t)512 << 20)) return false;
  const int64_t tile_shares = L * ((P + 255) / 256) * H;
  if (tile_shares > (Q > 16 && P > kFewRows ? 144 : 208) && tile_shares <= 256) return false;
  if (T == 32 && H == 2 && mb > 500.0) return false;
  if (Q <= 8) return Q <= 3 || mb <= 3000.0;
  return Q <= 16 ? mb <= 2500.0 : L * ((P + kFewRows - 1) / kFewRows) * H <= 512;
}

rc_status few_search_heads(const FewArgs& a, const char* who) {
  hipStream_t st = static_cast<hipStream_t>(a.hip_stream);
  const int L = a.qdesc->n_layers;
  HeadParams hp;
  hp.kq = static_cast<const char*>(a.kq);
  hp.vq = static_cast<const char*>(a.vq);
  hp.kp = static_cast<const char*>(a.kp);
  hp.vp = static_cast<const char*>(a.vp);
  hp.q_ksq = a.q_ksq;
  hp.q_vsq = a.q_vsq;
  hp.p_ksq = a.p_ksq;
  hp.p_vsq = a.p_vsq;
  hp.dpart = static_cast<float*>(a.workspace);
  hp.q_lstride_b = a.qdesc->layer_stride * 2;
  hp.p_lstride_b = a.pdesc->layer_stride * 2;
  hp.Q = (int)a.Q;
  hp.P = (int)a.P;
  hp.T = a.qdesc->block_tokens;
  hp.H = a.qdesc->n_kv_heads;
  hp.npt = (int)((a.P + kFewRows - 1) / kFewRows);
  const unsigned wgs = (unsigned)((int64_t)L * hp.npt * hp.H);
  const bool bf = a.qdesc->dtype == RC_BF16;
  if (bf)
    head_shares_kernel<true><<<wgs, kHeadThreads, 0, st>>>(hp);
  else
    head_shares_kernel<false><<<wgs, kHeadThreads, 0, st>>>(hp);
  if (rc_status s = check_launch(who)) return s;
  few_select_kernel<Few::kHeads><<<dim3((unsigned)a.Q, (unsigned)L), 64 * kSelWaves, 0, st>>>(
      hp.dpart, hp.H, L, hp.Q, hp.P, hp.npt, select_waves(a.P), 1.0f, nullptr, nullptr, nullptr, nullptr, a.live, a.threshold,
      a.best_idx, a.best_value, a.match_idx, a.second_value);
  return check_launch(who);
}

}  // namespace rc
