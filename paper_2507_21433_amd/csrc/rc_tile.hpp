// What the search kernels share: the matrix instruction, the norms' factors, loads from memory straight into LDS.
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>

namespace rc {
namespace {

typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef int i32x4 __attribute__((ext_vector_type(4)));
typedef short i16x2 __attribute__((ext_vector_type(2)));

// Two scores in [-1, 1] onto the grid of 1/32767 (signed normalised 16 bit, round to nearest).  The
// per-head-all mode keeps its minimum over heads on this grid; both of its paths call this.
__device__ __forceinline__ i16x2 quantise_pair(float a, float b) { return __builtin_amdgcn_cvt_pknorm_i16(a, b); }

constexpr int kBK = 64;             // reduction elements per pipeline step
constexpr int kRowBytes = kBK * 2;  // bytes of one block's slice in LDS (one 128-byte line)

template <bool BF16>
__device__ __forceinline__ f32x16 mfma(uint4 a, uint4 b, f32x16 c) {
  if (BF16)
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
  else
    return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), c, 0, 0, 0);
}

// From the squared norms of a block's K and V tensors: ratio = aK/aV and av = aV with
// a = 1/sqrt(squared norm).  A zero K norm gives aK = 0 (cosine defined as 0); a zero V norm
// gives aV = 1, which is harmless because every V dot product of that block is 0 as well.
// v_rsq_f32 is good to 1 ulp; the scores only need 2e-3.
__device__ __forceinline__ void norm_factors(float ksq, float vsq, float& ratio, float& av) {
  const float ak = ksq > 0.f ? __builtin_amdgcn_rsqf(ksq) : 0.f;
  av = vsq > 0.f ? __builtin_amdgcn_rsqf(vsq) : 1.f;
  const float inv_av = vsq > 0.f ? vsq * av : 1.f;  // sqrt(vsq)
  ratio = ak * inv_av;
}

// Raw buffer descriptor (base, no stride, byte range, 32-bit raw data format) in scalar registers.
__device__ __forceinline__ i32x4 make_srd(const void* base, uint32_t bytes) {
  const unsigned long long a = (unsigned long long)base;
  i32x4 r;
  r[0] = __builtin_amdgcn_readfirstlane((int)(uint32_t)a);
  r[1] = __builtin_amdgcn_readfirstlane((int)((a >> 32) & 0xffffu));
  r[2] = __builtin_amdgcn_readfirstlane((int)bytes);
  r[3] = 0x00020000;
  return r;
}

// 16 bytes per lane, global -> LDS without passing through registers: lane l lands at LDS byte
// lds_base + 16*l.  Completion is counted by vmcnt, in issue order.  Written as asm so that the
// pipeline's waits are exactly the ones placed by hand below.
// STREAM marks the load non-temporal: the pool slices are read once (or by the few query tiles of
// the same pool tile, close together in time), so they should not displace the query slices that
// every pool tile of the layer re-reads from the L2.  Measured: 2.5 % on cfg2, 1.5 % on cfg3.
template <bool STREAM>
__device__ __forceinline__ void dma16(i32x4 srd, uint32_t voff, uint32_t soff, uint32_t lds_base) {
  // the descriptor, the scalar offset and the LDS base are the same for the whole wave
  srd[0] = __builtin_amdgcn_readfirstlane(srd[0]);
  srd[1] = __builtin_amdgcn_readfirstlane(srd[1]);
  srd[2] = __builtin_amdgcn_readfirstlane(srd[2]);
  srd[3] = __builtin_amdgcn_readfirstlane(srd[3]);
  soff = __builtin_amdgcn_readfirstlane(soff);
  lds_base = __builtin_amdgcn_readfirstlane(lds_base);
  if (STREAM)
    asm volatile("s_mov_b32 m0, %3\n\ts_nop 0\n\tbuffer_load_dwordx4 %0, %1, %2 offen nt lds"
                 :
                 : "v"(voff), "s"(srd), "s"(soff), "s"(lds_base)
                 : "memory", "m0");
  else
    asm volatile("s_mov_b32 m0, %3\n\ts_nop 0\n\tbuffer_load_dwordx4 %0, %1, %2 offen lds"
                 :
                 : "v"(voff), "s"(srd), "s"(soff), "s"(lds_base)
                 : "memory", "m0");
}

__device__ __forceinline__ uint32_t lds_offset(const void* p) {
  return (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) char*)p;
}

}  // namespace
}  // namespace rc
