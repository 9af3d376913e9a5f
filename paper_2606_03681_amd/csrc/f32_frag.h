// Helpers of the float32-arithmetic kernels: the fp32 matrix-core product and pieces of four values.
//
// v_mfma_f32_16x16x4_f32 (float32 operands and accumulators; 157 TFLOP/s, as much as the vector
// unit's FMAs could reach with every slot filled).  Lane layout, with g = lane / 16 and
// c = lane % 16:
//   A (16 x 4): lane holds A[c][g];  B (4 x 16): lane holds B[g][c];
//   D (16 x 16): lane holds D[4g .. 4g+3][c].
// Any bijection between the contraction index and (instruction, g) that A and B share gives the
// same product, which the kernels use to read operands 16 bytes per lane and, in the attention
// kernels, to feed a D tile straight back in as a B operand.
#pragma once

#include "mfma.h"

namespace tfm {

__device__ __forceinline__ f32x4 mfma32(float a, float b, const f32x4& c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// Four consecutive values of either storage type.
__device__ __forceinline__ float4 ld4(const float* p) {
  return *reinterpret_cast<const float4*>(p);
}
__device__ __forceinline__ float4 ld4(const bf16* p) {
  const uint2 u = *reinterpret_cast<const uint2*>(p);
  return make_float4(__uint_as_float(u.x << 16), __uint_as_float(u.x & 0xffff0000u),
                     __uint_as_float(u.y << 16), __uint_as_float(u.y & 0xffff0000u));
}
__device__ __forceinline__ void st4(float* p, const float4& v) {
  *reinterpret_cast<float4*>(p) = v;
}
__device__ __forceinline__ void st4(bf16* p, const float4& v) {
  *reinterpret_cast<uint2*>(p) = make_uint2((uint32_t)f2bf(v.x) | ((uint32_t)f2bf(v.y) << 16),
                                            (uint32_t)f2bf(v.z) | ((uint32_t)f2bf(v.w) << 16));
}
template <class T>
__device__ __forceinline__ void st4(T* p, const f32x4& v) {
  st4(p, make_float4(v[0], v[1], v[2], v[3]));
}
__device__ __forceinline__ float4 zf4() { return make_float4(0.f, 0.f, 0.f, 0.f); }

}  // namespace tfm
