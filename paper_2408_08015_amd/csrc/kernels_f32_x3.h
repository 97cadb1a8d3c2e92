// Products of fp32 matrices on the bf16 matrix cores: every operand is split into three bf16 pieces
// (x = x1 + x2 + x3, each the rounding of what is left), which together hold its 24 bits, and a product keeps the six
// piece products that reach 32-bit precision.  v_mfma_f32_32x32x16_bf16 takes 32 cycles for a contraction of 16 where
// v_mfma_f32_32x32x2_f32 takes 512: six of them are 2.7 times faster.  The five small products add up in an accumulator of
// their own, so the large sum is rounded once per 16 terms.  Relative error of a product of normal matrices against 64
// bits, fp32 matrix instructions / this: contraction 24 9.0e-8 / 3.6e-8, 256 2.9e-7 / 8.9e-8, 2304 8.6e-7 / 2.9e-7; with one
// operand behind a ReLU 6.5e-8 / 3.1e-8, 2.1e-7 / 7.0e-8, 6.0e-7 / 2.2e-7.
//
// An infinity or a NaN in an operand, and a value within half a bf16 ulp of the largest finite one, makes a piece or a
// piece product that is not finite, so the result is not finite either: results that are not finite are computed again by
// their definition.
#pragma once
#include "device_utils.h"

namespace ast {

// pieces of two neighbouring values, the first in the low half of each word
__device__ __forceinline__ void split3(float a, float b, uint32_t& p1, uint32_t& p2, uint32_t& p3) {
  p1 = f2bf_pk(a, b);
  a -= __uint_as_float(p1 << 16);
  b -= __uint_as_float(p1 & 0xffff0000u);
  p2 = f2bf_pk(a, b);
  a -= __uint_as_float(p2 << 16);
  b -= __uint_as_float(p2 & 0xffff0000u);
  p3 = f2bf_pk(a, b);
}
__device__ __forceinline__ void split3(const float (&v)[8], uint4 (&p)[3]) {
  split3(v[0], v[1], p[0].x, p[1].x, p[2].x);
  split3(v[2], v[3], p[0].y, p[1].y, p[2].y);
  split3(v[4], v[5], p[0].z, p[1].z, p[2].z);
  split3(v[6], v[7], p[0].w, p[1].w, p[2].w);
}
__device__ __forceinline__ floatx16 mfma_bf16(uint4 a, uint4 b, floatx16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}
__device__ __forceinline__ bool finite_f(float v) { return fabsf(v) < __builtin_inff(); }

constexpr unsigned kOutside = 0x80000000u;  // buffer offset beyond every extent: a load gives 0, a store is dropped
// descriptor of `words` words from p on (uniform over the wavefront)
__device__ __forceinline__ __amdgpu_buffer_rsrc_t rsrc_words(const float* p, size_t words) {
  const unsigned n = (unsigned)min(words, (size_t)0x1ffffffc) * 4u;
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(p), 0, __builtin_amdgcn_readfirstlane(n), 0x00020000);
}

// Sample (counted from the first one) of position r of consecutive planes of HW pixels, r < HW + 512: floor(r / HW) without
// the forty instructions of a division.  rHW: ceil(2^20 / HW) where planes are small enough for r to pass several.
__host__ __device__ constexpr unsigned plane_reciprocal(int HW) { return HW >= 512 ? 0u : ((1u << 20) + HW - 1) / HW; }
__device__ __forceinline__ unsigned plane_of(unsigned r, unsigned HW, unsigned rHW) {
  return rHW ? r * rHW >> 20 : r >= HW;  // (rHW is uniform; the error of r * rHW is below 1024 * 512)
}

}  // namespace ast
