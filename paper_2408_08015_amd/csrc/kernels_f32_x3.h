// Products of fp32 matrices on the bf16 matrix cores: every operand is split into three bf16 pieces
// (x = x1 + x2 + x3, each the rounding of what is left), which together hold its 24 bits, and a product keeps the six
// piece products that reach 32-bit precision (the scheme of Henry, Tang and Heinecke, "Leveraging the bfloat16 Artificial
// Intelligence Datatype For Higher-Precision Computations", ARITH 2019).  v_mfma_f32_32x32x16_bf16 takes 32 cycles for a
// contraction of 16 where v_mfma_f32_32x32x2_f32 takes 512: six of them are 2.7 times faster.  The five small products add up
// in an accumulator of their own, so the large sum is rounded twice per 16 terms: the instruction adds the terms 0 to 7 and
// then 8 to 15, each time rounding to nearest, ties to even.  (Measured.  Where a product is larger than what it is added to,
// that is first cut downwards to a multiple of half the product's ulp: the large products go straight to the growing sum and
// are not collected step by step from zero.)  Relative error of a product of normal matrices against 64 bits, fp32
// matrix instructions / this: contraction 24 9.0e-8 / 3.6e-8, 256 2.9e-7 / 8.9e-8, 2304 8.6e-7 / 2.9e-7; with one operand
// behind a ReLU 6.5e-8 / 3.1e-8, 2.1e-7 / 7.0e-8, 6.0e-7 / 2.2e-7.
//
// The pieces end at 2^-133, the smallest bf16 value: an operand below 2^-110 loses what lies under that, so a product of
// operands that are all so small has fewer than 24 bits (17 at 2^-117).
//
// An infinity or a NaN in an operand, and a value within half a bf16 ulp of the largest finite one, makes a piece or a
// piece product that is not finite, so the sum is not finite either: a wavefront that holds such sums forms them again on
// the fp32 matrix instructions from the operands themselves, and takes those.  Where every value is NaN that is the time of
// both and of loads that nothing hides: forward and backward of 24 -> 144 channels at 8 x 56x56 31 us finite, 59 us NaN; 64 ->
// 64 3x3 at 4 x 56x56 63 and 155; 256 -> 256 3x3 at 2 x 14x14 56 and 126.  (By their definition, element by element, they
// took 490, 2070 and 2950 us.)
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
// the eight values of a split word: every finite weight is the sum of its pieces, another one is the first of them
__device__ __forceinline__ void join3(const uint4 (&p)[3], float (&v)[8]) {
  auto pair = [](uint32_t a, uint32_t b, uint32_t c, float& lo, float& hi) __attribute__((always_inline)) {
    lo = __uint_as_float(a << 16) + (__uint_as_float(b << 16) + __uint_as_float(c << 16));
    hi = __uint_as_float(a & 0xffff0000u) + (__uint_as_float(b & 0xffff0000u) + __uint_as_float(c & 0xffff0000u));
  };
  pair(p[0].x, p[1].x, p[2].x, v[0], v[1]);
  pair(p[0].y, p[1].y, p[2].y, v[2], v[3]);
  pair(p[0].z, p[1].z, p[2].z, v[4], v[5]);
  pair(p[0].w, p[1].w, p[2].w, v[6], v[7]);
}
// c += a b over 16 terms in fp32, the operands laid out as those of mfma_bf16
__device__ __forceinline__ floatx16 mfma_f32(const float (&a)[8], const float (&b)[8], floatx16 c) {
#pragma unroll
  for (int e = 0; e < 8; ++e) c = __builtin_amdgcn_mfma_f32_32x32x2f32(a[e], b[e], c, 0, 0, 0);
  return c;
}
// zeros made where they stand: the compiler would make them for rare code at the kernel's start
__device__ __forceinline__ floatx16 zero16() {
  float o = 0.f;
  asm volatile("" : "+v"(o));
  floatx16 z;
#pragma unroll
  for (int r = 0; r < 16; ++r) z[r] = o;
  return z;
}
// c += s, and bad + 0 * c: 0 as long as every c is finite, else NaN
__device__ __forceinline__ float add_small(floatx16& c, const floatx16& s, float bad) {
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    c[r] += s[r];
    bad = fmaf(c[r], 0.f, bad);
  }
  return bad;
}
// (NaN != 0; what follows is rare, and laid out behind the rest of the kernel)
__device__ __forceinline__ bool any_not_finite(float bad) { return __builtin_expect(__any(bad != 0.f), 0); }
__device__ __forceinline__ void take_not_finite(floatx16& c, const floatx16& again) {
#pragma unroll
  for (int r = 0; r < 16; ++r) c[r] = fabsf(c[r]) < __builtin_inff() ? c[r] : again[r];
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
