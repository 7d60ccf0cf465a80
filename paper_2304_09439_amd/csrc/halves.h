// A float as the sum of two halves, x0 = half(x) and x1 = half(x - x0): the rules of the kernels whose FP32 products are
// three 16-bit ones (net_split.hip, voxel.hip).  Both halves keep all their bits from 2^-2 to 2^16, so that operands are
// first multiplied by powers of two; a product is x0 y0 + x0 y1 + x1 y0, each operand exact to 2^-23 and the product
// left out at most 2^-22 of the whole.
#pragma once

#include <hip/hip_runtime.h>

namespace locc {

typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));

// Two floats to halves (round to nearest even), packed; the floats become the exact remainders.
__device__ __forceinline__ unsigned split_part(float& a, float& b) {
  const f16x2 h = __builtin_convertvector((f32x2){a, b}, f16x2);
  a = __builtin_fmaf((float)h[0], -1.f, a);
  b = __builtin_fmaf((float)h[1], -1.f, b);
  return __builtin_bit_cast(unsigned, h);
}
__device__ __forceinline__ unsigned last_part(float a, float b) {
  return __builtin_bit_cast(unsigned, __builtin_convertvector((f32x2){a, b}, f16x2));
}

constexpr float kHalvesLeast = 0x1p-2f;

// A power of two: v times it in [2^14, 2^15) (v at least 2^-100).
__device__ __forceinline__ float halves_scale(float v) {
  const int e = (int)((__float_as_uint(fmaxf(v, 0x1p-100f)) >> 23) & 255u) - 127;
  return __uint_as_float((unsigned)(127 + 14 - e) << 23);
}

// 1 / s of such a power of two.
__device__ __forceinline__ float halves_unscale(float s) { return __uint_as_float((254u << 23) - __float_as_uint(s)); }

// Whether too many of a row's values have halves short of bits: one may, and a `share`-th of those that are not 0
// (`count`: those that are not 0 << 16 | those short of bits).  By chance 2e-5 of the values are, so that three of 32
// activations, or three of 64 weights, are not: both limits leave out what the other catches, since few activations
// far below the others matter only with weights as far above the others'.
__host__ __device__ __forceinline__ bool halves_short(int count, int share) {
  return (count & 0xffff) > 1 + (count >> 16) / share;
}
constexpr int kShortWeights = 64, kShortActivations = 16;

}  // namespace locc
