// float32 values as three bfloat16 parts (split.hip says why) and the CELU of
// the float32 model, for the kernels that use them.
#pragma once

#include "internal.h"

namespace nnp {

typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float floatx2 __attribute__((ext_vector_type(2)));

constexpr int kPartChunk = 3 * 32;  // elements of a row's 32-column chunk, its three parts

// CELU(z) = z for z > 0, else alpha expm1(t) with t = z / alpha.  expm1 is its
// Taylor polynomial to t^9 for t > -0.5 (the remainder is below 3e-10 of the
// value), and the hardware exp2 minus one below that, where the subtraction
// loses under two bits: within 2 ulp either way, a third of the instructions
// of the library function, which took as long as the MFMAs of a layer.
__device__ inline float celu32(float z, float alpha, float inv_alpha) {
  const float t = z * inv_alpha;
  float p = fmaf(t, 2.7557319e-6f, 2.4801587e-5f);
  p = fmaf(t, p, 1.9841270e-4f);
  p = fmaf(t, p, 1.3888889e-3f);
  p = fmaf(t, p, 8.3333333e-3f);
  p = fmaf(t, p, 4.1666667e-2f);
  p = fmaf(t, p, 1.6666667e-1f);
  p = fmaf(t, p, 0.5f);
  p = fmaf(t * t, p, t);
  const float e = __builtin_amdgcn_exp2f(t * 1.4426950408889634f) - 1.f;
  return z > 0.f ? z : alpha * (t > -0.5f ? p : e);
}
__device__ inline float dcelu32(float h, float inv_alpha) { return h > 0.f ? 1.f : 1.f + h * inv_alpha; }

// The three parts of eight floats.
struct Parts {
  bf16x8 p1, p2, p3;
};
__device__ inline uint32_t round2(float lo, float hi) {
  return __builtin_bit_cast(uint32_t, __builtin_convertvector((floatx2){lo, hi}, bf16x2));
}
// Rounds x[0..7] to bfloat16 and leaves in x what the rounding dropped (exact).
__device__ inline bf16x8 take_part(float (&x)[8]) {
  uint4 u;
  uint32_t w[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    w[k] = round2(x[2 * k], x[2 * k + 1]);
    x[2 * k] -= __uint_as_float(w[k] << 16);
    x[2 * k + 1] -= __uint_as_float(w[k] & 0xffff0000u);
  }
  u.x = w[0]; u.y = w[1]; u.z = w[2]; u.w = w[3];
  return __builtin_bit_cast(bf16x8, u);
}
__device__ inline Parts split8(const float (&v)[8]) {
  float x[8];
#pragma unroll
  for (int k = 0; k < 8; ++k) x[k] = v[k];
  Parts s;
  s.p1 = take_part(x);
  s.p2 = take_part(x);
  uint4 u;
  u.x = round2(x[0], x[1]); u.y = round2(x[2], x[3]); u.z = round2(x[4], x[5]); u.w = round2(x[6], x[7]);
  s.p3 = __builtin_bit_cast(bf16x8, u);
  return s;
}
// Largest magnitude of eight floats (NaNs do not count: their parts are NaN).
__device__ inline float max8(const float (&x)[8]) {
  float m = fmaxf(fmaxf(fabsf(x[0]), fabsf(x[1])), fabsf(x[2]));
  m = fmaxf(fmaxf(m, fabsf(x[3])), fabsf(x[4]));
  m = fmaxf(fmaxf(m, fabsf(x[5])), fabsf(x[6]));
  return fmaxf(m, fabsf(x[7]));
}
constexpr float kPartMax = 3.3895314e38f;  // largest finite bfloat16: above it the first part may overflow

// A value from its parts, `stride` elements apart (exact for what the parts
// hold: all bits of a weight, and of an activation of at least 2^-102).
template <class P>
__device__ inline float joined(P p, int stride) {
  const float a = __uint_as_float((uint32_t)p[0] << 16), b = __uint_as_float((uint32_t)p[stride] << 16);
  return a + (b + __uint_as_float((uint32_t)p[2 * stride] << 16));
}

}  // namespace nnp
