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

// CELU(z) = z for z > 0, else alpha expm1(t) with t = z / alpha.
//   expm1(t) = 2^n expm1(r) + (2^n - 1),  t = n ln 2 + r,  |r| <= ln 2 / 2:
// 2^n and 2^n - 1 are exact, ln 2 comes in two parts of which the first times
// n is exact, and expm1(r) is its Taylor polynomial to r^9 (the remainder is
// below 2^-30 of the value).  Below t = -25 the value is -1.  n is the low bits
// of a sum large enough that its unit is 1.  Over 16.7 million values (alpha = 1)
// 0.884 units in the last place are lost at most and 0.250 on average, as with
// the library's expm1f (0.883 and 0.250), in three quarters of its time in a
// loop of nothing else; exp2(x) - 1, faster on paper, cancels (1.76 near
// t = -0.52) and took as long.
__device__ inline float celu32(float z, float alpha, float inv_alpha) {
  constexpr float kUnit = 12582912.f;  // 1.5 x 2^23
  float t = z * inv_alpha;
  t = t < -25.f ? -25.f : t;  // (a NaN stays one)
  const float k = fmaf(t, 1.4426950408889634f, kUnit), n = k - kUnit;
  const float r = fmaf(n, -1.42860677e-6f, fmaf(n, -0.693145752f, t));
  float q = fmaf(r, 2.7557319e-6f, 2.4801587e-5f);
  q = fmaf(r, q, 1.9841270e-4f);
  q = fmaf(r, q, 1.3888889e-3f);
  q = fmaf(r, q, 8.3333333e-3f);
  q = fmaf(r, q, 4.1666667e-2f);
  q = fmaf(r, q, 1.6666667e-1f);
  q = fmaf(r, q, 0.5f);
  q = fmaf(r * r, q, r);
  const float two_n = __uint_as_float((__float_as_uint(k) << 23) + 0x3f800000u);
  return z > 0.f ? z : alpha * fmaf(two_n, q, two_n - 1.f);
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
