// Device pieces shared by the dense kernels (dense.hip, trunk.hip).
//
// MFMA: v_mfma_f64_16x16x4f64.  Lane l supplies A[l % 16][l / 16] and
// B[l / 16][l % 16] of a 16x4 by 4x16 product; its four accumulator registers
// hold rows (l / 16) + 4 i of column l % 16.
#pragma once

#include "common.h"
#include "dense.h"

namespace helm {

typedef double d4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ d4 mfma16(double a, double b, d4 c) {
  return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ int acc_row(int lane, int i) { return (lane >> 4) + 4 * i; }

// tanh for the fp64 layers from expm1: t = e^{2|x|} - 1, tanh|x| = t / (t + 2),
// sign restored (no cancellation near 0).  2|x| = n ln 2 + r with |r| <= ln 2 / 2,
// e^r - 1 by its Taylor series to r^13 (the rest is below 2e-17 r), then
// t = 2^n (e^r - 1) + (2^n - 1), exact in its second term; the quotient by
// Newton's iteration on the reciprocal of t + 2 in [2, 2^64] and one correction.
// About 35 fp64 instructions, where the library expm1 and a general division
// take about 60: the vector fp64 work shares its units with the fp64 matrix
// products, so it adds to their time.  Past 2|x| = 44 the result is 1; NaN
// stays NaN.
__device__ __forceinline__ double tanh_fast(double x) {
  const double ax = 2.0 * fabs(x);
  const double y = ax > 44.0 ? 44.0 : ax;
  const double n = rint(y * 1.4426950408889634);
  double r = fma(n, -0.6931471805599453, y);
  r = fma(n, -2.3190468138462996e-17, r);
  double q = 1.0 / 6227020800.0;
  q = fma(q, r, 1.0 / 479001600.0);
  q = fma(q, r, 1.0 / 39916800.0);
  q = fma(q, r, 1.0 / 3628800.0);
  q = fma(q, r, 1.0 / 362880.0);
  q = fma(q, r, 1.0 / 40320.0);
  q = fma(q, r, 1.0 / 5040.0);
  q = fma(q, r, 1.0 / 720.0);
  q = fma(q, r, 1.0 / 120.0);
  q = fma(q, r, 1.0 / 24.0);
  q = fma(q, r, 1.0 / 6.0);
  q = fma(q, r, 0.5);
  const double p = fma(r * r, q, r);
  const double s = __hiloint2double(((int)n + 1023) << 20, 0);
  const double t = fma(s, p, s - 1.0);
  const double d = t + 2.0;
  double v = __builtin_amdgcn_rcp(d);
  v = fma(v, fma(-d, v, 1.0), v);
  v = fma(v, fma(-d, v, 1.0), v);
  const double u = t * v;
  return copysign(fma(v, fma(-d, u, t), u), x);
}

template <typename T>
__device__ __forceinline__ T activate(T x, int act) {
  if (act == ACT_TANH) return tanh_fast(x);
  if (act == ACT_RELU) return x > T(0) ? x : T(0);
  if (act == ACT_LEAKY) return x > T(0) ? x : T(0.01) * x;
  return x;
}

}  // namespace helm
