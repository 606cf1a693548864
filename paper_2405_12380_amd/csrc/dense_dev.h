// Device pieces shared by the dense kernels (dense.hip, trunk.hip, gram.hip).
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

// tanh for the fp64 layers from expm1: with t = (e^{2|x|} - 1) / 2, tanh|x| = t / (t + 1),
// sign restored (no cancellation near 0).  |x| = n ln 2 / 2 + r with |r| <= ln 2 / 4,
// (e^{2r} - 1) / 2 = r + r^2 q(r), q the degree-10 interpolant at the Chebyshev
// nodes of the range (error 8e-19 of the value), then t = 2^n (r + r^2 q) +
// (2^n - 1) / 2, exact in its second term; n and 2^n without conversions, from the
// low word of |x| 2 / ln 2 + 1.5 * 2^52; the quotient by one third-order step on the
// reciprocal of t + 1 in [1, 2^63] and one correction.  27 fp64 instructions, where
// the library expm1 and a general division take about 60: fp64 work adds to the
// time of the matrix products beside it.  Past |x| = 22 the result is 1; NaN
// stays NaN.
__device__ __forceinline__ double tanh_fast(double x) {
  const double ax = fabs(x);
  const double y = ax > 22.0 ? 22.0 : ax;
  const double m = fma(y, 2.8853900817779268, 6755399441055744.0), n = m - 6755399441055744.0;
  double r = fma(n, -0.34657359027997264, y);
  r = fma(n, -1.1600963245594897e-17, r);
  double q = 4.283334771688116e-06;
  q = fma(q, r, 2.5707771489828415e-05);
  q = fma(q, r, 0.00014109323851772937);
  q = fma(q, r, 0.0007054657366917812);
  q = fma(q, r, 0.0031746031778077236);
  q = fma(q, r, 0.012698412719909201);
  q = fma(q, r, 0.044444444444425406);
  q = fma(q, r, 0.13333333333321806);
  q = fma(q, r, 0.33333333333333337);
  q = fma(q, r, 0.6666666666666669);
  q = fma(q, r, 1.0);
  const double p = fma(r * r, q, r);
  const double s = __hiloint2double((__double2loint(m) << 20) + 0x3FF00000, 0);
  const double t = fma(s, p, fma(s, 0.5, -0.5));
  const double d = t + 1.0;
  double v = __builtin_amdgcn_rcp(d);
  const double e = fma(-d, v, 1.0);
  v = fma(v, fma(e, e, e), v);
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

constexpr int TRUNK_WAVES = 8;
// Workgroups of TRUNK_WAVES wavefronts as 32 x 16 threads: a launch has fewer
// than 2^32 work-items on an axis, and a grid of 2^31 nodes in 32-row blocks
// has 2^26 workgroups.
inline dim3 trunk_block() { return dim3(32, 2 * TRUNK_WAVES); }
__device__ __forceinline__ int trunk_thread() { return threadIdx.x + 32 * threadIdx.y; }

// One layer for RT x 16 rows and the CT column tiles wave, wave + 8 (16 columns
// each): acc = H W over k < kend (a multiple of 8 DEPTH, at most W's K rows; columns
// past N hold other columns' values or 0).  A from LDS, two consecutive k per 16-byte read: lane
// group g = lane / 16 holds k = 8 c + 2 g + s of step s of chunk c, which is the
// k its W rows are loaded from.  W comes straight from memory (1.8 MB at the
// 3-256x4-128 trunk: it stays in every XCD's L2) into registers DEPTH chunks
// ahead, so the k loop has no barrier.
template <int RT, int CT>
__device__ __forceinline__ void trunk_layer(const double* __restrict__ h, int lda, const double* __restrict__ W, int K,
                                            int N, int wave, int lane, d4 (&acc)[RT][CT], int kend) {
  constexpr int DEPTH = RT > 1 ? 2 : 4;
  // buffer loads: a fixed lane offset and a uniform one that advances, so the
  // loop carries one scalar for all of W's addresses
  const __amdgpu_buffer_rsrc_t wr =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<double*>(W), 0, 8 * K * N, 0x00020000);
  const int wo = 8 * (2 * (lane >> 4) * N + (lane & 15));
  int so = 128 * wave;
  const double* ap = h + (lane & 15) * lda + 2 * (lane >> 4);
  double bq[DEPTH][2][CT];
  double2 av[2][RT];
  // the scheduling barriers keep the loads here: W's DEPTH chunks ahead of
  // their use, A's one
  auto load = [&](int d) {
#pragma unroll
    for (int s = 0; s < 2; ++s)
#pragma unroll
      for (int j = 0; j < CT; ++j)
        bq[d][s][j] = __builtin_bit_cast(
            double, __builtin_amdgcn_raw_buffer_load_b64(wr, wo + 128 * TRUNK_WAVES * j, so + 8 * s * N, 0));
    so += 64 * N;
    __builtin_amdgcn_sched_barrier(0);
  };
  auto load_a = [&](int d) {
#pragma unroll
    for (int i = 0; i < RT; ++i) av[d][i] = *reinterpret_cast<const double2*>(ap + i * 16 * lda);
    ap += 8;
    __builtin_amdgcn_sched_barrier(0);
  };
  auto multiply = [&](int d) {
#pragma unroll
    for (int s = 0; s < 2; ++s)
#pragma unroll
      for (int i = 0; i < RT; ++i)
#pragma unroll
        for (int j = 0; j < CT; ++j)
          acc[i][j] = mfma16(s ? av[d & 1][i].y : av[d & 1][i].x, bq[d][s][j], acc[i][j]);
  };
#pragma unroll
  for (int i = 0; i < RT; ++i)
#pragma unroll
    for (int j = 0; j < CT; ++j) acc[i][j] = d4{0, 0, 0, 0};
#pragma unroll
  for (int d = 0; d < DEPTH; ++d) load(d);
  load_a(0);
  for (int k = 8 * DEPTH; k < kend; k += 8 * DEPTH) {
#pragma unroll
    for (int d = 0; d < DEPTH; ++d) {
      load_a((d + 1) & 1);
      multiply(d);
      load(d);
    }
  }
#pragma unroll
  for (int d = 0; d < DEPTH; ++d) {
    if (d + 1 < DEPTH) load_a((d + 1) & 1);
    multiply(d);
  }
}

}  // namespace helm
