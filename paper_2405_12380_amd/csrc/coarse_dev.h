// Device bodies of the skinny products of the trunk-basis correction (App. C),
// shared by the single-grid kernels and the batched ones:
//   qt_sweep      partials of Q^T x;
//   skinny_sweep  y_i = sum_j Q_ij c_j.
#pragma once

#include "common.h"
#include "dense_dev.h"

namespace helm {

enum { SK_ADD = 0, SK_SYNTH = 1 };

// 16 bytes of a basis row from column c (2 fp64 or 4 fp32 values): cached
// or streaming loads where rows are 16-byte aligned, otherwise one value at a
// time, 0 past column r.  Columns at or past r in the 16-byte forms
// read columns 0.. of the row instead (their factors are 0).
enum { LD_VALUES = 0, LD_CACHED = 1, LD_STREAM = 2 };
template <typename T> struct qvec;
template <> struct qvec<double> { using type = double __attribute__((ext_vector_type(2))); };
template <> struct qvec<float> { using type = float __attribute__((ext_vector_type(4))); };
template <typename T, int LD>
__device__ __forceinline__ typename qvec<T>::type ldq16(const T* row, int c, int r) {
  using V = typename qvec<T>::type;
  constexpr int VL = 16 / sizeof(T);
  const T* p = row + (c < r ? c : 0);
  if (LD == LD_STREAM) return __builtin_nontemporal_load(reinterpret_cast<const V*>(p));
  if (LD == LD_CACHED) return *reinterpret_cast<const V*>(p);
  V v;
#pragma unroll
  for (int k = 0; k < VL; ++k) v[k] = c + k < r ? row[c + k] : T(0);
  return v;
}

// Restriction: out[2j + {0,1}] = sum over a workgroup's rows of Q_ij x_i (sh: LDS)
// (complex x, real Q, j < r <= 128).  A row is read by LPR lanes, 16 bytes
// each (LPR the power of two that covers it), so a wavefront reads 64 / LPR
// rows per load whatever r is; rows go in groups of 4 such loads, wavefront w
// of the W in the grid taking groups w, w + W, ...: the grid reads one
// contiguous stretch of Q at a time.  What bounds it is the bytes in flight,
// so the next group's loads are issued before a group is used (two alternating
// register sets, no branch inside the loop).  The row-to-block assignment
// depends only on n and r: the partials are reproducible.  Against lanes owning
// columns l and l + 64 with one group in flight: 64^3, r = 128, from HBM 45 -> 43
// us (6.2 TB/s; 38 us where part of it is cached), 56 x 48 x 52, r = 96: 36.6 ->
// 17.2, 63^3, r = 32: 29.6 -> 11.8, 24 x 20 x 27, r = 48: 23.2 -> 3.5 us; fp32 13.0
// -> 4.4.
constexpr int QT_U = 4, QT_WAVES = 16;
// lanes that read one row of r columns of esz-byte values, 16 bytes each
__host__ __device__ inline int qt_lanes(int r, size_t esz) {
  const int need = (int)((r * esz + 15) / 16);
  return need <= 8 ? 8 : need <= 16 ? 16 : need <= 32 ? 32 : 64;
}
template <typename T, typename S, int LPR, int LD>
__device__ __forceinline__ void qt_sweep(size_t n, int r, const T* __restrict__ Q, const cplx_t<S>* __restrict__ x,
                                         size_t w, size_t W, double (*sh)[256], double* __restrict__ out) {
  // fewer loads a group where they are single values (registers)
  constexpr int VL = 16 / sizeof(T), RPW = 64 / LPR, U = LD == LD_VALUES ? 1 : QT_U;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int sub = lane / LPR, c0 = (lane % LPR) * VL;
  constexpr int GR = RPW * U;  // rows of a group
  const size_t nf = n / GR;    // whole groups
  const size_t qs = W * GR * r, xs = W * GR;
  const T* qp = Q + (w * GR + sub) * r;
  const cplx_t<S>* xp = x + w * GR + sub;
  struct Set {
    typename qvec<T>::type q[U];
    cplx_t<S> x[U];
  };
  auto load = [&](Set& s) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      s.q[u] = ldq16<T, LD>(qp + (size_t)(u * RPW * r), c0, r);
      s.x[u] = xp[u * RPW];
    }
    qp += qs;
    xp += xs;
    __builtin_amdgcn_sched_barrier(0);  // the loads stay ahead of the sums that follow
  };
  double ar[VL], ai[VL];
#pragma unroll
  for (int k = 0; k < VL; ++k) ar[k] = ai[k] = 0.0;
  auto add = [&](const Set& s) {
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int k = 0; k < VL; ++k) {
        ar[k] += (double)s.q[u][k] * (double)s.x[u].x;
        ai[k] += (double)s.q[u][k] * (double)s.x[u].y;
      }
  };
  if (w < nf) {
    Set a, b;
    size_t g = w;
    load(a);
    for (; g + 2 * W < nf; g += 2 * W) {
      load(b);
      add(a);
      load(a);
      add(b);
    }
    if (g + W < nf) {
      load(b);
      add(a);
      add(b);
    } else {
      add(a);
    }
  }
  if (n % GR && nf % W == w) {  // the rows past the last whole group
    Set s;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const size_t i = nf * GR + u * RPW + sub, ii = i < n ? i : n - 1;
      s.q[u] = ldq16<T, LD>(Q + ii * r, c0, r);
      s.x[u] = x[ii];
      if (i >= n) s.x[u].x = s.x[u].y = S(0);
    }
    add(s);
  }
#pragma unroll
  for (int off = LPR; off < 64; off <<= 1)
#pragma unroll
    for (int k = 0; k < VL; ++k) {
      ar[k] += __shfl_xor(ar[k], off, 64);
      ai[k] += __shfl_xor(ai[k], off, 64);
    }
  if (sub == 0)
#pragma unroll
    for (int k = 0; k < VL; ++k)
      if (c0 + k < r) {
        sh[wave][2 * (c0 + k)] = ar[k];
        sh[wave][2 * (c0 + k) + 1] = ai[k];
      }
  __syncthreads();
  for (int e = threadIdx.x; e < 2 * r; e += blockDim.x) {
    double v = 0.0;
#pragma unroll
    for (int k = 0; k < QT_WAVES; ++k) v += sh[k][e];
    out[e] = v;
  }
}

// Sums over the 16 (or 8) lanes of a row (half row) by data-parallel moves; every
// lane gets the total.
template <int CTRL>
__device__ __forceinline__ double dpp_add(double v) {
  const int lo = __double2loint(v), hi = __double2hiint(v);
  return v + __hiloint2double(__builtin_amdgcn_update_dpp(hi, hi, CTRL, 0xf, 0xf, false),
                              __builtin_amdgcn_update_dpp(lo, lo, CTRL, 0xf, 0xf, false));
}
template <int LANES>
__device__ __forceinline__ double row_sum(double v) {
  if (LANES == 16) v = dpp_add<0x140>(v);  // mirror of the row
  v = dpp_add<0x141>(v);                   // mirror of the half row
  v = dpp_add<0x4E>(v);                    // quads: lanes 2, 3, 0, 1
  return dpp_add<0xB1>(v);                 // lanes 1, 0, 3, 2
}
// a's sum over lanes l and l ^ 32 (l ^ 16) in the lanes whose bit 5 (bit 4) is
// clear, b's in the others: half of the partial sums move, none is kept twice
template <int BIT>
__device__ __forceinline__ double fold(double a, double b) {
  typedef unsigned u2 __attribute__((ext_vector_type(2)));
  u2 lo, hi;
  if (BIT == 32) {
    lo = __builtin_amdgcn_permlane32_swap((unsigned)__double2loint(a), (unsigned)__double2loint(b), false, false);
    hi = __builtin_amdgcn_permlane32_swap((unsigned)__double2hiint(a), (unsigned)__double2hiint(b), false, false);
  } else {
    lo = __builtin_amdgcn_permlane16_swap((unsigned)__double2loint(a), (unsigned)__double2loint(b), false, false);
    hi = __builtin_amdgcn_permlane16_swap((unsigned)__double2hiint(a), (unsigned)__double2hiint(b), false, false);
  }
  return __hiloint2double((int)hi[0], (int)lo[0]) + __hiloint2double((int)hi[1], (int)lo[1]);
}

// Prolongation: y_i = sum_j Q_ij c_j (complex c), z_i += y_i (SK_ADD) or z_i =
// scal[0] y_i, 0 on masked nodes (SK_SYNTH).  Lanes, rows and prefetch as in
// qt_sweep; the 4 loads' 8 partial sums per lane (re and im) are folded over
// lane bits 5 and 4 and summed within 16-lane rows by register moves alone (a
// shuffle through LDS per step was the dependent chain that bounded it where
// the basis comes from the memory-side cache).  56 x 48 x 52, r = 96: 25.2 -> 16.7
// us; 63^3, r = 32: 38.3 -> 12.8; 64^3, r = 128, from HBM: 45 -> 43; fp32 48^3,
// r = 128: 16.0 -> 11.0.
template <typename T, typename S, int MODE, int LPR, int LD>
__device__ __forceinline__ void skinny_sweep(size_t n, int r, const T* __restrict__ Q, const double* __restrict__ c,
                                             cplx_t<S>* __restrict__ z, const uint8_t* __restrict__ mask,
                                             const double* __restrict__ scal, size_t w, size_t W) {
  constexpr int VL = 16 / sizeof(T), RPW = 64 / LPR, U = 4;
  const int lane = threadIdx.x & 63;
  const int sub = lane / LPR, c0 = (lane % LPR) * VL;
  double cr[VL], ci[VL];
#pragma unroll
  for (int k = 0; k < VL; ++k) {
    cr[k] = c0 + k < r ? c[2 * (c0 + k)] : 0.0;
    ci[k] = c0 + k < r ? c[2 * (c0 + k) + 1] : 0.0;
  }
  const double sc = MODE == SK_SYNTH ? scal[0] : 1.0;
  S* zs = reinterpret_cast<S*>(z);
  // where this lane's result belongs: load u and component comp, or none
  const int m = lane % (LPR < 16 ? LPR : 16);
  int u_out, comp = m & 1;
  bool writes;
  if (LPR == 64) {
    u_out = (lane >> 5 << 1) | ((lane >> 4) & 1);
    writes = m < 2;
  } else if (LPR == 32) {
    u_out = (((lane >> 4) & 1) << 1) | ((m >> 1) & 1);
    writes = m < 4;
  } else {
    u_out = (m >> 1) & 3;
    writes = m < 8;
  }
  constexpr int GR = RPW * U;  // rows of a group
  const size_t nf = n / GR;    // whole groups
  const int ro = u_out * RPW + sub;  // this lane's result's row in its group
  const size_t qs = W * GR * r, zst = W * GR;
  const T* qp = Q + (w * GR + sub) * r;
  size_t zi = w * GR + ro;
  struct Set {
    typename qvec<T>::type q[U];
    double z;  // the old value (ADD), or the factor (SYNTH)
  };
  auto load = [&](Set& s) {
#pragma unroll
    for (int u = 0; u < U; ++u) s.q[u] = ldq16<T, LD>(qp + (size_t)(u * RPW * r), c0, r);
    if (MODE == SK_ADD) s.z = (double)zs[2 * zi + comp];
    else s.z = mask[zi] ? 0.0 : sc;
    qp += qs;
    zi += zst;
    __builtin_amdgcn_sched_barrier(0);
  };
  auto put = [&](const Set& s, size_t g) {
    double v[2 * U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      double a = 0.0, b = 0.0;
#pragma unroll
      for (int k = 0; k < VL; ++k) {
        a += (double)s.q[u][k] * cr[k];
        b += (double)s.q[u][k] * ci[k];
      }
      v[2 * u] = a;
      v[2 * u + 1] = b;
    }
    double y;
    if (LPR == 64) {
      double f[4], h[2];
#pragma unroll
      for (int k = 0; k < 4; ++k) f[k] = fold<32>(v[k], v[k + 4]);
#pragma unroll
      for (int k = 0; k < 2; ++k) h[k] = row_sum<16>(fold<16>(f[k], f[k + 2]));
      y = comp ? h[1] : h[0];
    } else if (LPR == 32) {
      double f[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) f[k] = row_sum<16>(fold<16>(v[k], v[k + 4]));
      y = m & 2 ? (comp ? f[3] : f[2]) : (comp ? f[1] : f[0]);
    } else {
#pragma unroll
      for (int k = 0; k < 8; ++k) v[k] = row_sum<LPR == 16 ? 16 : 8>(v[k]);
      const double a = m & 2 ? (comp ? v[3] : v[2]) : (comp ? v[1] : v[0]);
      const double b = m & 2 ? (comp ? v[7] : v[6]) : (comp ? v[5] : v[4]);
      y = m & 4 ? b : a;
    }
    const size_t i = g * GR + ro;
    if (writes && i < n) zs[2 * i + comp] = (S)(MODE == SK_ADD ? s.z + y : s.z != 0.0 ? y * s.z : 0.0);
  };
  if (w < nf) {
    Set a, b;
    size_t g = w;
    load(a);
    for (; g + 2 * W < nf; g += 2 * W) {
      load(b);
      put(a, g);
      load(a);
      put(b, g + W);
    }
    if (g + W < nf) {
      load(b);
      put(a, g);
      put(b, g + W);
    } else {
      put(a, g);
    }
  }
  if (n % GR && nf % W == w) {  // the rows past the last whole group
    Set s;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const size_t i = nf * GR + u * RPW + sub;
      s.q[u] = ldq16<T, LD>(Q + (i < n ? i : n - 1) * r, c0, r);
    }
    const size_t i = nf * GR + ro, ii = i < n ? i : n - 1;
    if (MODE == SK_ADD) s.z = (double)zs[2 * ii + comp];
    else s.z = mask[ii] ? 0.0 : sc;
    put(s, nf);
  }
}

}  // namespace helm
