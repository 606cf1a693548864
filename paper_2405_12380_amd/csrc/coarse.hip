// Trunk-basis coarse space of App. C and its per-application correction.
//
// Setup (once per network, p_used and k^2): P = first p_used trunk columns with
// scatterer rows zeroed; Cholesky of P^T P with column dropping, Q1 = P S1.
// fp64 basis: the solves use Q1 (it spans the space of the orthonormal
// Q = Q1 S2 of a second CholeskyQR pass, and the correction depends only on
// that span).  fp32 basis: the second pass is run and Q rounded to fp32.  In
// either basis X: B = (L - diag(Re s)) X by a batched real stencil; the
// Galerkin matrix X^T B - i X^T diag(Im s) X (= X^T A X); its inverse by
// Gauss-Jordan with partial pivoting.
//
// Correction z += X (X^T A X)^{-1} X^T r1 (HBM-bound skinny products):
//   k_qt_part      per-block partials of Q^T r1;
//   k_reduce_ainv  their sum y and c = A_c^{-1} y;
//   k_skinny       z_i += sum_j Q_ij c_j.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <type_traits>
#include <vector>

#include "common.h"
#include "dense.h"
#include "internal.h"
#include "lib.h"
#include "prof.h"
#include "coarse_dev.h"
#include "stencil_dev.h"

namespace helm {

static constexpr size_t QT_MAXB = 256;
// How a basis is loaded: through the caches up to 192 MB, where most of it is
// still in the 256 MB memory-side cache at the next pass (56 x 48 x 52, r = 96,
// 107 MB: one inversion step 4870 us, against 5170 streaming); streaming
// beyond, where it would only push the Krylov vectors out (64^3, r = 128, 268 MB:
// a 60-step GMRES solve 14020 us, against 14290 cached).  Rows that are not
// 16-byte aligned go value by value.
static int q_load(size_t n, int r, size_t esz) {
  if (r * esz % 16) return LD_VALUES;
  return n * r * esz <= ((size_t)192 << 20) ? LD_CACHED : LD_STREAM;
}
// workgroups of the restriction: at most one to a CU (the partials they write
// are read again by every workgroup of k_reduce_ainv), fewer where a
// wavefront would have no rows
static int qt_nblocks(size_t n, int r, size_t esz) {
  const size_t rows = (size_t)QT_WAVES * QT_U * (64 / qt_lanes(r, esz));
  const size_t nb = (n + rows - 1) / rows;
  return (int)(nb < QT_MAXB ? nb : QT_MAXB);
}

template <typename T, typename S, int LPR, int LD>
__global__ __launch_bounds__(64 * QT_WAVES) void k_qt_part(size_t n, int r, const T* __restrict__ Q,
                                                           const cplx_t<S>* __restrict__ x,
                                                           double* __restrict__ part) {
  __shared__ double sh[QT_WAVES][256];
  qt_sweep<T, S, LPR, LD>(n, r, Q, x, (blockIdx.x * (size_t)blockDim.x + threadIdx.x) >> 6,
                          ((size_t)gridDim.x * blockDim.x) >> 6, sh, part + (size_t)blockIdx.x * 2 * r);
}

// y = the sum of the restriction's nb partials (in a fixed order), c = Ainv y
// (r x r complex, row-major).  Workgroup b forms y for itself and then rows 16 b
// .. 16 b + 15 of c, a wavefront each, with the row of Ainv loaded before the
// partials.  What bounds it is the 2 r nb doubles one CU reads: 8.8 us at
// r = 128 and 256 partials (two launches, the sums and the product, took 4.8 and
// 4.6 us and a gap), 4.5 us on small grids (two launches: 6.4 to 9).
__global__ __launch_bounds__(1024) void k_reduce_ainv(int r, int nb, const double* __restrict__ part,
                                                      const double* __restrict__ Ainv, double* __restrict__ c) {
  __shared__ double2 sh[8][128], y[128];
  const int t = threadIdx.x, lane = t & 63, j = blockIdx.x * 16 + (t >> 6);
  const double2* A = reinterpret_cast<const double2*>(Ainv) + (size_t)(j < r ? j : 0) * r;
  const double2 a0 = lane < r ? A[lane] : czero(), a1 = lane + 64 < r ? A[lane + 64] : czero();
  const int e = t & 127, s = t >> 7;
  const double2* p2 = reinterpret_cast<const double2*>(part) + e;
  double2 acc = czero();
  if (e < r)
    for (int b0 = s; b0 < nb; b0 += 8 * 16) {
      double2 v[16];
#pragma unroll
      for (int u = 0; u < 16; ++u) v[u] = b0 + 8 * u < nb ? p2[(size_t)(b0 + 8 * u) * r] : czero();
#pragma unroll
      for (int u = 0; u < 16; ++u) acc = cadd(acc, v[u]);
    }
  sh[s][e] = acc;
  __syncthreads();
  if (t < 128) {
    double2 v = sh[0][t];
#pragma unroll
    for (int k = 1; k < 8; ++k) v = cadd(v, sh[k][t]);
    y[t] = v;
  }
  __syncthreads();
  double2 v = czero();
  if (lane < r) v = cmul(a0, y[lane]);
  if (lane + 64 < r) v = cadd(v, cmul(a1, y[lane + 64]));
  v.x = wave_sum(v.x);
  v.y = wave_sum(v.y);
  if (lane == 0 && j < r) {
    c[2 * j] = v.x;
    c[2 * j + 1] = v.y;
  }
}

template <typename T, typename S, int MODE, int LPR, int LD>
__global__ __launch_bounds__(256) void k_skinny(size_t n, int r, const T* __restrict__ Q, const double* __restrict__ c,
                                                cplx_t<S>* __restrict__ z, const uint8_t* __restrict__ mask,
                                                const double* __restrict__ scal) {
  skinny_sweep<T, S, MODE, LPR, LD>(n, r, Q, c, z, mask, scal, (blockIdx.x * (size_t)blockDim.x + threadIdx.x) >> 6,
                                ((size_t)gridDim.x * blockDim.x) >> 6);
}

// B = (L - diag(Re s)) Q on real columns (n x r, row-major); masked rows -> 0.
// A wavefront takes an (x, y) column of nodes and marches along a segment of z, its
// lanes V columns of Q each: z neighbours pass through registers, and each XCD gets
// one range of (x, y), so the x and y neighbours' rows are read while they lie in
// its L2.  Absent neighbours (ghost or masked) come from the node's neighbour code;
// an absent one reads the node itself, so that a node's loads are issued together.
// Bound by reading Q and writing B (104 us at 64^3 x 128 at 5.15 TB/s).  A node at
// a time over all XCDs, 8-byte loads behind seven branches took 217 us (every row
// fetched for each of its three planes), node ranges by XCD 206, this 173 (89 -> 57
// at 56 x 48 x 52 x 96, 376 -> 281 at 80 x 72 x 76 x 128).
template <typename S, int V>
__global__ __launch_bounds__(256) void k_batched_lap(StencilGeom g, int r, int seg, size_t w0, const double* __restrict__ Q,
                                                     const cplx_t<S>* __restrict__ sc, const uint8_t* __restrict__ code,
                                                     double* __restrict__ B) {
  typedef double dv __attribute__((ext_vector_type(V)));
  const size_t nxy = (size_t)g.nx * g.ny, ry = (size_t)g.nx * r, rz = nxy * r;
  // logical wavefront, from w0 on: segment fastest
  const unsigned nseg = (g.nz + seg - 1) / seg;
  const size_t lw = w0 + (size_t)xcd_remap(blockIdx.x, gridDim.x) * 4 + __builtin_amdgcn_readfirstlane(threadIdx.y);
  const size_t q = lw / nseg;
  if (q >= nxy) return;
  const int z0 = (int)(lw % nseg) * seg, z1 = min(g.nz, z0 + seg);
  auto at = [&](size_t e) { return *reinterpret_cast<const dv*>(Q + e); };
  for (int j = threadIdx.x * V; j < r; j += 64 * V) {
    size_t p = q + z0 * nxy;
    dv c = at(p * r + j), zm = z0 > 0 ? at((p - nxy) * r + j) : dv(0.0);
    for (int z = z0; z < z1; ++z, p += nxy) {
      const size_t e = p * r + j;
      const unsigned cd = __builtin_amdgcn_readfirstlane((unsigned)code[p]);
      const double sre = ldc(sc, p).x;
      dv xm = at(e - ((cd & NB_XM) ? 0 : r)), xp = at(e + ((cd & NB_XP) ? 0 : r));
      dv ym = at(e - ((cd & NB_YM) ? 0 : ry)), yp = at(e + ((cd & NB_YP) ? 0 : ry));
      const dv zn = at(e + (z + 1 < g.nz ? rz : 0));
      if (cd & NB_XM) xm = dv(0.0);
      if (cd & NB_XP) xp = dv(0.0);
      if (cd & NB_YM) ym = dv(0.0);
      if (cd & NB_YP) yp = dv(0.0);
      dv acc = ((c - xm) + (c - xp)) * g.ih2[0];
      acc = acc + ((c - ym) + (c - yp)) * g.ih2[1];
      if (g.dim == 3)
        acc = acc + ((c - ((cd & NB_ZM) ? dv(0.0) : zm)) + (c - ((cd & NB_ZP) ? dv(0.0) : zn))) * g.ih2[2];
      acc = acc - sre * c;
      __builtin_nontemporal_store((cd & NB_SELF) ? dv(0.0) : acc, reinterpret_cast<dv*>(B + e));
      zm = c;
      c = zn;
    }
  }
}

// P = T[:, :pu] (T: n x p, dtype precision) in fp64 with masked rows zeroed
template <typename T>
__global__ void k_mask_cols(size_t n, int p, int pu, const T* __restrict__ Tm, const uint8_t* __restrict__ mask,
                            double* __restrict__ P) {
  const size_t total = n * pu;
  for (size_t e = blockIdx.x * (size_t)blockDim.x + threadIdx.x; e < total; e += (size_t)gridDim.x * blockDim.x) {
    const size_t i = e / pu;
    const int j = (int)(e % pu);
    P[e] = mask[i] ? 0.0 : (double)Tm[i * p + j];
  }
}

// rows of scatterer nodes zeroed in place (T: n x p): the op's cached trunk
// matrix is kept masked, which the network synthesis (zero on the scatterer)
// does not see and the coarse space needs
template <typename T>
__global__ __launch_bounds__(256) void k_zero_masked_rows(size_t n, int p, const uint8_t* __restrict__ mask,
                                                          T* __restrict__ Tm) {
  // one row per wavefront step (threadIdx.y), the lanes across its p entries
  for (size_t i = blockIdx.x * (size_t)blockDim.y + threadIdx.y; i < n; i += (size_t)gridDim.x * blockDim.y)
    if (mask[i])
      for (int c = threadIdx.x; c < p; c += 64) Tm[i * p + c] = T(0);
}

// Qs = (T) Q and Q <- (double) Qs, so the coarse matrix is built from the basis
// actually stored.
template <typename T>
__global__ void k_round_q(size_t total, double* __restrict__ Q, T* __restrict__ Qs) {
  for (size_t e = blockIdx.x * (size_t)blockDim.x + threadIdx.x; e < total; e += (size_t)gridDim.x * blockDim.x) {
    const T v = (T)Q[e];
    Qs[e] = v;
    Q[e] = (double)v;
  }
}

// Ac = S^T M S for real S (r x r, row-major) and complex M (r x r, interleaved,
// row-major): workgroup i forms row i, first u = S[:, i]^T M (a row, in LDS),
// then Ac[i][j] = sum_b u_b S[b][j]; sums in index order.
__global__ __launch_bounds__(128) void k_sandwich(int r, const double* __restrict__ S, const double* __restrict__ M,
                                                  double* __restrict__ Ac) {
  __shared__ double2 u[128];
  const int i = blockIdx.x, t = threadIdx.x;
  if (t < r) {
    double2 acc = czero();
    for (int a = 0; a < r; ++a) {
      const double sa = S[(size_t)a * r + i];
      acc.x += sa * M[2 * ((size_t)a * r + t)];
      acc.y += sa * M[2 * ((size_t)a * r + t) + 1];
    }
    u[t] = acc;
  }
  __syncthreads();
  if (t < r) {
    double2 acc = czero();
    for (int b = 0; b < r; ++b) {
      const double sb = S[(size_t)b * r + t];
      acc.x += u[b].x * sb;
      acc.y += u[b].y * sb;
    }
    Ac[2 * ((size_t)i * r + t)] = acc.x;
    Ac[2 * ((size_t)i * r + t) + 1] = acc.y;
  }
}

static unsigned ew_grid(size_t total) {
  size_t nb = (total + 255) / 256;
  if (nb > 16384) nb = 16384;
  if (nb < 1) nb = 1;
  return (unsigned)nb;
}

// ---- launchers used by other units ------------------------------------------------
// the kernels' instances by lanes per row and by whether rows are 16-byte aligned
template <typename T, typename S, int LD>
static void qt_launch(int lpr, int nb, size_t n, int r, const T* Q, const cplx_t<S>* x, double* part, hipStream_t st) {
  const dim3 grid(nb), block(64 * QT_WAVES);
  switch (lpr) {
    case 8: hipLaunchKernelGGL((k_qt_part<T, S, 8, LD>), grid, block, 0, st, n, r, Q, x, part); break;
    case 16: hipLaunchKernelGGL((k_qt_part<T, S, 16, LD>), grid, block, 0, st, n, r, Q, x, part); break;
    case 32: hipLaunchKernelGGL((k_qt_part<T, S, 32, LD>), grid, block, 0, st, n, r, Q, x, part); break;
    default: hipLaunchKernelGGL((k_qt_part<T, S, 64, LD>), grid, block, 0, st, n, r, Q, x, part);
  }
}
template <typename T, typename S, int MODE, int LD>
static void skinny_launch(int lpr, size_t n, int r, const T* Q, const double* c, cplx_t<S>* z, const uint8_t* mask,
                          const double* scal, hipStream_t st) {
  const size_t rows = 4 * 4 * (64 / lpr);  // of a workgroup's four wavefronts
  size_t nb = (n + rows - 1) / rows;
  if (nb > 1024) nb = 1024;
  const dim3 grid((unsigned)nb), block(256);
  switch (lpr) {
    case 8: hipLaunchKernelGGL((k_skinny<T, S, MODE, 8, LD>), grid, block, 0, st, n, r, Q, c, z, mask, scal); break;
    case 16: hipLaunchKernelGGL((k_skinny<T, S, MODE, 16, LD>), grid, block, 0, st, n, r, Q, c, z, mask, scal); break;
    case 32: hipLaunchKernelGGL((k_skinny<T, S, MODE, 32, LD>), grid, block, 0, st, n, r, Q, c, z, mask, scal); break;
    default: hipLaunchKernelGGL((k_skinny<T, S, MODE, 64, LD>), grid, block, 0, st, n, r, Q, c, z, mask, scal);
  }
}

// returns the number of partial rows written
template <typename T, typename S>
int qt_partials(size_t n, int r, const T* Q, const void* x, double* part, hipStream_t st) {
  const int nb = qt_nblocks(n, r, sizeof(T)), lpr = qt_lanes(r, sizeof(T));
  const cplx_t<S>* xc = (const cplx_t<S>*)x;
  kprof_begin(KP_QT, st);
  switch (q_load(n, r, sizeof(T))) {
    case LD_VALUES: qt_launch<T, S, LD_VALUES>(lpr, nb, n, r, Q, xc, part, st); break;
    case LD_CACHED: qt_launch<T, S, LD_CACHED>(lpr, nb, n, r, Q, xc, part, st); break;
    default: qt_launch<T, S, LD_STREAM>(lpr, nb, n, r, Q, xc, part, st);
  }
  kprof_end(KP_QT, (double)n * (sizeof(T) * r + 2 * sizeof(S)), st);
  return nb;
}

template <typename T, typename S>
void skinny_apply(size_t n, int r, const T* Q, const double* c, void* z, const uint8_t* mask, const double* scal,
                  int synth, hipStream_t st) {
  kprof_begin(KP_SKINNY, st);
  const int lpr = qt_lanes(r, sizeof(T));
  const int ld = q_load(n, r, sizeof(T));
  cplx_t<S>* zc = (cplx_t<S>*)z;
  auto launch = [&](auto mode) {
    constexpr int MODE = decltype(mode)::value;
    if (ld == LD_VALUES) skinny_launch<T, S, MODE, LD_VALUES>(lpr, n, r, Q, c, zc, mask, scal, st);
    else if (ld == LD_CACHED) skinny_launch<T, S, MODE, LD_CACHED>(lpr, n, r, Q, c, zc, mask, scal, st);
    else skinny_launch<T, S, MODE, LD_STREAM>(lpr, n, r, Q, c, zc, mask, scal, st);
  };
  if (synth) launch(std::integral_constant<int, SK_SYNTH>{});
  else launch(std::integral_constant<int, SK_ADD>{});
  // Q once; z read and written (ADD) or du written and the mask read (SYNTH)
  kprof_end(KP_SKINNY, (double)n * (sizeof(T) * r + (synth ? 2 * sizeof(S) + 1 : 4 * sizeof(S))), st);
}
template void skinny_apply<double, double>(size_t, int, const double*, const double*, void*, const uint8_t*,
                                           const double*, int, hipStream_t);
template void skinny_apply<float, float>(size_t, int, const float*, const double*, void*, const uint8_t*,
                                         const double*, int, hipStream_t);
template void skinny_apply<float, double>(size_t, int, const float*, const double*, void*, const uint8_t*,
                                          const double*, int, hipStream_t);

// ---- setup -----------------------------------------------------------------------
void coarse_trim(helm_op_s* op) {
  Coarse& c = op->coarse;
  c.T.release();
  c.T_serial = -1;
  c.W1.release();
  c.W2.release();
}

void coarse_release(helm_op_s* op) {
  Coarse& c = op->coarse;
  c.Q.release();
  c.Ainv.release();
  c.Ac.release();
  c.T.release();
  c.W1.release();
  c.W2.release();
  c.small.release();
  c.qpart.release();
  if (c.pending) {
    (void)hipEventSynchronize(c.ev1);
    (void)hipEventDestroy(c.ev0);
    (void)hipEventDestroy(c.ev1);
    c.pending = false;
  }
  c.valid = false;
  c.T_serial = -1;
}

// Checks the inverse's record (8 ints, then the condition estimate) that the
// set-up copied to host memory, and settles the space: valid with its
// condition estimate and set-up time, or invalid with the error.
static helm_status coarse_settle(helm_op_s* op, const void* rec_host) {
  Coarse& c = op->coarse;
  const int* rec = (const int*)rec_host;
  helm_status s = HELM_OK;
  if (!c.pass1 && (rec[3] != 0 || rec[2] != c.rank))
    s = fail(HELM_E_SINGULAR, "coarse: second CholeskyQR pass lost rank (%d of %d)", rec[2], c.rank);
  else if (rec[0] != 0)
    s = fail(HELM_E_SINGULAR, "coarse: A_c is singular (zero pivot)");
  c.cond_est = *(const double*)(rec + 8);
  float ms = 0.f;
  (void)hipEventElapsedTime(&ms, c.ev0, c.ev1);
  c.setup_ms = ms;
  (void)hipEventDestroy(c.ev0);
  (void)hipEventDestroy(c.ev1);
  c.pending = false;
  c.valid = s == HELM_OK;
  return s;
}

helm_status coarse_finish(helm_op_s* op) {
  Coarse& c = op->coarse;
  if (!c.pending) return HELM_OK;
  hipError_t e = hipEventSynchronize(c.ev1);
  if (e != hipSuccess) {
    (void)hipEventDestroy(c.ev0);
    (void)hipEventDestroy(c.ev1);
    c.pending = false;
    c.valid = false;
    return hip_fail(e, "coarse: inverse wait");
  }
  return coarse_settle(op, op->host + COARSE_REC);
}

template <typename TT, typename S>
static helm_status coarse_build(helm_op_s* op, don_s* net, int p_used, bool qf32, bool defer, hipStream_t st) {
  Coarse& c = op->coarse;
  const size_t n = op->nn;
  helm_status s;
  hipEvent_t e0, e1;
  (void)hipEventCreate(&e0);
  (void)hipEventCreate(&e1);
  (void)hipEventRecord(e0, st);
  // trunk matrix at the op's nodes (cached per network)
  const int p = don_p(net);
  if (c.T_serial != don_serial(net)) {
    if ((s = c.T.ensure(n * (size_t)p * sizeof(TT)))) return s;
    if ((s = don_trunk(net, op, c.T.ptr, st))) return s;
    c.T_serial = don_serial(net);
  }
  const int pu = p_used;
  // fp64 trunk (C128): P is the masked trunk matrix itself, read with its row
  // stride p; fp32 trunk (C64): P is widened into W1
  const bool wide_t = sizeof(TT) == sizeof(double);
  c.q_f32 = qf32 || !wide_t;
  c.pass1 = !c.q_f32;  // fp64 basis: the first pass's basis is the one used
  if (!wide_t && (s = c.W1.ensure(n * (size_t)pu * sizeof(double)))) return s;
  if (c.q_f32 && (s = c.W2.ensure(n * (size_t)pu * sizeof(double)))) return s;
  const size_t small_doubles = gram_part(n, pu) + 7 * (size_t)pu * pu + 4096;
  if ((s = c.small.ensure(small_doubles * sizeof(double)))) return s;
  double* part = (double*)c.small.ptr;
  double* G = part + gram_part(n, pu);
  double* S1 = G + (size_t)pu * pu;
  double* G2 = S1 + (size_t)pu * pu;
  double* gjw = G2 + (size_t)pu * pu;  // 4 pu^2
  int* info = (int*)(gjw + 4 * (size_t)pu * pu);
  double* cond = (double*)(info + 8);
  double* Q1 = (double*)c.W2.ptr;
  // P = masked first pu columns of T
  const double* P;
  size_t ldp;
  if (wide_t) {
    const size_t nbz = std::min<size_t>((n + 3) / 4, 8192);
    hipLaunchKernelGGL((k_zero_masked_rows<TT>), dim3((unsigned)nbz), dim3(64, 4), 0, st, n, p, op->mask,
                       (TT*)c.T.ptr);
    P = (const double*)c.T.ptr;
    ldp = (size_t)p;
  } else {
    hipLaunchKernelGGL((k_mask_cols<TT>), dim3(ew_grid(n * pu)), dim3(256), 0, st, n, p, pu, (const TT*)c.T.ptr,
                       op->mask, (double*)c.W1.ptr);
    P = (const double*)c.W1.ptr;
    ldp = (size_t)pu;
  }
  // pass 1: G = P^T P, Cholesky with dropping -> S1 (pu x r)
  gram(n, pu, P, ldp, part, G, st);
  const double tau = op->dt == HELM_C128 ? 1e-7 : 1e-5;
  chol_drop(pu, G, tau * tau, 1, S1, info, st);
  hipError_t e = hipMemcpyAsync(op->host, info, 2 * sizeof(int), hipMemcpyDeviceToHost, st);
  if (e != hipSuccess) return hip_fail(e, "coarse: rank readback");
  if ((s = sync_stream(st, "coarse: pass 1"))) return s;
  const int r = ((int*)op->host)[0];
  c.rank = r;
  c.p_used = pu;
  if (r == 0) {
    c.valid = true;
    c.cond_est = 0.0;
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    return HELM_OK;
  }
  if ((s = c.Q.ensure(n * (size_t)r * (c.q_f32 ? sizeof(float) : sizeof(double)))) ||
      (s = c.W1.ensure(n * (size_t)r * sizeof(double))) || (s = c.Ac.ensure(2 * sizeof(double) * r * r)) ||
      (s = c.Ainv.ensure(2 * sizeof(double) * r * r)) ||
      (s = c.qpart.ensure(sizeof(double) * 2 * (size_t)r * qt_nblocks(n, r, c.q_f32 ? sizeof(float) : sizeof(double)))))
    return s;
  // the Galerkin matrix X^T A X = X^T B - i X^T diag(Im s) X of an n x r basis
  // X into out (complex r x r), B = (L - diag(Re s)) X
  auto galerkin = [&](const double* X, double* B, double* out) {
    auto lap = r % 2 ? k_batched_lap<S, 1> : k_batched_lap<S, 2>;  // rows of an odd length are not 16-byte aligned
    // eight wavefronts per SIMD, if need be by shorter marches
    const size_t nxy = n / op->geom.nz, want = (8192 + nxy - 1) / nxy;
    const int seg = std::max(1, (int)(op->geom.nz / want));
    const size_t waves = nxy * ((op->geom.nz + seg - 1) / seg);
    // 2^26 wavefronts per launch (a 2D grid has one per node): below 2^32 work-items on an axis
    constexpr size_t WMAX = (size_t)1 << 26;
    for (size_t w0 = 0; w0 < waves; w0 += WMAX)
      hipLaunchKernelGGL(lap, dim3((unsigned)((std::min(waves - w0, WMAX) + 3) / 4)), dim3(64, 4), 0, st, op->geom, r,
                         seg, w0, X, (const cplx_t<S>*)op->sc, op->code, B);
    gram_galerkin<S>(n, r, X, B, (const cplx_t<S>*)op->sc, part, out, st);
  };
  double* Ac = (double*)c.Ac.ptr;
  if (c.pass1) {
    // fp64 basis: the solves use Q1 = P S1 itself.  The correction
    // Q (Q^T A Q)^{-1} Q^T depends only on the span of the basis, and Q1 spans
    // what Q = Q1 S2 spans (Q1^T Q1 = I up to about cond(P)^2 eps <= 1e-2 at
    // the drop threshold, so Q1^T A Q1 is as well conditioned as A_c); the
    // second pass is run only when the orthonormal basis is inspected.
    basis(n, pu, r, P, ldp, S1, r == pu, (double*)c.Q.ptr, st);
    galerkin((const double*)c.Q.ptr, (double*)c.W1.ptr, Ac);
  } else {
    // fp32 stored basis (when requested, or for C64): CholeskyQR2, Q rounded
    // to its stored values, A_c formed from the rounded basis.  Pass 2:
    // G2 = Q1^T Q1, Cholesky without dropping -> S2 (r x r, into S1); its rank
    // record goes to info[2..3], read back with the inverse's record (every
    // kernel below is sized by r alone, so a lost rank only spoils values).
    basis(n, pu, r, P, ldp, S1, r == pu, Q1, st);
    gram(n, r, Q1, r, part, G2, st);
    chol_drop(r, G2, 0.0, 0, S1, info + 2, st);
    double* Q = (double*)c.W1.ptr;
    basis(n, r, r, Q1, r, S1, true, Q, st);
    // Q <- its stored values (rounded in place), then B in Q1
    hipLaunchKernelGGL((k_round_q<float>), dim3(ew_grid(n * r)), dim3(256), 0, st, n * (size_t)r, Q, (float*)c.Q.ptr);
    galerkin(Q, Q1, Ac);
  }
  gj_inverse(r, Ac, nullptr, (double*)c.Ainv.ptr, info, cond, st);
  // the inverse's record goes to its own pinned slot; with defer set the
  // space is returned pending and the record is checked by coarse_finish
  // (a caller that waits on later work in the stream finds it complete)
  e = hipMemcpyAsync(op->host + COARSE_REC, info, sizeof(int) * 8 + sizeof(double), hipMemcpyDeviceToHost, st);
  if (e != hipSuccess) return hip_fail(e, "coarse: inverse readback");
  (void)hipEventRecord(e1, st);
  c.ev0 = e0;
  c.ev1 = e1;
  c.pending = true;
  c.valid = true;
  if ((s = launch_check("coarse setup"))) return s;
  return defer ? HELM_OK : coarse_finish(op);
}

helm_status coarse_ensure(helm_op_s* op, don_s* net, int p_used, bool q_fp32, bool no_drop, hipStream_t st,
                          bool defer) {
  Coarse& c = op->coarse;
  helm_status s0 = coarse_finish(op);  // a space left pending by an earlier call
  if (s0) return s0;
  const bool want_f32 = q_fp32 || op->dt == HELM_C64;
  if (!(c.valid && c.net_serial == don_serial(net) && c.p_used == p_used && c.ksq_version == op->ksq_version &&
        c.q_f32 == want_f32)) {
    c.valid = false;
    helm_status s = op->dt == HELM_C128 ? coarse_build<double, double>(op, net, p_used, q_fp32, defer, st)
                                        : coarse_build<float, float>(op, net, p_used, true, defer, st);
    if (s) return s;
    c.net_serial = don_serial(net);
    c.ksq_version = op->ksq_version;
  }
  // the space stays cached either way: a later call that allows dropping uses it
  if (no_drop && c.rank < p_used)
    return fail(HELM_E_SINGULAR, "coarse: %d of the %d trunk columns are numerically dependent and no_drop is set",
                p_used - c.rank, p_used);
  return HELM_OK;
}

helm_status coarse_orthonormal(helm_op_s* op, double* Qout, double* Acout, hipStream_t st) {
  Coarse& c = op->coarse;
  if (!c.valid || !c.pass1) return fail(HELM_E_INVAL, "coarse: no first-pass basis to orthonormalize");
  const size_t n = op->nn;
  const int r = c.rank, pu = c.p_used;
  if (r == 0) return HELM_OK;
  // the regions of the set-up's small buffer (laid out as in coarse_build)
  double* part = (double*)c.small.ptr;
  double* G = part + gram_part(n, pu);
  double* S2 = G + (size_t)pu * pu;
  double* G2 = S2 + (size_t)pu * pu;
  double* gjw = G2 + (size_t)pu * pu;
  int* info = (int*)(gjw + 4 * (size_t)pu * pu);
  const double* Q1 = (const double*)c.Q.ptr;
  // second CholeskyQR pass: G2 = Q1^T Q1 = S2^-T S2^-1
  gram(n, r, Q1, r, part, G2, st);
  chol_drop(r, G2, 0.0, 0, S2, info + 2, st);
  if (Qout) basis(n, r, r, Q1, r, S2, true, Qout, st);
  hipError_t e;
  if (Acout) {
    // A_c = Q^T A Q = S2^T (Q1^T A Q1) S2, formed in the work region, copied out
    hipLaunchKernelGGL(k_sandwich, dim3(r), dim3(128), 0, st, r, (const double*)S2, (const double*)c.Ac.ptr, gjw);
    e = hipMemcpyAsync(Acout, gjw, sizeof(double) * 2 * r * r, hipMemcpyDeviceToHost, st);
    if (e != hipSuccess) return hip_fail(e, "coarse: A_c readback");
  }
  e = hipMemcpyAsync(op->host, info + 2, 2 * sizeof(int), hipMemcpyDeviceToHost, st);
  if (e != hipSuccess) return hip_fail(e, "coarse: second pass readback");
  helm_status s = sync_stream(st, "coarse: second pass");
  if (s) return s;
  const int* rec = (const int*)op->host;
  if (rec[1] != 0 || rec[0] != r)
    return fail(HELM_E_SINGULAR, "coarse: second CholeskyQR pass lost rank (%d of %d)", rec[0], r);
  return launch_check("coarse: orthonormal basis");
}

template <typename S>
helm_status coarse_correct(helm_op_s* op, const void* r1, void* z, hipStream_t st) {
  Coarse& c = op->coarse;
  const int r = c.rank;
  if (r == 0) return HELM_OK;
  const size_t n = op->nn;
  double* part = (double*)c.qpart.ptr;
  double* cc = op->red + 2048;
  const int nb = c.q_f32 ? qt_partials<float, S>(n, r, (const float*)c.Q.ptr, r1, part, st)
                         : qt_partials<double, S>(n, r, (const double*)c.Q.ptr, r1, part, st);
  hipLaunchKernelGGL(k_reduce_ainv, dim3((r + 15) / 16), dim3(1024), 0, st, r, nb, (const double*)part,
                     (const double*)c.Ainv.ptr, cc);
  if (c.q_f32) skinny_apply<float, S>(n, r, (const float*)c.Q.ptr, cc, z, op->mask, nullptr, 0, st);
  else skinny_apply<double, S>(n, r, (const double*)c.Q.ptr, cc, z, op->mask, nullptr, 0, st);
  return launch_check("coarse correction");
}

template helm_status coarse_correct<double>(helm_op_s*, const void*, void*, hipStream_t);
template helm_status coarse_correct<float>(helm_op_s*, const void*, void*, hipStream_t);

}  // namespace helm
