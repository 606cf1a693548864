// Dense kernels: the DeepONet layers (MFMA GEMM with fused bias + activation,
// split-K GEMV for small batches, the coordinate input layer of the trunk),
// and one-workgroup factorizations of small matrices (Cholesky with column
// dropping, triangular inverse, Gauss-Jordan inverse of the complex coarse
// matrix).
// Both dtypes evaluate the network layers in fp64 (a C64 network's fp32
// weights widened exactly).
#include "common.h"
#include "dense_dev.h"
#include "prof.h"

namespace helm {

// ---- trunk input layer: h = act(x W + b) at grid-node coordinates --------------
// Workgroup b takes rows [b rpb, (b + 1) rpb) of the output, threads its
// columns (W and b of a column loaded once); the node indices of the first
// row come from one division, the next rows by stepping x, then y, then z.
constexpr int CL_TAB = 1024;  // node coordinates tabulated in LDS per axis up to this length
template <typename T, bool TABBED>
__global__ __launch_bounds__(256) void k_coord_layer(int dim, int nx, int ny, int nz, size_t row0, size_t nrows,
                                                     size_t rpb, const T* __restrict__ W, const T* __restrict__ b,
                                                     int N, int act, T* __restrict__ out) {
  // TABBED: coordinate x_i = (i + 1) / (n + 1) of each axis formed once per
  // workgroup (the same quotients every element would form)
  __shared__ T tab[3][TABBED ? CL_TAB : 1];
  constexpr bool tabbed = TABBED;
  if (tabbed) {
    for (int i = threadIdx.x; i < nx; i += blockDim.x) tab[0][i] = T(i + 1) / T(nx + 1);
    for (int i = threadIdx.x; i < ny; i += blockDim.x) tab[1][i] = T(i + 1) / T(ny + 1);
    for (int i = threadIdx.x; i < nz; i += blockDim.x) tab[2][i] = T(i + 1) / T(nz + 1);
    __syncthreads();
  }
  const size_t r0 = (size_t)blockIdx.x * rpb, r1 = min(nrows, r0 + rpb);
  if (r0 >= r1) return;
  const size_t p0 = row0 + r0;
  int ix = (int)(p0 % nx), iy = (int)((p0 / nx) % ny), iz = (int)(p0 / ((size_t)nx * ny));
  for (int c0 = 0; c0 < N; c0 += blockDim.x) {
    const int c = c0 + threadIdx.x;
    const bool on = c < N;
    const T w0 = on ? W[c] : T(0), w1 = on && dim > 1 ? W[(size_t)N + c] : T(0),
            w2 = on && dim > 2 ? W[2 * (size_t)N + c] : T(0), bc = on ? b[c] : T(0);
    int jx = ix, jy = iy, jz = iz;
    for (size_t r = r0; r < r1; ++r) {
      if (on) {
        const T xc[3] = {tabbed ? tab[0][jx] : T(jx + 1) / T(nx + 1), tabbed ? tab[1][jy] : T(jy + 1) / T(ny + 1),
                         tabbed ? tab[2][jz] : T(jz + 1) / T(nz + 1)};
        T acc = xc[0] * w0;
        if (dim > 1) acc += xc[1] * w1;
        if (dim > 2) acc += xc[2] * w2;
        out[r * (size_t)N + c] = activate<T>(acc + bc, act);
      }
      if (++jx == nx) {
        jx = 0;
        if (++jy == ny) {
          jy = 0;
          ++jz;
        }
      }
    }
  }
}

// ---- MFMA GEMM: C = act(A W + b) ---------------------------------------------
// A: M x K (lda), W: K x N (ldw), C: M x N (ldc), all row-major.  128 x 128 tile
// per workgroup of four wavefronts, each 64 x 64 (4 x 4 MFMA tiles, so every
// operand value read from LDS feeds four products); K staged 16 at a time
// through LDS (A stored k-major) with the next chunk's loads in registers while
// the current chunk is multiplied.  Products are accumulated in k order, four
// at a time.
constexpr int GB_M = 128, GB_N = 128, GB_K = 16, GB_PAD = 4;

template <typename T>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) void k_gemm(int M, int N, int K, const T* __restrict__ A, size_t lda,
                                              const T* __restrict__ W, size_t ldw, const T* __restrict__ bias,
                                              int act, T* __restrict__ C, size_t ldc) {
  __shared__ T As[GB_K][GB_M + GB_PAD];
  __shared__ T Ws[GB_K][GB_N + GB_PAD];
  const int nbn = (N + GB_N - 1) / GB_N;
  const unsigned lb = xcd_remap(blockIdx.x, gridDim.x);
  const int bm = (int)(lb / nbn) * GB_M, bn = (int)(lb % nbn) * GB_N;
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const int wm = (wave >> 1) * 64, wn = (wave & 1) * 64;
  d4 acc[4][4];
#pragma unroll
  for (int a = 0; a < 4; ++a)
#pragma unroll
    for (int b = 0; b < 4; ++b) acc[a][b] = d4{0, 0, 0, 0};
  // A chunk: 128 rows x 16 k (16 consecutive threads read 16 consecutive k of a
  // row); W chunk: 16 k x 128 n (consecutive threads read consecutive n)
  T va[8], vw[8];
  auto load = [&](int k0) {
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      const int e = t + 256 * q;
      const int r = e >> 4, kk = e & 15, gr = bm + r, gk = k0 + kk;
      va[q] = (gr < M && gk < K) ? A[(size_t)gr * lda + gk] : T(0);
      const int wk = e >> 7, c = e & 127, gkw = k0 + wk, gn = bn + c;
      vw[q] = (gkw < K && gn < N) ? W[(size_t)gkw * ldw + gn] : T(0);
    }
  };
  load(0);
  for (int k0 = 0; k0 < K; k0 += GB_K) {
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      const int e = t + 256 * q;
      As[e & 15][e >> 4] = va[q];
      Ws[e >> 7][e & 127] = vw[q];
    }
    __syncthreads();
    if (k0 + GB_K < K) load(k0 + GB_K);
#pragma unroll
    for (int kk = 0; kk < GB_K; kk += 4) {
      T av[4], bv[4];
#pragma unroll
      for (int a = 0; a < 4; ++a) av[a] = As[kk + (lane >> 4)][wm + a * 16 + (lane & 15)];
#pragma unroll
      for (int b = 0; b < 4; ++b) bv[b] = Ws[kk + (lane >> 4)][wn + b * 16 + (lane & 15)];
#pragma unroll
      for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int b = 0; b < 4; ++b) acc[a][b] = mfma16(av[a], bv[b], acc[a][b]);
    }
    __syncthreads();
  }
#pragma unroll
  for (int a = 0; a < 4; ++a)
#pragma unroll
    for (int b = 0; b < 4; ++b)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int gr = bm + wm + a * 16 + acc_row(lane, i);
        const int gc = bn + wn + b * 16 + (lane & 15);
        if (gr < M && gc < N) {
          T v = acc[a][b][i];
          if (bias) v += bias[gc];
          C[(size_t)gr * ldc + gc] = activate<T>(v, act);
        }
      }
}

// ---- small-batch dense layer (GEMV class), split over K ------------------------
// part[ks][b][n] = sum_{k in split ks} x[b][k] W[k][n]; then finalize adds the
// splits in order, the bias and the activation.
constexpr int SK_COLS = 64;
template <typename T>
__global__ __launch_bounds__(256) void k_small_part(int B, int N, int K, int ksplit, const T* __restrict__ x,
                                                    const T* __restrict__ W, double* __restrict__ part) {
  __shared__ double sh[4][4][SK_COLS];
  const int ncb = (N + SK_COLS - 1) / SK_COLS;
  const int cb = blockIdx.x % ncb, ks = blockIdx.x / ncb;
  const int lane = threadIdx.x & 63, grp = threadIdx.x >> 6;
  const int col = cb * SK_COLS + lane;
  const int kchunk = (K + ksplit - 1) / ksplit;
  const int kb = ks * kchunk, ke = min(K, kb + kchunk);
  double acc[4] = {0, 0, 0, 0};
  if (col < N)
    for (int k = kb + grp; k < ke; k += 4) {
      const double w = (double)W[(size_t)k * N + col];
      for (int b = 0; b < B; ++b) acc[b] += (double)x[(size_t)b * K + k] * w;
    }
  for (int b = 0; b < 4; ++b) sh[grp][b][lane] = acc[b];
  __syncthreads();
  if (grp == 0 && col < N)
    for (int b = 0; b < B; ++b)
      part[((size_t)ks * B + b) * N + col] = (sh[0][b][lane] + sh[1][b][lane]) + (sh[2][b][lane] + sh[3][b][lane]);
}

template <typename T>
__global__ void k_small_final(int B, int N, int ksplit, const double* __restrict__ part, const T* __restrict__ bias,
                              int act, T* __restrict__ y) {
  const int e = blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= B * N) return;
  const int b = e / N, n = e % N;
  double acc = 0.0;
  for (int ks = 0; ks < ksplit; ++ks) acc += part[((size_t)ks * B + b) * N + n];
  if (bias) acc += (double)bias[n];
  y[e] = (T)activate<double>(acc, act);  // fp64 arithmetic, rounded once to the stored type
}

// one lane's value, wave-uniform; the largest of a wavefront
__device__ __forceinline__ double lane_val(double v, int lane) {
  return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), lane),
                          __builtin_amdgcn_readlane(__double2loint(v), lane));
}
template <int CTRL>
__device__ __forceinline__ double dpp_max(double v) {
  const int lo = __double2loint(v), hi = __double2hiint(v);
  return fmax(v, __hiloint2double(__builtin_amdgcn_update_dpp(hi, hi, CTRL, 0xf, 0xf, false),
                                  __builtin_amdgcn_update_dpp(lo, lo, CTRL, 0xf, 0xf, false)));
}
__device__ __forceinline__ double wave_max(double v) {
  v = dpp_max<0xB1>(dpp_max<0x4E>(dpp_max<0x141>(dpp_max<0x140>(v))));  // within the 16-lane rows
  return fmax(fmax(lane_val(v, 0), lane_val(v, 16)), fmax(lane_val(v, 32), lane_val(v, 48)));
}

// ---- one-workgroup Cholesky with column dropping -------------------------------
// G: p x p (symmetric, fp64) = P^T P, p <= 128.  G = R^T R column by column; a
// column whose Schur-complement diagonal is <= tau2 * max_j G[j][j] is dropped (its
// remaining norm is at most tau times the largest column norm), which matches
// Householder QR that skips such columns.  Outputs: S (p x r row-major) with
// S[kept[a]][:] = (R1^{-1})[a][:] (R1: the kept rows and columns of R) and zero
// rows for dropped columns, so that Q = P S has orthonormal columns in exact
// arithmetic; info[0] = r; info[1] = 1 if a column had to be dropped while
// allow_drop = 0.
//
// R1^{-1} comes out of the elimination itself: with G = L D L^T (L unit lower,
// R = D^{1/2} L^T) the steps that turn G into D L^T turn I into L^{-1}, and
// R1^{-1} = L^{-T} D^{-1/2}.  L^{-1} fills the lower triangle that the
// elimination leaves free: step j takes (row a's entry j) / d_j times row j from
// every row a > j (the still symmetric part of G right of column j, L^{-1} left of
// it), and column j becomes minus that factor.  The matrix stays in registers:
// thread (tx, ty) of a 32 x 32 grid holds rows tx + 32 v, columns ty + 32 u; row j is
// published in LDS, double-buffered, one barrier per step.
// What bounds it: the serial chain of p steps (row through LDS, reciprocal, the
// next row's update).  Factoring with a square root and a division per step and
// then inverting row by row in LDS took 241 us at p = 128 (75 at 48);
// this takes 92 us (35).
__global__ __launch_bounds__(1024) void k_chol_drop(int p, const double* __restrict__ G, double tau2, int allow_drop,
                                                    double* __restrict__ S, int* __restrict__ info) {
  __shared__ double rowj[2][128];
  __shared__ double dpiv[128];  // d_j of a kept column
  __shared__ int slot[128];     // its place among the kept columns; -1: dropped
  __shared__ double s_max[2];
  const int t = threadIdx.x, tx = t & 31, ty = t >> 5;
  double g[4][4];
#pragma unroll
  for (int u = 0; u < 4; ++u)
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int a = tx + 32 * v, c = ty + 32 * u;
      g[u][v] = (a < p && c < p) ? G[c * p + a] : 0.0;
    }
  if (t < 128) {  // largest squared column norm of P
    const double m = wave_max(t < p ? G[t * p + t] : 0.0);
    if ((t & 63) == 0) s_max[t >> 6] = m;
  }
  int nk = 0;
  bool fail = false;
  double thr2 = 0.0;
  for (int j = 0; j < p; ++j) {
    double* row = rowj[j & 1];
    if (tx == (j & 31))
#pragma unroll
      for (int v = 0; v < 4; ++v)
        if (v == j >> 5)
#pragma unroll
          for (int u = 0; u < 4; ++u) row[ty + 32 * u] = g[u][v];
    __syncthreads();
    if (j == 0) thr2 = tau2 * fmax(s_max[0], s_max[1]);
    const double dj = row[j];
    const bool keep = dj > thr2;
    if (t == 0) {
      slot[j] = keep ? nk : -1;
      dpiv[j] = dj;
    }
    if (keep) {
      ++nk;
      double ra[4], rc[4];
#pragma unroll
      for (int v = 0; v < 4; ++v) ra[v] = tx + 32 * v > j ? row[tx + 32 * v] : 0.0;
#pragma unroll
      for (int u = 0; u < 4; ++u) rc[u] = row[ty + 32 * u];
      const double dinv = 1.0 / dj;
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        ra[v] *= dinv;
#pragma unroll
        for (int u = 0; u < 4; ++u) g[u][v] = fma(-ra[v], rc[u], g[u][v]);
      }
      if (ty == (j & 31))
#pragma unroll
        for (int u = 0; u < 4; ++u)
          if (u == j >> 5)
#pragma unroll
            for (int v = 0; v < 4; ++v)
              if (tx + 32 * v > j) g[u][v] = -ra[v];
    } else {
      fail |= !allow_drop;
    }
  }
  __syncthreads();
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    const int a = tx + 32 * v, b = a < p ? slot[a] : -1;
    if (b < 0) continue;
    const double pinv = 1.0 / sqrt(dpiv[a]);
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int c = ty + 32 * u;
      if (c < p) S[(size_t)c * nk + b] = c == a ? pinv : c < a && slot[c] >= 0 ? g[u][v] * pinv : 0.0;
    }
  }
  if (t == 0) {
    info[0] = nk;
    info[1] = fail;
  }
}

// ---- Gauss-Jordan inverse of a complex r x r matrix (r <= 128), one workgroup ----
// In-place Gauss-Jordan with partial pivoting (largest |Re| + |Im| among the rows
// not yet used as pivot rows, lowest row on ties), without moving rows, eight
// columns at a time.  A panel's eight steps touch only its own columns: wavefront 8
// takes the 128 x 8 panel in registers (lane l rows l and l + 64), with no
// barrier between pivots.  They leave in the panel the columns F_t = G
// e_{p_t} of the transformation G of the eight steps (p_t: step t's pivot row);
// every other column a becomes G a = a with its pivot rows zeroed + sum_t
// a[p_t] F_t, a product of depth eight that wavefronts 0 .. 7 run on the matrix
// pipe, the matrix in their accumulators (wavefront w: rows 16 w .. + 15, eight
// 16 x 16 tiles, Re and Im).  They update the next panel's columns first, so its
// pivots are found while the other columns are updated.  Row p of the final
// table is row k of the inverse where p was column k's pivot row, and its column c
// is column p_c (the pivot row of column c) of the inverse.  The matrix is padded
// with the identity to whole blocks.  info[0] = 1 if a pivot was zero or
// non-finite; cond[0] = ||A||_1 ||A^{-1}||_1.
// What bounds it: the panels' chain of pivot searches, reciprocals and rank-one
// updates in one wavefront; the products (55 us of one CU's fp64 rate at r = 128)
// run beside it.  One pivot at a time over the whole matrix, two barriers and
// 563 instructions each, took 378 us at r = 128 (118 at 48); this one
// takes 187 us (55 at 48).
constexpr int GJ_P = 8;
// 1 / z, scaled by the exponent of the larger part (no overflow of |z|^2)
__device__ __forceinline__ double2 crcp(double2 z) {
  const int k = -ilogb(fmax(fabs(z.x), fabs(z.y)));
  const double x = ldexp(z.x, k), y = ldexp(z.y, k), d = x * x + y * y;  // d in [1, 8)
  double v = __builtin_amdgcn_rcp(d);
  v = fma(v, fma(-d, v, 1.0), v);
  v = fma(v, fma(-d, v, 1.0), v);
  return make_double2(ldexp(x * v, k), ldexp(-y * v, k));
}

__global__ __launch_bounds__(576) void k_gj_inverse(int r, const double* __restrict__ A, double* __restrict__ Ainv,
                                                    int* __restrict__ info, double* __restrict__ cond) {
  // panel kp (then its F), its pivot rows' entries in all columns, and each
  // row's step in it (-1: none), alternating
  __shared__ double2 pan[2][128][GJ_P + 1], prow[2][GJ_P][128 + 2];
  __shared__ int rowt[2][128];
  __shared__ double csum[128], npart[4][128];
  __shared__ int perm[128], rowof[128];
  __shared__ int s_bad;
  const int t = threadIdx.x, lane = t & 63, w = __builtin_amdgcn_readfirstlane(t >> 6);
  const int m = lane & 15, g = lane >> 4;
  const int nb = (r + 15) / 16, np = 2 * nb;
  // ||M||_1 partials: column t % 128 over rows t / 128 + 4 u (coalesced), later added in order
  auto norm1 = [&](const double2* M) {
    const int c = t & 127, r0 = t >> 7;
    if (r0 > 3) return;
    double sm = 0.0;
    if (c < r)
      for (int i = r0; i < r; i += 4) {
        const double2 v = M[(size_t)i * r + c];
        sm += hypot(v.x, v.y);
      }
    npart[r0][c] = sm;
  };
  norm1(reinterpret_cast<const double2*>(A));
  if (t == 0) s_bad = 0;
  if (t < 128) {
    rowof[t] = t;  // every row maps in range even if a failed pivot search repeats a row
    perm[t] = t;
  }
  __syncthreads();
  if (t < 128) csum[t] = (npart[0][t] + npart[1][t]) + (npart[2][t] + npart[3][t]);
  if (w == 8) {
    __syncthreads();  // panel 0 is laid out
    bool used0 = lane >= 16 * nb, used1 = lane + 64 >= 16 * nb;
    for (int kp = 0; kp < np; ++kp) {
      double2(*pn)[GJ_P + 1] = pan[kp & 1];
      double2 v0[GJ_P], v1[GJ_P];
#pragma unroll
      for (int c = 0; c < GJ_P; ++c) {
        v0[c] = pn[lane][c];
        v1[c] = pn[lane + 64][c];
      }
      int t0 = -1, t1 = -1;
#pragma unroll
      for (int c = 0; c < GJ_P; ++c) {
        const double a0 = used0 ? -1.0 : fabs(v0[c].x) + fabs(v0[c].y);
        const double a1 = used1 ? -1.0 : fabs(v1[c].x) + fabs(v1[c].y);
        const double best = wave_max(fmax(a0, a1));
        const unsigned long long b0 = __ballot(a0 == best), b1 = __ballot(a1 == best);
        const int p = b0 ? __ffsll(b0) - 1 : b1 ? 63 + __ffsll(b1) : 0;
        const int pl = p & 63;
        // the pivot row (uniform) times 1 / pivot; every other row minus (its entry / pivot) times the pivot row
        double2 pr[GJ_P], f0, f1, ipiv;
        if (p < 64) {
#pragma unroll
          for (int j = 0; j < GJ_P; ++j) pr[j] = make_double2(lane_val(v0[j].x, pl), lane_val(v0[j].y, pl));
          ipiv = crcp(pr[c]);
          f0 = cmul(v0[c], ipiv);
          f1 = cmul(v1[c], ipiv);
          if (lane == pl) {
            used0 = true;
            t0 = c;
            f0 = make_double2(-ipiv.x, -ipiv.y);
#pragma unroll
            for (int j = 0; j < GJ_P; ++j) v0[j] = czero();
          }
        } else {
#pragma unroll
          for (int j = 0; j < GJ_P; ++j) pr[j] = make_double2(lane_val(v1[j].x, pl), lane_val(v1[j].y, pl));
          ipiv = crcp(pr[c]);
          f0 = cmul(v0[c], ipiv);
          f1 = cmul(v1[c], ipiv);
          if (lane == pl) {
            used1 = true;
            t1 = c;
            f1 = make_double2(-ipiv.x, -ipiv.y);
#pragma unroll
            for (int j = 0; j < GJ_P; ++j) v1[j] = czero();
          }
        }
        pr[c] = make_double2(1.0, 0.0);
        v0[c] = v1[c] = czero();
#pragma unroll
        for (int j = 0; j < GJ_P; ++j) {
          v0[j].x = fma(-f0.x, pr[j].x, fma(f0.y, pr[j].y, v0[j].x));
          v0[j].y = fma(-f0.x, pr[j].y, fma(-f0.y, pr[j].x, v0[j].y));
          v1[j].x = fma(-f1.x, pr[j].x, fma(f1.y, pr[j].y, v1[j].x));
          v1[j].y = fma(-f1.x, pr[j].y, fma(-f1.y, pr[j].x, v1[j].y));
        }
        if (lane == 0) {
          perm[GJ_P * kp + c] = p;
          rowof[p] = GJ_P * kp + c;
          if (!(best > 0.0) || !isfinite(best)) s_bad = 1;
        }
      }
#pragma unroll
      for (int c = 0; c < GJ_P; ++c) {
        pn[lane][c] = v0[c];
        pn[lane + 64][c] = v1[c];
      }
      rowt[kp & 1][lane] = t0;
      rowt[kp & 1][lane + 64] = t1;
      __syncthreads();  // F is there
      __syncthreads();  // its pivot rows are published
      __syncthreads();  // the next panel is laid out
    }
  } else {
    const bool on = w < nb;
    const double2* A2 = reinterpret_cast<const double2*>(A);
    // tile q holds column block (q + rot) & 7: the tiles move down one place after
    // each two panels, so the panel's own tile is tile 0 and no index is dynamic
    d4 re[8], im[8];
    int rot = 0;
#pragma unroll
    for (int q = 0; q < 8; ++q)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int row = 16 * w + acc_row(lane, i), col = 16 * q + m;
        const double2 v = row < r && col < r ? A2[(size_t)row * r + col] : make_double2(row == col ? 1.0 : 0.0, 0.0);
        re[q][i] = v.x;
        im[q][i] = v.y;
      }
    // half h of tile q as a panel
    auto lay_out = [&](int h, const d4& x, const d4& y) {
      if (on && (m >> 3) == h)
#pragma unroll
        for (int i = 0; i < 4; ++i) pan[h][16 * w + acc_row(lane, i)][m & 7] = make_double2(x[i], y[i]);
    };
    lay_out(0, re[0], im[0]);
    __syncthreads();
    for (int kp = 0; kp < np; kp += 2) {
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        __syncthreads();  // F of panel kp + h
        if (on)
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const int tt = rowt[h][16 * w + acc_row(lane, i)];
            if (tt >= 0)
#pragma unroll
              for (int q = 0; q < 8; ++q) {
                prow[h][tt][16 * ((q + rot) & 7) + m] = make_double2(re[q][i], im[q][i]);
                re[q][i] = im[q][i] = 0.0;
              }
          }
        __syncthreads();  // the pivot rows
        double2 f[2];
#pragma unroll
        for (int s = 0; s < 2; ++s) f[s] = pan[h][16 * w + m][g + 4 * s];
        auto update = [&](int cb, d4& x, d4& y) {
#pragma unroll
          for (int s = 0; s < 2; ++s) {
            const double2 v = prow[h][g + 4 * s][16 * cb + m];
            x = mfma16(f[s].x, v.x, x);
            y = mfma16(f[s].x, v.y, y);
            x = mfma16(-f[s].y, v.y, x);
            y = mfma16(f[s].y, v.x, y);
          }
        };
        auto own = [&]() {  // the panel's own columns are F
          update(rot, re[0], im[0]);
          if ((m >> 3) == h)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              const double2 v = pan[h][16 * w + acc_row(lane, i)][m & 7];
              re[0][i] = v.x;
              im[0][i] = v.y;
            }
        };
        if (on) {
          if (h == 0) {
            own();
            lay_out(1, re[0], im[0]);
          } else if (rot + 1 < nb) {
            update(rot + 1, re[1], im[1]);
            lay_out(0, re[1], im[1]);
          }
        }
        __syncthreads();  // panel kp + h + 1
        if (on) {
          if (h == 1) own();
#pragma unroll
          for (int q = 1; q < 8; ++q) {
            const int cb = (q + rot) & 7;
            if (cb < nb && (h == 0 || q > 1 || cb == 0)) update(cb, re[q], im[q]);
          }
        }
      }
      const d4 x = re[0], y = im[0];
#pragma unroll
      for (int q = 0; q < 7; ++q) {
        re[q] = re[q + 1];
        im[q] = im[q + 1];
      }
      re[7] = x;
      im[7] = y;
      ++rot;
    }
    // row i of the table is row rowof[i] of the inverse; its column c is column perm[c] (rot == nb)
    double2* I2 = reinterpret_cast<double2*>(Ainv);
#pragma unroll
    for (int q = 0; q < 8; ++q)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int row = 16 * w + acc_row(lane, i), col = 16 * ((q + rot) & 7) + m;
        if (row < r && col < r) {
          const int tr = rowof[row], tc = perm[col];
          if (tr < r && tc < r) I2[(size_t)tr * r + tc] = make_double2(re[q][i], im[q][i]);
        }
      }
  }
  __syncthreads();
  norm1(reinterpret_cast<const double2*>(Ainv));
  __syncthreads();
  if (t < 128) npart[0][t] = (npart[0][t] + npart[1][t]) + (npart[2][t] + npart[3][t]);
  __syncthreads();
  if (t == 0) {
    double na = 0.0, ni = 0.0;
    for (int c = 0; c < r; ++c) {
      na = fmax(na, csum[c]);
      ni = fmax(ni, npart[0][c]);
    }
    cond[0] = na * ni;
    info[0] = s_bad;
  }
}

// ---- launchers -------------------------------------------------------------------
template <typename T>
void coord_layer(int dim, const int n[3], size_t row0, size_t nrows, const T* W, const T* b, int N, int act, T* out,
                 hipStream_t st) {
  // about 4096 workgroups of at least 16 rows each
  size_t rpb = (nrows + 4095) / 4096;
  if (rpb < 16) rpb = 16;
  const size_t nb = (nrows + rpb - 1) / rpb;
  if (nb == 0) return;
  const int ny = dim > 1 ? n[1] : 1, nz = dim > 2 ? n[2] : 1;  // absent axes have one node
  if (n[0] <= CL_TAB && ny <= CL_TAB && nz <= CL_TAB)
    hipLaunchKernelGGL((k_coord_layer<T, true>), dim3((unsigned)nb), dim3(256), 0, st, dim, n[0], ny, nz, row0, nrows,
                       rpb, W, b, N, act, out);
  else
    hipLaunchKernelGGL((k_coord_layer<T, false>), dim3((unsigned)nb), dim3(256), 0, st, dim, n[0], ny, nz, row0, nrows,
                       rpb, W, b, N, act, out);
}

template <typename T>
void gemm(int M, int N, int K, const T* A, size_t lda, const T* W, size_t ldw, const T* bias, int act, T* C,
          size_t ldc, hipStream_t st) {
  kprof_begin(KP_MFMA, st);
  const int nb = ((M + GB_M - 1) / GB_M) * ((N + GB_N - 1) / GB_N);
  hipLaunchKernelGGL((k_gemm<T>), dim3(nb), dim3(256), 0, st, M, N, K, A, lda, W, ldw, bias, act, C, ldc);
  kprof_end(KP_MFMA, 2.0 * M * N * K, st);
}

int small_ksplit(int K) {
  int ks = (K + 255) / 256;
  if (ks > 64) ks = 64;
  if (ks < 1) ks = 1;
  return ks;
}

template <typename T>
void dense_small(int B, int N, int K, const T* x, const T* W, const T* bias, int act, T* y, double* part,
                 hipStream_t st) {
  const int ks = small_ksplit(K);
  const int ncb = (N + SK_COLS - 1) / SK_COLS;
  hipLaunchKernelGGL((k_small_part<T>), dim3(ncb * ks), dim3(256), 0, st, B, N, K, ks, x, W, part);
  hipLaunchKernelGGL((k_small_final<T>), dim3((B * N + 255) / 256), dim3(256), 0, st, B, N, ks, part, bias, act, y);
}

void chol_drop(int p, const double* G, double tau2, int allow_drop, double* S, int* info, hipStream_t st) {
  hipLaunchKernelGGL(k_chol_drop, dim3(1), dim3(1024), 0, st, p, G, tau2, allow_drop, S, info);
}

void gj_inverse(int r, const double* A, double* work, double* Ainv, int* info, double* cond, hipStream_t st) {
  (void)work;
  hipLaunchKernelGGL(k_gj_inverse, dim3(1), dim3(576), 0, st, r, A, Ainv, info, cond);
}

template void coord_layer<double>(int, const int*, size_t, size_t, const double*, const double*, int, int, double*,
                                  hipStream_t);
template void gemm<double>(int, int, int, const double*, size_t, const double*, size_t, const double*, int, double*,
                           size_t, hipStream_t);
template void dense_small<double>(int, int, int, const double*, const double*, const double*, int, double*, double*,
                                  hipStream_t);
template void dense_small<float>(int, int, int, const float*, const float*, const float*, int, float*, double*,
                                 hipStream_t);

}  // namespace helm
