// DeepONet inference (App. B architecture; App. C trunk matrix).
//
// Trunk: the coordinate input layer is evaluated directly from node indices
// (no coordinate array), the hidden and output layers are fp64 MFMA GEMMs with
// fused bias + activation (both dtypes), row-chunked so the activations stay
// within a bounded buffer at any grid size.  The result T (n x p) is what the trunk-basis
// coarse space and the output synthesis consume.
//
// Full correction du = s N(r / s):  ||r|| (two-stage reduction) -> branch input
// (scaled residual, identity or multilinear resampling onto the branch grid, k
// appended) -> branch layers (split-K GEMV, batch 1 or 2) -> coefficients
// c = b_re + i b_im -> du_i = s sum_j T_ij c_j, zero on scatterer nodes.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <cstring>
#include <cmath>
#include <vector>

#include "common.h"
#include "dense_dev.h"
#include "internal.h"
#include "lib.h"

namespace helm {

static std::atomic<int> g_serial{1};

int don_p(const don_s* net) { return net->p; }
int don_serial(const don_s* net) { return net->serial; }
void don_touch(don_s* net) { net->serial = g_serial.fetch_add(1); }

static int map_act(int a) { return a == DON_TANH ? ACT_TANH : a == DON_RELU ? ACT_RELU : ACT_LEAKY; }

helm_status check_net_for_op(const don_s* net, const helm_op_s* op, int p_used) {
  if (!net) return fail(HELM_E_INVAL, "network is NULL");
  if (net->dt != op->dt) return fail(HELM_E_INVAL, "network dtype %d does not match the op's %d", net->dt, op->dt);
  if (net->tw[0] != op->dim)
    return fail(HELM_E_INVAL, "trunk input width %d does not match grid dimension %d", net->tw[0], op->dim);
  if (op->dim == 2 && net->bgrid[2] != 1) return fail(HELM_E_INVAL, "2D op needs branch_grid[2] = 1");
  if (p_used < 1 || p_used > net->p) return fail(HELM_E_INVAL, "p_used = %d outside [1, %d]", p_used, net->p);
  if ((size_t)p_used > op->nn) return fail(HELM_E_INVAL, "p_used = %d exceeds the node count", p_used);
  return HELM_OK;
}

// ---- kernels ----------------------------------------------------------------------
// s = sqrt(ss / n) and 1/s (0 when s = 0), from the reduced ||r||^2
__global__ void k_scale_of(const double* ss, double n, double* out) {
  if (threadIdx.x == 0 && blockIdx.x == 0) {
    const double s = sqrt(ss[0] / n);
    out[0] = s;
    out[1] = s > 0.0 ? 1.0 / s : 0.0;
  }
}

// branch input, identity sampling: x[0][i] = Re r_i / s, x[1][i] = Im r_i / s
// (SPLIT_INPUT) or x[0][i], x[0][n + i] (SPLIT_OUTPUT); optional k at x[0][2n]
template <typename T, typename S>
__global__ void k_branch_in_identity(size_t n, const cplx_t<S>* __restrict__ r, const double* __restrict__ sv,
                                     int split_input, int k_input, double k, T* __restrict__ x) {
  const double inv = sv[1];
  for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) {
    const double2 v = ldc(r, i);
    const size_t off = split_input ? n : n;
    x[i] = (T)(v.x * inv);
    x[off + i] = (T)(v.y * inv);
    if (!split_input && k_input && i == 0) x[2 * n] = (T)k;
  }
}

// r sampled at branch-grid node j by multilinear interpolation (zero ghosts)
struct SampleGrid {
  int dim, n[3], m[3];  // op grid, branch grid
};
template <typename S>
__device__ __forceinline__ double2 sample_node(const SampleGrid& g, const cplx_t<S>* __restrict__ r, size_t j) {
  const int jj[3] = {(int)(j % g.m[0]), (int)((j / g.m[0]) % g.m[1]), (int)(j / ((size_t)g.m[0] * g.m[1]))};
  int i0[3];
  double w[3];
  for (int a = 0; a < 3; ++a) {
    if (a < g.dim && g.m[a] != g.n[a]) {
      const double xt = (double)(jj[a] + 1) / (double)(g.m[a] + 1);
      const double t = __dmul_rn(xt, (double)(g.n[a] + 1)) - 1.0;
      i0[a] = (int)floor(t);
      w[a] = t - i0[a];
    } else {
      i0[a] = jj[a];
      w[a] = 0.0;
    }
  }
  double2 acc = czero();
  const int nc = 1 << g.dim;
  for (int cidx = 0; cidx < nc; ++cidx) {
    double wt = 1.0;
    int idx[3] = {0, 0, 0};
    bool inside = true;
    for (int a = 0; a < 3; ++a) {
      const int bit = a < g.dim ? (cidx >> a) & 1 : 0;
      idx[a] = i0[a] + bit;
      wt *= bit ? w[a] : 1.0 - w[a];
      if (a < g.dim && (idx[a] < 0 || idx[a] >= g.n[a])) inside = false;
    }
    if (!inside || wt == 0.0) continue;
    const size_t p = (size_t)idx[0] + (size_t)g.n[0] * ((size_t)idx[1] + (size_t)g.n[1] * idx[2]);
    const double2 v = ldc(r, p);
    acc.x += wt * v.x;
    acc.y += wt * v.y;
  }
  return acc;
}

// branch input by multilinear interpolation onto the branch grid (zero ghosts):
// x[0][j] = sample(Re r / s), x[0][m + j] = sample(Im r / s), x[0][2m] = k
template <typename T, typename S>
__global__ void k_branch_in_sample(SampleGrid g, const cplx_t<S>* __restrict__ r, const double* __restrict__ sv,
                                   int split_input, int k_input, double k, T* __restrict__ x) {
  const size_t m = (size_t)g.m[0] * g.m[1] * g.m[2];
  const double inv = sv[1];
  for (size_t j = blockIdx.x * (size_t)blockDim.x + threadIdx.x; j < m; j += (size_t)gridDim.x * blockDim.x) {
    const double2 acc = sample_node<S>(g, r, j);
    const size_t off = m;
    x[j] = (T)(acc.x * inv);
    x[off + j] = (T)(acc.y * inv);
    if (!split_input && k_input && j == 0) x[2 * m] = (T)k;
  }
}

// ---- branch network in two launches ------------------------------------------------
// k_branch_first: the input layer's product, split over k: workgroup (i, c)
// takes input entries [64 i, 64 i + 64) and columns [256 c, 256 c + 256), each
// thread one column and half of the entries, its 32 weights all in flight.
// They are issued first: the scale s = ||r|| / sqrt(n) (every workgroup sums the
// norm's partials itself, in one order) and the workgroup's entries of the
// branch input (sampled here, no array of them is formed) then cost no extra
// memory latency.  k_branch_tail: one workgroup sums those products in order,
// then runs the remaining layers (each thread a column and a quarter of k, BT_K
// weights in flight, the next layer's first ones issued before this layer's sums
// meet in LDS) and forms the coefficients c_j.  What bounds both is latency:
// the 9.4 MB of weights (fp32, 8193-256x5) would take 2 us.  A launch per layer
// and half layer, each thread walking its k with one load in flight and the
// 256-wide layers on four workgroups, took 27.8 us per product and 16 launches
// per correction (48^3 complex64: 179 -> 59 us, 16 of them
// the synthesis).
constexpr int BF_K = 64;        // input entries per workgroup
constexpr int BT_K = 16;       // weights in flight per thread of the tail
constexpr int BT_MAXL = 16;     // layers
constexpr int BT_MAXW = 1024;   // outputs of a layer
// weights of the layers after the input layer, their columns in whole blocks of
// 256, that one CU reads as fast as a launch or two per layer: at most so much
// for two layers, more for each further one, and in all
constexpr size_t BT_TWO = (size_t)4 << 20, BT_LAYER = (size_t)1 << 20, BT_ALL = (size_t)6 << 20;

template <typename T>
__global__ __launch_bounds__(512) void k_branch_first(SampleGrid g, const cplx_t<T>* __restrict__ r, size_t n,
                                                      const double* __restrict__ npart, int nb, int B, int K, int N,
                                                      int split_input, double kval, const T* __restrict__ W,
                                                      double* __restrict__ part, double* __restrict__ sc) {
  __shared__ double xs[2][BF_K], cmb[2][256], sh[16], s_inv;
  const int t = threadIdx.x, half = t >> 8;
  const int col = blockIdx.y * 256 + (t & 255), k0 = blockIdx.x * BF_K + half * (BF_K / 2);
  T w[BF_K / 2];
#pragma unroll
  for (int u = 0; u < BF_K / 2; ++u) w[u] = (col < N && k0 + u < K) ? W[(size_t)(k0 + u) * N + col] : T(0);
  double acc = 0.0;
  if (t < 256)
    for (int b0 = 0; b0 < nb; b0 += 4 * 256) {
      double v[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int b = b0 + t + 256 * q;
        v[q] = b < nb ? npart[b] : 0.0;
      }
#pragma unroll
      for (int q = 0; q < 4; ++q) acc += v[q];
    }
  const size_t m = (size_t)g.m[0] * g.m[1] * g.m[2];
  // entry k of input row b: split input Re (b = 0) and Im (b = 1) of node k;
  // split output Re, then Im of the nodes, then the wave number
  double xv = 0.0;
  const int xb = t / BF_K, xk = blockIdx.x * BF_K + (t & (BF_K - 1));
  bool scaled = true;
  if (xb < B && xk < K) {
    if (split_input) {
      const double2 v = sample_node<T>(g, r, (size_t)xk);
      xv = xb ? v.y : v.x;
    } else if ((size_t)xk < 2 * m) {
      const bool im = (size_t)xk >= m;
      const double2 v = sample_node<T>(g, r, im ? xk - m : (size_t)xk);
      xv = im ? v.y : v.x;
    } else {
      xv = kval;
      scaled = false;
    }
  }
  acc = block_sum(acc, sh);
  if (t == 0) {
    const double s = sqrt(acc / (double)n), inv = s > 0.0 ? 1.0 / s : 0.0;
    s_inv = inv;
    if (blockIdx.x == 0 && blockIdx.y == 0) {
      sc[0] = s;
      sc[1] = inv;
    }
  }
  __syncthreads();
  if (xb < B) xs[xb][t & (BF_K - 1)] = (double)(T)(scaled ? xv * s_inv : xv);
  __syncthreads();
  for (int b = 0; b < B; ++b) {
    double a = 0.0;
#pragma unroll
    for (int u = 0; u < BF_K / 2; ++u) a += xs[b][half * (BF_K / 2) + u] * (double)w[u];
    if (half) cmb[b][t & 255] = a;
    __syncthreads();
    if (!half && col < N) part[((size_t)blockIdx.x * B + b) * N + col] = a + cmb[b][t];
  }
}

__device__ __forceinline__ double ld_weight(__amdgpu_buffer_rsrc_t r, int vo, int so, const double*) {
  return __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(r, vo, so, 0));
}
__device__ __forceinline__ float ld_weight(__amdgpu_buffer_rsrc_t r, int vo, int so, const float*) {
  return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, vo, so, 0));
}

struct BranchTail {
  int L, B, p, act, ns;           // layers; input rows; coefficients; activation; partials of the first product
  int w[BT_MAXL + 1];             // widths
  const void *W[BT_MAXL], *b[BT_MAXL];
};

template <typename T>
__global__ __launch_bounds__(1024) void k_branch_tail(BranchTail a, const double* __restrict__ part,
                                                      double* __restrict__ coef) {
  __shared__ double x[2][2][BT_MAXW], red[4][2][256];
  const int t = threadIdx.x, c = t & 255;
  const int g = __builtin_amdgcn_readfirstlane(t >> 8);  // quarter of k; uniform in a wavefront
  // the BT_K weights of the whole k chunk ch (entries BT_K ch and on) in
  // column col (a column past the end reads 0, out of the buffer's range)
  T wp[BT_K];
  auto fetch = [&](int l, int ch, int col) {
    const int K = a.w[l], N = a.w[l + 1], sz = (int)sizeof(T);
    const __amdgpu_buffer_rsrc_t wr =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(a.W[l]), 0, K * N * sz, 0x00020000);
    const int vo = col < N ? (BT_K * ch * N + col) * sz : 0x7f000000;
#pragma unroll
    for (int u = 0; u < BT_K; ++u) wp[u] = ld_weight(wr, vo, u * N * sz, (const T*)nullptr);
  };
  // sums of a layer's output (row b, column col) meet in LDS: bias, activation
  // (fp64 arithmetic, rounded once to the stored type)
  auto finish = [&](int l, int dst, int col) {
    const int N = a.w[l + 1];
    __syncthreads();
    if (g < a.B && col < N) {
      double v = (red[0][g][c] + red[1][g][c]) + (red[2][g][c] + red[3][g][c]);
      v += (double)((const T*)a.b[l])[col];
      x[dst][g][col] = (double)(T)activate<double>(v, l + 1 < a.L ? a.act : ACT_NONE);
    }
    __syncthreads();
  };
  if (a.L > 1 && BT_K * (g + 1) <= a.w[1]) fetch(1, g, c);
  {
    const int N = a.w[1];
    for (int n0 = 0; n0 < N; n0 += 256) {
      const int col = n0 + c;
      for (int b = 0; b < a.B; ++b) {
        double acc = 0.0;
        const double* q = part + (size_t)b * N + (col < N ? col : 0);
        const size_t step = (size_t)a.B * N;
#pragma unroll 1
        for (int s0 = g; s0 < a.ns; s0 += 4 * 8) {
          double v[8];
#pragma unroll
          for (int u = 0; u < 8; ++u) v[u] = s0 + 4 * u < a.ns ? q[(size_t)(s0 + 4 * u) * step] : 0.0;
#pragma unroll
          for (int u = 0; u < 8; ++u) acc += v[u];
        }
        red[g][b][c] = acc;
      }
      finish(0, 0, col);
    }
  }
  int cur = 0;
#pragma unroll 1
  for (int l = 1; l < a.L; ++l) {
    const int K = a.w[l], N = a.w[l + 1], nch = K / BT_K;
#pragma unroll 1
    for (int n0 = 0; n0 < N; n0 += 256) {
      const int col = n0 + c;
      double acc0 = 0.0, acc1 = 0.0;
#pragma unroll 1
      for (int ch = g; ch < nch; ch += 4) {
        if (n0 > 0 || ch > g) fetch(l, ch, col);
        const double* x0 = x[cur][0] + BT_K * ch;
        const double* x1 = x[cur][1] + BT_K * ch;
#pragma unroll
        for (int u = 0; u < BT_K; ++u) acc0 += x0[u] * (double)wp[u];
        if (a.B > 1)
#pragma unroll
          for (int u = 0; u < BT_K; ++u) acc1 += x1[u] * (double)wp[u];
      }
      if (K % BT_K && g == (nch & 3) && col < N) {  // the entries past the last whole chunk
        const T* W = (const T*)a.W[l];
        for (int k = BT_K * nch; k < K; ++k) {
          const double wk = (double)W[(size_t)k * N + col];
          acc0 += x[cur][0][k] * wk;
          if (a.B > 1) acc1 += x[cur][1][k] * wk;
        }
      }
      if (n0 + 256 >= N && l + 1 < a.L && BT_K * (g + 1) <= N) fetch(l + 1, g, c);
      red[g][0][c] = acc0;
      red[g][1][c] = acc1;
      finish(l, 1 - cur, col);
    }
    cur = 1 - cur;
  }
  for (int j = t; j < a.p; j += blockDim.x) {
    coef[2 * j] = x[cur][0][j];
    coef[2 * j + 1] = a.B > 1 ? x[cur][1][j] : x[cur][0][a.p + j];
  }
}

// coefficients c_j = b_re_j + i b_im_j (fp64)
template <typename T>
__global__ void k_coef(int p, int split_input, const T* __restrict__ b, double* __restrict__ c) {
  const int j = blockIdx.x * blockDim.x + threadIdx.x;
  if (j >= p) return;
  c[2 * j] = (double)b[j];
  c[2 * j + 1] = split_input ? (double)b[p + j] : (double)b[p + j];
}

// fp64 trunk rows rounded once to the stored fp32 trunk matrix (C64)
__global__ void k_narrow(size_t cnt, const double* __restrict__ src, float* __restrict__ dst) {
  for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < cnt; i += (size_t)gridDim.x * blockDim.x)
    dst[i] = (float)src[i];
}

// ---- drivers -------------------------------------------------------------------------
// The trunk matrix is evaluated in fp64 arithmetic for both dtypes (a C64
// network's fp32 weights widened exactly): the basis of App. C is set-up
// algebra, and an fp32 evaluation's few-ulp errors per layer (about 5e-7 of T
// at the 3D trunk) reach the meta-solver's iterate amplified.  A C64 trunk
// matrix is rounded to fp32 once, as it is stored.
template <typename T>
static helm_status trunk_eval(don_s* net, helm_op_s* op, T* out, hipStream_t st) {
  constexpr bool wide = sizeof(T) == sizeof(double);
  const size_t n = op->nn;
  const int L = (int)net->tw.size() - 1;
  if (trunk_fused_fits(L, net->tw.data())) {
    const std::vector<void*>& Wf = wide ? net->tW : net->tW64;
    const std::vector<void*>& Bf = wide ? net->tB : net->tB64;
    trunk_fused<T>(op->dim, op->n, L, net->tw.data(), (const double* const*)Wf.data(), (const double* const*)Bf.data(),
                   map_act(net->act), out, st);
    return launch_check("trunk");
  }
  int maxw = 1;
  for (int w : net->tw) maxw = w > maxw ? w : maxw;
  const size_t chunk = n < (size_t)262144 ? n : (size_t)262144;
  helm_status s;
  if ((s = net->tact0.ensure(chunk * maxw * sizeof(double))) ||
      (s = net->tact1.ensure(chunk * maxw * sizeof(double))))
    return s;
  const std::vector<void*>& W = wide ? net->tW : net->tW64;
  const std::vector<void*>& B = wide ? net->tB : net->tB64;
  const int act = map_act(net->act);
  const int p = net->p;
  for (size_t r0 = 0; r0 < n; r0 += chunk) {
    const size_t rc = n - r0 < chunk ? n - r0 : chunk;
    double* h[2] = {(double*)net->tact0.ptr, (double*)net->tact1.ptr};
    // the last layer writes the stored matrix directly (C128) or a scratch chunk
    auto last_out = [&](int slot) { return wide ? (double*)(void*)(out + r0 * p) : h[slot]; };
    double* o = L == 1 ? last_out(1) : h[0];
    coord_layer<double>(op->dim, op->n, r0, rc, (const double*)W[0], (const double*)B[0], net->tw[1],
                        L == 1 ? ACT_NONE : act, o, st);
    int cur = 0;
    for (int l = 1; l < L; ++l) {
      const bool last = l == L - 1;
      o = last ? last_out(1 - cur) : h[1 - cur];
      gemm<double>((int)rc, net->tw[l + 1], net->tw[l], h[cur], net->tw[l], (const double*)W[l], net->tw[l + 1],
                   (const double*)B[l], last ? ACT_NONE : act, o, net->tw[l + 1], st);
      cur = 1 - cur;
    }
    if (!wide) {
      const size_t cnt = rc * (size_t)p;
      hipLaunchKernelGGL(k_narrow, dim3((unsigned)std::min<size_t>((cnt + 255) / 256, 16384)), dim3(256), 0, st, cnt,
                         o, (float*)(void*)(out + r0 * p));
    }
  }
  return launch_check("trunk");
}

helm_status don_trunk(don_s* net, helm_op_s* op, void* out, hipStream_t st) {
  return net->dt == HELM_C128 ? trunk_eval<double>(net, op, (double*)out, st)
                              : trunk_eval<float>(net, op, (float*)out, st);
}

static bool same_grid(const don_s* net, const helm_op_s* op) {
  for (int a = 0; a < 3; ++a)
    if (net->bgrid[a] != op->n[a]) return false;
  return true;
}

static SampleGrid sample_grid(const don_s* net, const helm_op_s* op) {
  SampleGrid g;
  g.dim = op->dim;
  for (int a = 0; a < 3; ++a) {
    g.n[a] = op->n[a];
    g.m[a] = net->bgrid[a];
  }
  return g;
}

// k_branch_first + k_branch_tail: layer widths within the tail's LDS, its
// weights few enough that one CU (20 us per MB) is done before the launches of
// layer by layer (about 20 us per layer).  Whole corrections, layer by layer and
// in two launches, us (12960 nodes, inputs 8193; MB with columns in whole blocks):
// fp32 768-768-256 3.0 MB 116 and 93, 1024-768-256 3.8 MB 120 and 112, 900-900-256
// 4.4 MB 116 and 124, 960-896-256 4.6 MB 114 and 128, 600-600-600-256 4.1 MB 133
// and 112, five of 512 4.5 MB 157 and 117; fp64 768-512-256 4.0 MB 107 and 93,
// 640-640-256 5.0 MB 99 and 107, 1024-384-256 4.8 MB 101 and 111, four of 384 5.3
// MB 136 and 106.
static bool branch_fits(const don_s* net) {
  const int L = (int)net->bw.size() - 1;
  size_t bytes = 0;
  if (L > BT_MAXL) return false;
  for (int l = 0; l < L; ++l) {
    if (net->bw[l + 1] > BT_MAXW) return false;
    if (l > 0) bytes += (size_t)net->bw[l] * ((net->bw[l + 1] + 255) / 256 * 256) * (net->dt == HELM_C128 ? 8 : 4);
  }
  const size_t more = L > 3 ? L - 3 : 0;  // layers after the input layer and two
  return bytes <= std::min(BT_TWO + more * BT_LAYER, BT_ALL);
}

template <typename T>
static helm_status full_eval(don_s* net, helm_op_s* op, const void* r, double k, void* du, hipStream_t st,
                             bool input_only = false) {
  const size_t n = op->nn;
  Coarse& c = op->coarse;
  helm_status s;
  if (!input_only && c.T_serial != net->serial) {
    if ((s = c.T.ensure(n * (size_t)net->p * sizeof(T)))) return s;
    if ((s = trunk_eval<T>(net, op, (T*)c.T.ptr, st))) return s;
    c.T_serial = net->serial;
  }
  // s = ||r|| / sqrt(n)
  double* part;
  const int nb = red_nblocks(n);
  if ((s = op_part(op, (size_t)nb, &part))) return s;
  nrm2_part<T>(n, r, part, st);
  double* sv = op->red + 3072;  // [ss, s, 1/s]
  if (!input_only && branch_fits(net)) {
    const int B = net->head == DON_SPLIT_INPUT ? 2 : 1, K = net->bw[0], N = net->bw[1];
    const int ns = (K + BF_K - 1) / BF_K;
    if ((s = net->part.ensure((size_t)ns * B * N * sizeof(double))) ||
        (s = net->coef.ensure(2 * (size_t)net->p * sizeof(double))))
      return s;
    hipLaunchKernelGGL((k_branch_first<T>), dim3(ns, (N + 255) / 256), dim3(512), 0, st, sample_grid(net, op),
                       (const cplx_t<T>*)r, n, (const double*)part, nb, B, K, N, B == 2, k, (const T*)net->bW[0],
                       (double*)net->part.ptr, sv + 1);
    BranchTail a{};
    a.L = (int)net->bw.size() - 1;
    a.B = B;
    a.p = net->p;
    a.act = map_act(net->act);
    a.ns = ns;
    for (int l = 0; l <= a.L; ++l) a.w[l] = net->bw[l];
    for (int l = 0; l < a.L; ++l) {
      a.W[l] = net->bW[l];
      a.b[l] = net->bB[l];
    }
    hipLaunchKernelGGL((k_branch_tail<T>), dim3(1), dim3(1024), 0, st, a, (const double*)net->part.ptr,
                       (double*)net->coef.ptr);
    skinny_apply<T, T>(n, net->p, (const T*)c.T.ptr, (const double*)net->coef.ptr, du, op->mask, sv + 1, 1, st);
    return launch_check("deeponet full");
  }
  reduce_cols(part, nb, 1, sv, st);
  hipLaunchKernelGGL(k_scale_of, dim3(1), dim3(64), 0, st, sv, (double)n, sv + 1);
  const double* sc = sv + 1;
  // branch input
  const int B = net->head == DON_SPLIT_INPUT ? 2 : 1;
  const int K0 = net->bw[0];
  int maxw = 1;
  for (int w : net->bw) maxw = w > maxw ? w : maxw;
  if ((s = net->act0.ensure((size_t)B * maxw * sizeof(T) + 64)) || (s = net->act1.ensure((size_t)B * maxw * sizeof(T) + 64)))
    return s;
  T* x0 = (T*)net->act0.ptr;
  T* x1 = (T*)net->act1.ptr;
  const int split_in = net->head == DON_SPLIT_INPUT;
  if (same_grid(net, op)) {
    int g = (int)((n + 255) / 256);
    if (g > 8192) g = 8192;
    hipLaunchKernelGGL((k_branch_in_identity<T, T>), dim3(g), dim3(256), 0, st, n, (const cplx_t<T>*)r, sc, split_in,
                       net->k_input, k, x0);
  } else {
    const size_t m = (size_t)net->bgrid[0] * net->bgrid[1] * net->bgrid[2];
    int g = (int)((m + 255) / 256);
    if (g > 8192) g = 8192;
    hipLaunchKernelGGL((k_branch_in_sample<T, T>), dim3(g), dim3(256), 0, st, sample_grid(net, op),
                       (const cplx_t<T>*)r, sc, split_in, net->k_input, k, x0);
  }
  if (input_only) {
    hipError_t e = hipMemcpyAsync(du, x0, (size_t)B * K0 * sizeof(T), hipMemcpyDeviceToDevice, st);
    if (e != hipSuccess) return hip_fail(e, "deeponet branch input");
    return launch_check("deeponet branch input");
  }
  // branch layers
  const int L = (int)net->bw.size() - 1;
  size_t pneed = 0;
  for (int l = 0; l < L; ++l) {
    const size_t q = (size_t)small_ksplit(net->bw[l]) * B * net->bw[l + 1];
    pneed = q > pneed ? q : pneed;
  }
  if ((s = net->part.ensure(pneed * sizeof(double)))) return s;
  T* h[2] = {x0, x1};
  int cur = 0;
  const int act = map_act(net->act);
  for (int l = 0; l < L; ++l) {
    dense_small<T>(B, net->bw[l + 1], net->bw[l], h[cur], (const T*)net->bW[l], (const T*)net->bB[l],
                   l == L - 1 ? ACT_NONE : act, h[1 - cur], (double*)net->part.ptr, st);
    cur = 1 - cur;
  }
  // coefficients and synthesis
  if ((s = net->coef.ensure(2 * (size_t)net->p * sizeof(double)))) return s;
  hipLaunchKernelGGL((k_coef<T>), dim3((net->p + 63) / 64), dim3(64), 0, st, net->p, split_in, h[cur],
                     (double*)net->coef.ptr);
  skinny_apply<T, T>(n, net->p, (const T*)c.T.ptr, (const double*)net->coef.ptr, du, op->mask, sc, 1, st);
  return launch_check("deeponet full");
}

helm_status don_full(don_s* net, helm_op_s* op, const void* r, double k, void* du, hipStream_t st) {
  return net->dt == HELM_C128 ? full_eval<double>(net, op, r, k, du, st) : full_eval<float>(net, op, r, k, du, st);
}

static helm_status don_branch_input(don_s* net, helm_op_s* op, const void* r, double k, void* out, hipStream_t st) {
  return net->dt == HELM_C128 ? full_eval<double>(net, op, r, k, out, st, true)
                              : full_eval<float>(net, op, r, k, out, st, true);
}

}  // namespace helm

using namespace helm;

extern "C" {

helm_status deeponet_load(helm_dtype dt, const don_desc* d, const double* const* Wb, don_net* out) {
  if (!out) return fail(HELM_E_INVAL, "deeponet_load: out is NULL");
  *out = nullptr;
  if (!d || !Wb || !d->branch_w || !d->trunk_w) return fail(HELM_E_INVAL, "deeponet_load: NULL argument");
  if (dt != HELM_C64 && dt != HELM_C128) return fail(HELM_E_INVAL, "deeponet_load: unknown dtype");
  if (d->n_branch < 2 || d->n_trunk < 2) return fail(HELM_E_INVAL, "deeponet_load: each network needs >= 1 layer");
  if (d->act < DON_TANH || d->act > DON_LEAKY) return fail(HELM_E_INVAL, "deeponet_load: unknown activation");
  if (d->head != DON_SPLIT_OUTPUT && d->head != DON_SPLIT_INPUT) return fail(HELM_E_INVAL, "deeponet_load: unknown head");
  if (d->p < 1 || d->p > 128) return fail(HELM_E_INVAL, "deeponet_load: p = %d outside [1, 128]", d->p);
  for (int i = 0; i < d->n_branch; ++i)
    if (d->branch_w[i] < 1) return fail(HELM_E_INVAL, "deeponet_load: branch width %d < 1", i);
  for (int i = 0; i < d->n_trunk; ++i)
    if (d->trunk_w[i] < 1) return fail(HELM_E_INVAL, "deeponet_load: trunk width %d < 1", i);
  if (d->trunk_w[0] != 2 && d->trunk_w[0] != 3) return fail(HELM_E_INVAL, "deeponet_load: trunk input must be 2 or 3");
  if (d->trunk_w[d->n_trunk - 1] != d->p) return fail(HELM_E_INVAL, "deeponet_load: trunk output must equal p");
  size_t m = 1;
  for (int a = 0; a < 3; ++a) {
    if (d->branch_grid[a] < 1) return fail(HELM_E_INVAL, "deeponet_load: branch_grid[%d] < 1", a);
    m *= (size_t)d->branch_grid[a];
  }
  if (d->trunk_w[0] == 2 && d->branch_grid[2] != 1) return fail(HELM_E_INVAL, "deeponet_load: 2D needs branch_grid[2] = 1");
  if (d->head == DON_SPLIT_OUTPUT) {
    if ((size_t)d->branch_w[0] != 2 * m + (d->k_input ? 1 : 0))
      return fail(HELM_E_INVAL, "deeponet_load: branch input width must be 2*prod(branch_grid)%s", d->k_input ? "+1" : "");
    if (d->branch_w[d->n_branch - 1] != 2 * d->p) return fail(HELM_E_INVAL, "deeponet_load: branch output must be 2p");
  } else {
    if ((size_t)d->branch_w[0] != m || d->k_input)
      return fail(HELM_E_INVAL, "deeponet_load: SPLIT_INPUT needs input width prod(branch_grid) and no k input");
    if (d->branch_w[d->n_branch - 1] != d->p) return fail(HELM_E_INVAL, "deeponet_load: branch output must be p");
  }
  const int nl = (d->n_branch - 1) + (d->n_trunk - 1);
  for (int i = 0; i < 2 * nl; ++i)
    if (!Wb[i]) return fail(HELM_E_INVAL, "deeponet_load: weight pointer %d is NULL", i);
  don_s* net = new don_s();
  net->dt = dt;
  net->act = d->act;
  net->head = d->head;
  net->p = d->p;
  net->k_input = d->k_input ? 1 : 0;
  for (int a = 0; a < 3; ++a) net->bgrid[a] = d->branch_grid[a];
  net->bw.assign(d->branch_w, d->branch_w + d->n_branch);
  net->tw.assign(d->trunk_w, d->trunk_w + d->n_trunk);
  net->serial = g_serial.fetch_add(1);
  const size_t rs = dt == HELM_C128 ? sizeof(double) : sizeof(float);
  auto upload = [&](const double* src, size_t cnt, void** dst) -> helm_status {
    helm_status s = dalloc(dst, cnt * rs);
    if (s) return s;
    std::vector<char> tmp(cnt * rs);
    if (dt == HELM_C128) {
      std::memcpy(tmp.data(), src, cnt * rs);
    } else {
      float* f = (float*)tmp.data();
      for (size_t i = 0; i < cnt; ++i) f[i] = (float)src[i];
    }
    hipError_t e = hipMemcpy(*dst, tmp.data(), cnt * rs, hipMemcpyHostToDevice);
    if (e != hipSuccess) return hip_fail(e, "deeponet_load: upload");
    return HELM_OK;
  };
  // fp64 copy of the fp32-rounded values (the trunk of a C64 network)
  auto upload_widened = [&](const double* src, size_t cnt, void** dst) -> helm_status {
    helm_status s = dalloc(dst, cnt * sizeof(double));
    if (s) return s;
    std::vector<double> tmp(cnt);
    for (size_t i = 0; i < cnt; ++i) tmp[i] = (double)(float)src[i];
    hipError_t e = hipMemcpy(*dst, tmp.data(), cnt * sizeof(double), hipMemcpyHostToDevice);
    if (e != hipSuccess) return hip_fail(e, "deeponet_load: upload");
    return HELM_OK;
  };
  int wi = 0;
  helm_status s = HELM_OK;
  for (int l = 0; l + 1 < d->n_branch && !s; ++l) {
    void *W = nullptr, *b = nullptr;
    s = upload(Wb[wi++], (size_t)d->branch_w[l] * d->branch_w[l + 1], &W);
    if (!s) s = upload(Wb[wi++], (size_t)d->branch_w[l + 1], &b);
    net->bW.push_back(W);
    net->bB.push_back(b);
  }
  for (int l = 0; l + 1 < d->n_trunk && !s; ++l) {
    void *W = nullptr, *b = nullptr;
    const double* srcW = Wb[wi++];
    const double* srcb = Wb[wi++];
    const size_t cW = (size_t)d->trunk_w[l] * d->trunk_w[l + 1], cb = (size_t)d->trunk_w[l + 1];
    s = upload(srcW, cW, &W);
    if (!s) s = upload(srcb, cb, &b);
    net->tW.push_back(W);
    net->tB.push_back(b);
    if (!s && dt == HELM_C64) {
      void *W64 = nullptr, *b64 = nullptr;
      s = upload_widened(srcW, cW, &W64);
      if (!s) s = upload_widened(srcb, cb, &b64);
      net->tW64.push_back(W64);
      net->tB64.push_back(b64);
    }
  }
  if (s) {
    deeponet_free(net);
    return s;
  }
  *out = net;
  return HELM_OK;
}

void deeponet_free(don_net net) {
  if (!net) return;
  for (void* p : net->bW) dfree(p);
  for (void* p : net->bB) dfree(p);
  for (void* p : net->tW) dfree(p);
  for (void* p : net->tB) dfree(p);
  for (void* p : net->tW64) dfree(p);
  for (void* p : net->tB64) dfree(p);
  net->act0.release();
  net->act1.release();
  net->tact0.release();
  net->tact1.release();
  net->part.release();
  net->coef.release();
  delete net;
}

helm_status deeponet_infer(don_net net, helm_op op, int mode, const void* r, double k, void* out, void* stream) {
  if (!net || !op || !out) return fail(HELM_E_INVAL, "deeponet_infer: NULL argument");
  if (mode != DON_TRUNK && mode != DON_FULL && mode != DON_BRANCH_INPUT)
    return fail(HELM_E_INVAL, "deeponet_infer: unknown mode %d", mode);
  helm_status s = check_net_for_op(net, op, 1);
  if (s) return s;
  hipStream_t st = (hipStream_t)stream;
  if (mode == DON_TRUNK) return don_trunk(net, op, out, st);
  if (!r) return fail(HELM_E_INVAL, "deeponet_infer: r is NULL");
  if (r == out) return fail(HELM_E_INVAL, "deeponet_infer: r and out alias");
  if (mode == DON_BRANCH_INPUT) return don_branch_input(net, op, r, k, out, st);
  return don_full(net, op, r, k, out, st);
}

}  // extern "C"
