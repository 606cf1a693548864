// Trunk evaluation in one launch (App. B architecture, App. C trunk matrix): a
// workgroup carries a block of grid nodes through every layer, the
// activations staying in LDS, so only T leaves the chip.
//
// What bounds it: the fp64 matrix instructions (the hidden layers are
// 2 w^2 flop per node and layer; at w = 256 a node's 2 KiB of activations would
// otherwise be written and read once per layer) and, since they share the
// fp64 units, the activation's vector arithmetic.  Layer by layer, with a
// 128 x 128 tile staged through LDS in 16-deep chunks, the products ran at 41
// of the 78.6 TFLOP/s peak: two barriers per chunk, and every activation value
// stored to and loaded from memory.  Measured (3-256x4-128 trunk): 10.13 ->
// 7.05 ms at 96^3 (58 TFLOP/s; the library's fp64 product of two 8192 x 8192
// matrices reaches 71), 287 -> 136 us at 24 x 20 x 27, 274 -> 41 us at
// 15 x 17 x 13, where most CUs had no tile; 3-32-32-16 at 96^3 731 -> 384 us.
// Splitting the products into exact int8 digit products is faster at 256 wide
// (5.7 ms), but its digits are relative to a node's largest activation and a
// column's largest weight: a column whose weights meet only small
// activations loses them, which neither shows alone.
#include "common.h"
#include "dense.h"
#include "dense_dev.h"
#include "prof.h"

namespace helm {

struct TrunkArgs {
  int L, dim, n[3], act, lda;   // layers; grid; hidden activation; LDS row stride
  int w[TRUNK_MAXL + 1];        // widths: w[0] = dim, ..., w[L] = p
  const double* W[TRUNK_MAXL];  // fan_in x fan_out, row-major
  const double* b[TRUNK_MAXL];
  size_t nn;
};

template <int RT, int CT>
__device__ __forceinline__ void trunk_store_act(double* __restrict__ h, int lda, const double* __restrict__ b, int wave,
                                                int lane, int act, const d4 (&acc)[RT][CT]) {
#pragma unroll
  for (int j = 0; j < CT; ++j) {
    const int col = 16 * (wave + TRUNK_WAVES * j) + (lane & 15);
    const double bc = b[col];
#pragma unroll
    for (int i = 0; i < RT; ++i)
#pragma unroll
      for (int q = 0; q < 4; ++q)
        h[(i * 16 + acc_row(lane, q)) * lda + col] = activate<double>(acc[i][j][q] + bc, act);
  }
}

template <int RT, int CT, typename T>
__device__ __forceinline__ void trunk_store_out(T* __restrict__ out, int N, size_t row0, size_t nn,
                                                const double* __restrict__ b, int wave, int lane,
                                                const d4 (&acc)[RT][CT]) {
#pragma unroll
  for (int j = 0; j < CT; ++j) {
    const int col = 16 * (wave + TRUNK_WAVES * j) + (lane & 15);
    const double bc = b[col];
#pragma unroll
    for (int i = 0; i < RT; ++i)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const size_t row = row0 + i * 16 + acc_row(lane, q);
        if (row < nn) out[row * N + col] = (T)(acc[i][j][q] + bc);
      }
  }
}

template <int RT, int CT, typename T>
__device__ __forceinline__ void trunk_step(const TrunkArgs& a, int l, double* h, size_t row0, int wave, int lane,
                                           T* __restrict__ out) {
  const int N = a.w[l + 1];
  d4 acc[RT][CT];
  trunk_layer<RT, CT>(h, a.lda, a.W[l], a.w[l], N, wave, lane, acc, a.w[l]);
  if (l + 1 == a.L) {
    trunk_store_out<RT, CT, T>(out, N, row0, a.nn, a.b[l], wave, lane, acc);
  } else {
    __syncthreads();  // every wavefront has read this layer's input
    trunk_store_act<RT, CT>(h, a.lda, a.b[l], wave, lane, a.act, acc);
  }
}

template <int RT, typename T>
__global__ __launch_bounds__(64 * TRUNK_WAVES, RT > 2 ? 2 : 4) void k_trunk(TrunkArgs a, T* __restrict__ out) {
  constexpr int ROWS = 16 * RT;
  extern __shared__ __attribute__((aligned(16))) double h[];  // ROWS x lda activations
  __shared__ double xc[ROWS][3];
  const int t = trunk_thread(), lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const size_t row0 = (size_t)blockIdx.x * ROWS;
  if (t < ROWS) {
    const size_t p = row0 + t < a.nn ? row0 + t : a.nn - 1;  // rows past the end repeat the last node
    const int nx = a.n[0], ny = a.n[1];
    xc[t][0] = (double)((int)(p % nx) + 1) / (double)(nx + 1);
    xc[t][1] = (double)((int)((p / nx) % ny) + 1) / (double)(ny + 1);
    xc[t][2] = (double)((int)(p / ((size_t)nx * ny)) + 1) / (double)(a.n[2] + 1);
  }
  __syncthreads();
  // input layer on the node coordinates
  const int N1 = a.w[1];
  for (int e = t; e < ROWS * N1; e += 64 * TRUNK_WAVES) {
    const int r = e / N1, c = e % N1;
    double v = xc[r][0] * a.W[0][c];
    v += xc[r][1] * a.W[0][N1 + c];
    if (a.dim > 2) v += xc[r][2] * a.W[0][2 * N1 + c];
    h[r * a.lda + c] = activate<double>(v + a.b[0][c], a.act);
  }
  for (int l = 1; l < a.L; ++l) {
    __syncthreads();
    const int nt = a.w[l + 1] / 16;
    if (wave + TRUNK_WAVES < nt) trunk_step<RT, 2, T>(a, l, h, row0, wave, lane, out);
    else if (wave < nt) trunk_step<RT, 1, T>(a, l, h, row0, wave, lane, out);
    else if (l + 1 < a.L) __syncthreads();  // a wavefront without columns keeps the barrier count
  }
}

bool trunk_fused_fits(int L, const int* w) {
  // hidden widths in whole 32-deep k steps, output columns in whole tiles, at
  // most two column tiles per wavefront; other widths go layer by layer
  if (L < 2 || L > TRUNK_MAXL || (w[0] != 2 && w[0] != 3)) return false;
  for (int l = 1; l < L; ++l)
    if (w[l] % 32 || w[l] > 256) return false;
  return w[L] % 16 == 0 && w[L] <= 256;
}

template <int RT, typename T>
static void trunk_launch(const TrunkArgs& a, T* out, hipStream_t st) {
  const size_t rows = 16 * RT, lds = rows * a.lda * sizeof(double);
  // per launch, not once per process: the limit is kept per device
  (void)hipFuncSetAttribute((const void*)k_trunk<RT, T>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  hipLaunchKernelGGL((k_trunk<RT, T>), dim3((unsigned)((a.nn + rows - 1) / rows)), trunk_block(), lds, st, a,
                     out);
}

template <typename T>
void trunk_fused(int dim, const int n[3], int L, const int* w, const double* const* W, const double* const* b, int act,
                 T* out, hipStream_t st) {
  TrunkArgs a{};
  a.L = L;
  a.dim = dim;
  a.act = act;
  a.nn = 1;
  for (int d = 0; d < 3; ++d) {
    a.n[d] = d < dim ? n[d] : 1;
    a.nn *= (size_t)a.n[d];
  }
  int maxw = 32;
  double flops = 0.0;
  for (int l = 0; l <= L; ++l) a.w[l] = w[l];
  for (int l = 0; l < L; ++l) {
    a.W[l] = W[l];
    a.b[l] = b[l];
    if (l > 0) {
      maxw = w[l] > maxw ? w[l] : maxw;
      flops += 2.0 * (double)a.nn * w[l] * w[l + 1];
    }
  }
  a.lda = maxw + 2;  // row stride odd in 16-byte units: a 16-row read touches every bank once
  kprof_begin(KP_MFMA, st);
  // 32-row blocks, two to a CU so that one's activations run beside the
  // other's products (96^3: 7.2 ms, against 7.7 ms for 64-row blocks, one to
  // a CU); grids that would give some of the 256 CUs no 32-row block take
  // 16-row blocks (3315 nodes: 41 us)
  if (a.nn > 256 * 32) trunk_launch<2, T>(a, out, st);
  else trunk_launch<1, T>(a, out, st);
  kprof_end(KP_MFMA, flops, st);
}
template void trunk_fused<double>(int, const int*, int, const int*, const double* const*, const double* const*, int,
                                  double*, hipStream_t);
template void trunk_fused<float>(int, const int*, int, const int*, const double* const*, const double* const*, int,
                                 float*, hipStream_t);

}  // namespace helm
