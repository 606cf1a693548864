// Products of the coarse space's set-up: the basis Q = P S, G = X^T X, and the Galerkin
// matrix X^T B - i X^T diag(Im s) X with B = (L - diag(Re s)) X, for X of n
// rows and r <= 128 columns (App. C).  All three are symmetric (L is, and X
// vanishes on masked rows), so only the 16 x 16 tiles on and above the diagonal are
// formed.
//
// Both operands of an MFMA on X^T Y hold row k of X or Y across 16 lanes, so
// they are loaded from memory as they lie, 16 columns of four rows at a time,
// three steps ahead, with no LDS and no barrier.  A product's tiles are split
// over two wavefronts of 18 (144 accumulator registers; NT = 4, r <= 64: five),
// rows {0, 1, 6, 7} and {2, 3, 4, 5} of the tile grid; X^T B and X^T diag(w) X run in
// one launch, four wavefronts reading the same rows of X.  A workgroup's
// wavefronts take its steps in turn and join their sums in order through LDS.
//
// What bounds it: the fp64 matrix instructions of the upper tiles (61 us at
// 64^3 x 128 for one product at the 78.6 TFLOP/s peak) against one reading of
// X (52 us at 5.15 TB/s) or of X and B.  The full square through LDS tiles with two
// barriers per 16 rows took 171 us for X^T X and 315 us for the other two at 64^3 x 128
// (76 us each for 12960 x 48, where few CUs had rows) and 28 us per sum of the
// blocks; this takes 88 and 180 us (5 and 6 us), the sums 5 and 9.
#include "common.h"
#include "dense.h"
#include "dense_dev.h"
#include "prof.h"

namespace helm {

// tile rows of role 0 and 1, and the tiles (row, column) they make
template <int NT>
struct GramTiles;
template <>
struct GramTiles<8> {
  static constexpr int N = 18, NR = 4;
  static constexpr int rows[2][4] = {{0, 1, 6, 7}, {2, 3, 4, 5}};
};
template <>
struct GramTiles<4> {
  static constexpr int N = 5, NR = 2;
  static constexpr int rows[2][4] = {{0, 3}, {1, 2}};
};

// one wavefront's tiles over the steps first, first + every, ... of four rows from x0
template <int NT, int ROLE, bool GAL, bool IM, typename S>
__device__ __forceinline__ void gram_sweep(const double* __restrict__ X, size_t ldx, const double* __restrict__ B,
                                           const cplx_t<S>* __restrict__ sc, size_t n, int r, size_t i0, int rows,
                                           int first, int every, int lane, d4 (&acc)[GramTiles<NT>::N]) {
  using G = GramTiles<NT>;
  constexpr int C0 = G::rows[ROLE][0], NC = NT - C0, DEPTH = 3;
  constexpr bool TWO = GAL && !IM;  // second operand from B
  const __amdgpu_buffer_rsrc_t xr = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<double*>(X + i0 * ldx), 0, (int)(8 * (size_t)rows * ldx), 0x00020000);
  const __amdgpu_buffer_rsrc_t br = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<double*>(TWO ? B + i0 * r : X), 0, TWO ? 8 * rows * r : 0, 0x00020000);
  // lane offsets; columns past r and rows past the range read as zero
  int xo[NC], bo[TWO ? NC : 1];
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    const int col = 16 * (C0 + c) + (lane & 15);
    xo[c] = col < r ? 8 * ((lane >> 4) * (int)ldx + col) : 0x7ffffff0;
    if (TWO) bo[c] = col < r ? 8 * ((lane >> 4) * r + col) : 0x7ffffff0;
  }
  const int steps = (rows + 3) / 4;
  double x[DEPTH][NC], y[DEPTH][TWO ? NC : 1], w[DEPTH];
  auto load = [&](int d, int s) {
    s = s < steps ? s : steps - 1;
    const int so = 32 * s * (int)ldx, sb = 32 * s * r;
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      bool need = !TWO;  // as a second operand, or as one of the role's rows
#pragma unroll
      for (int a = 0; a < G::NR; ++a) need |= G::rows[ROLE][a] == C0 + c;
      if (need) x[d][c] = __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(xr, xo[c], so, 0));
    }
    if constexpr (TWO)
#pragma unroll
      for (int c = 0; c < NC; ++c)
        y[d][c] = __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(br, bo[c], sb, 0));
    if constexpr (IM) {
      const size_t p = i0 + 4 * (size_t)s + (lane >> 4);
      w[d] = ldc(sc, p < n ? p : n - 1).y;
    }
    __builtin_amdgcn_sched_barrier(0);
  };
#pragma unroll
  for (int k = 0; k < G::N; ++k) acc[k] = d4{0, 0, 0, 0};
  if (rows == 0) return;  // a last block past the end
#pragma unroll
  for (int d = 0; d < DEPTH; ++d) load(d, first + d * every);
  for (int s = first; s < steps; s += DEPTH * every) {
#pragma unroll
    for (int d = 0; d < DEPTH; ++d) {
      if (s + d * every < steps) {
        int k = 0;
#pragma unroll
        for (int a = 0; a < G::NR; ++a) {
          const double av = IM ? w[d] * x[d][G::rows[ROLE][a] - C0] : x[d][G::rows[ROLE][a] - C0];
#pragma unroll
          for (int c = 0; c < NC; ++c)
            if (C0 + c >= G::rows[ROLE][a]) {
              acc[k] = mfma16(av, TWO ? y[d][c] : x[d][c], acc[k]);
              ++k;
            }
        }
      }
      load(d, s + (d + DEPTH) * every);
    }
  }
}

// block b: rows [b rpb, (b + 1) rpb); part[b][product][role][tile][register][lane].
// Eight wavefronts: role, product (GAL), and the share of the steps.
template <int NT, bool GAL, typename S>
__global__ __launch_bounds__(512, 2) void k_gram(size_t n, int r, const double* __restrict__ X, size_t ldx,
                                                 const double* __restrict__ B, const cplx_t<S>* __restrict__ sc,
                                                 size_t rpb, double* __restrict__ part) {
  using G = GramTiles<NT>;
  constexpr int KINDS = GAL ? 4 : 2, SHARES = 8 / KINDS;
  extern __shared__ __attribute__((aligned(16))) double sums[];  // KINDS x tiles x 256
  const int t = threadIdx.x, lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int kind = wave & (KINDS - 1), share = wave / KINDS;
  const size_t i0 = (size_t)blockIdx.x * rpb;
  const int rows = i0 < n ? (int)min(rpb, n - i0) : 0;
  d4 acc[G::N];
  if (kind == 0) gram_sweep<NT, 0, GAL, false, S>(X, ldx, B, sc, n, r, i0, rows, share, SHARES, lane, acc);
  else if (kind == 1) gram_sweep<NT, 1, GAL, false, S>(X, ldx, B, sc, n, r, i0, rows, share, SHARES, lane, acc);
  else if constexpr (GAL) {
    if (kind == 2) gram_sweep<NT, 0, true, true, S>(X, ldx, B, sc, n, r, i0, rows, share, SHARES, lane, acc);
    else gram_sweep<NT, 1, true, true, S>(X, ldx, B, sc, n, r, i0, rows, share, SHARES, lane, acc);
  }
  double* sum = sums + kind * G::N * 256 + lane;
  for (int h = 1; h < SHARES; ++h) {
    if (share == h)
#pragma unroll
      for (int k = 0; k < G::N; ++k)
#pragma unroll
        for (int i = 0; i < 4; ++i) sum[256 * k + 64 * i] = acc[k][i];
    __syncthreads();
    if (share == 0)
#pragma unroll
      for (int k = 0; k < G::N; ++k)
#pragma unroll
        for (int i = 0; i < 4; ++i) acc[k][i] += sum[256 * k + 64 * i];
    __syncthreads();
  }
  if (share == 0) {
    double* out = part + ((size_t)blockIdx.x * KINDS + kind) * G::N * 256 + lane;
#pragma unroll
    for (int k = 0; k < G::N; ++k)
#pragma unroll
      for (int i = 0; i < 4; ++i) out[256 * k + 64 * i] = acc[k][i];
  }
}

// out = the blocks' sum, mirrored to the full matrix (GAL: complex, -i times the second
// product).  A workgroup takes 64 entries, each wavefront an eighth of the blocks,
// eight loads in flight; one thread per entry over all blocks in turn took 28 us.
template <int NT, bool GAL>
__global__ __launch_bounds__(512) void k_gram_sum(int nb, int r, const double* __restrict__ part,
                                                  double* __restrict__ out) {
  using G = GramTiles<NT>;
  constexpr int WIDTH = (GAL ? 4 : 2) * G::N * 256;
  __shared__ double sh[8][64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, e = blockIdx.x * 64 + lane;
  const int each = (nb + 7) / 8, b1 = min(nb, (wave + 1) * each);
  double acc = 0.0;
  for (int b = wave * each; b < b1; b += 8) {
    double v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) v[u] = b + u < b1 ? part[(size_t)(b + u) * WIDTH + e] : 0.0;
#pragma unroll
    for (int u = 0; u < 8; ++u) acc += v[u];
  }
  sh[wave][lane] = acc;
  __syncthreads();
  if (wave) return;
#pragma unroll
  for (int u = 1; u < 8; ++u) acc += sh[u][lane];
  const int kind = e / (G::N * 256), k = e / 256 % G::N, role = kind & 1, im = kind >> 1;
  int row = 0, col = 0, at = 0;
  for (int a = 0; a < G::NR; ++a)
    for (int c = G::rows[role][a]; c < NT; ++c, ++at)
      if (at == k) {
        row = 16 * G::rows[role][a] + acc_row(lane, e / 64 % 4);
        col = 16 * c + (lane & 15);
      }
  if (row >= r || col >= r) return;
  auto put = [&](int i, int j) {
    if (GAL) out[2 * ((size_t)i * r + j) + im] = im ? -acc : acc;
    else out[(size_t)i * r + j] = acc;
  };
  put(row, col);
  if (row >> 4 != col >> 4) put(col, row);
}

// Q = P S (P: n x K, row stride ldp; S: K x r; K a multiple of 16): 32 rows of P
// through LDS, S from L2 into registers (trunk_layer), wavefront w the columns
// 16 w .. + 15.  upper: S is upper triangular, so those columns need k < 16 (w + 1)
// only.  Bound by the reading of P and the writing of Q (104 us at 64^3 x 128 at
// 5.15 TB/s); the 128 x 128 tiles of k_gemm over all k, two barriers per 16 k, took
// 216 us (106 at 56 x 48 x 52 x 96, 18 at 12960 x 48); this 157 (57, 6).
__global__ __launch_bounds__(64 * TRUNK_WAVES, 6) void k_basis(size_t n, int K, int r, const double* __restrict__ P,
                                                               size_t ldp, const double* __restrict__ S, int upper,
                                                               double* __restrict__ Q) {
  extern __shared__ __attribute__((aligned(16))) double h[];  // 32 x lda
  const int t = trunk_thread(), lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6), lda = K + 2;
  const size_t row0 = (size_t)blockIdx.x * 32;
  for (int e = t; e < 32 * K; e += 64 * TRUNK_WAVES) {
    const int i = e / K, k = e % K;
    h[i * lda + k] = row0 + i < n ? P[(row0 + i) * ldp + k] : 0.0;
  }
  __syncthreads();
  if (16 * wave >= r) return;
  d4 acc[2][1];
  trunk_layer<2, 1>(h, lda, S, K, r, wave, lane, acc, upper ? min(K, 16 * (wave + 1)) : K);
  const int col = 16 * wave + (lane & 15);
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const size_t row = row0 + 16 * a + acc_row(lane, i);
      if (row < n && col < r) Q[row * r + col] = acc[a][0][i];
    }
}

// One workgroup (eight wavefronts, two to a SIMD) per CU; fewer where a
// workgroup would get less than 32 rows, one step or more for each share.
static int gram_blocks(size_t n) { return (int)(n < 256 * 32 ? (n + 31) / 32 : 256); }

size_t gram_part(size_t n, int r) { return (size_t)gram_blocks(n) * 4 * 256 * (r > 64 ? 18 : 5); }

template <int NT, bool GAL, typename S>
static void gram_launch(size_t n, int r, const double* X, size_t ldx, const double* B, const cplx_t<S>* sc,
                        double* part, double* out, hipStream_t st) {
  constexpr int kinds = GAL ? 4 : 2, lds = kinds * GramTiles<NT>::N * 256 * (int)sizeof(double);
  const int nb = gram_blocks(n);
  const size_t rpb = ((n + nb - 1) / nb + 3) / 4 * 4;
  (void)hipFuncSetAttribute((const void*)k_gram<NT, GAL, S>, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
  kprof_begin(KP_MFMA, st);
  hipLaunchKernelGGL((k_gram<NT, GAL, S>), dim3(nb), dim3(512), lds, st, n, r, X, ldx, B, sc, rpb, part);
  kprof_end(KP_MFMA, (GAL ? 2.0 : 1.0) * (double)n * r * (r + 1), st);
  hipLaunchKernelGGL((k_gram_sum<NT, GAL>), dim3(kinds * GramTiles<NT>::N * 4), dim3(512), 0, st, nb, r, part, out);
}

void gram(size_t n, int r, const double* X, size_t ldx, double* part, double* out, hipStream_t st) {
  // columns past 64 need the 8 x 8 tile grid: 36 tiles instead of 10
  if (r > 64) gram_launch<8, false, double>(n, r, X, ldx, nullptr, nullptr, part, out, st);
  else gram_launch<4, false, double>(n, r, X, ldx, nullptr, nullptr, part, out, st);
}

template <typename S>
void gram_galerkin(size_t n, int r, const double* X, const double* B, const cplx_t<S>* sc, double* part, double* Ac,
                   hipStream_t st) {
  if (r > 64) gram_launch<8, true, S>(n, r, X, r, B, sc, part, Ac, st);
  else gram_launch<4, true, S>(n, r, X, r, B, sc, part, Ac, st);
}
template void gram_galerkin<double>(size_t, int, const double*, const double*, const cplx_t<double>*, double*, double*,
                                    hipStream_t);
template void gram_galerkin<float>(size_t, int, const double*, const double*, const cplx_t<float>*, double*, double*,
                                   hipStream_t);

void basis(size_t n, int K, int r, const double* P, size_t ldp, const double* S, bool upper, double* Q,
           hipStream_t st) {
  if (K % 16) {  // k steps that S's rows do not fill
    gemm<double>((int)n, r, K, P, ldp, S, r, nullptr, ACT_NONE, Q, r, st);
    return;
  }
  kprof_begin(KP_MFMA, st);
  hipLaunchKernelGGL(k_basis, dim3((unsigned)((n + 31) / 32)), trunk_block(),
                     32 * (K + 2) * sizeof(double), st, n, K, r, P, ldp, S, upper ? 1 : 0, Q);
  kprof_end(KP_MFMA, (upper ? 1.0 : 2.0) * (double)n * K * r, st);
}

}  // namespace helm
