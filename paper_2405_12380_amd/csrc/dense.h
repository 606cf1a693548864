// Launchers of the dense kernels (DeepONet layers, Gram products, small
// one-workgroup factorizations).  All enqueue on `st` and return at once.
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>

#include "common.h"

namespace helm {

enum { ACT_NONE = -1, ACT_TANH = 0, ACT_RELU = 1, ACT_LEAKY = 2 };

// h[r][c] = act(sum_d x_{row0+r}[d] W[d][c] + b[c]) with x_p the coordinates of
// grid node p (x-fastest numbering, (i+1)/(n+1) per axis), r < nrows, c < N
// (instantiated for double)
template <typename T>
void coord_layer(int dim, const int n[3], size_t row0, size_t nrows, const T* W, const T* b, int N, int act, T* out,
                 hipStream_t st);
// out = the trunk matrix T (nn x w[L], row-major) of the grid's nodes: all L layers
// (W[l]: w[l] x w[l + 1], hidden activation act, last layer linear) in one
// launch, fp64 arithmetic, rounded once to T as stored.  Only for widths that
// trunk_fused_fits accepts.
constexpr int TRUNK_MAXL = 8;
bool trunk_fused_fits(int L, const int* w);
template <typename T>
void trunk_fused(int dim, const int n[3], int L, const int* w, const double* const* W, const double* const* b, int act,
                 T* out, hipStream_t st);
// C = act(A W + bias) (fp64 MFMA; instantiated for double); bias may be NULL;
// act = ACT_NONE for linear
template <typename T>
void gemm(int M, int N, int K, const T* A, size_t lda, const T* W, size_t ldw, const T* bias, int act, T* C,
          size_t ldc, hipStream_t st);
// y[b][n] = act(sum_k x[b][k] W[k][n] + bias[n]) for a batch B <= 4 (split-K,
// fp64 accumulation, bias and activation; y rounded once to T);
// part needs small_ksplit(K) * B * N doubles
int small_ksplit(int K);
template <typename T>
void dense_small(int B, int N, int K, const T* x, const T* W, const T* bias, int act, T* y, double* part,
                 hipStream_t st);
// Q = P S (P: n x K, row stride ldp; S: K x r, upper: upper triangular; r, K <= 128)
void basis(size_t n, int K, int r, const double* P, size_t ldp, const double* S, bool upper, double* Q,
           hipStream_t st);
// out (r x r) = X^T X for X of n rows (row stride ldx), r <= 128; part: gram_part(n, r) doubles
size_t gram_part(size_t n, int r);
void gram(size_t n, int r, const double* X, size_t ldx, double* part, double* out, hipStream_t st);
// Ac (complex r x r) = X^T B - i X^T diag(Im s) X, both products symmetric (X, B:
// n x r; s: n complex values; instantiated for double and float)
template <typename S>
void gram_galerkin(size_t n, int r, const double* X, const double* B, const cplx_t<S>* s, double* part, double* Ac,
                   hipStream_t st);
// Cholesky with dropping of columns whose remaining squared norm is <= tau2 times
// the largest squared column norm, G (p x p, symmetric, p <= 128) = P^T P; S:
// p x rank so that P S is orthonormal (p * p capacity); info: 2 ints (rank, failed)
void chol_drop(int p, const double* G, double tau2, int allow_drop, double* S, int* info, hipStream_t st);
// inverse of the complex r x r matrix A (interleaved); work: 4*r*r doubles;
// info: 1 int (1 = singular); cond: 1 double
void gj_inverse(int r, const double* A, double* work, double* Ainv, int* info, double* cond, hipStream_t st);

}  // namespace helm
