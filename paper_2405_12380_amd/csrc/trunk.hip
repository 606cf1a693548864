// Trunk evaluation in one launch (App. B architecture, App. C trunk matrix): a
// workgroup carries a block of grid nodes through every layer, the
// activations staying in LDS, so only T leaves the chip.
//
// Two forms: products in fp64 (first), and the products of tanh layers in
// fixed point on the int8 matrix units (below).
//
// What bounds the fp64 form: the fp64 matrix instructions (the hidden layers are
// 2 w^2 flop per node and layer; at w = 256 a node's 2 KiB of activations would
// otherwise be written and read once per layer) and, since they share the
// fp64 units, the activation's vector arithmetic.  Layer by layer, with a
// 128 x 128 tile staged through LDS in 16-deep chunks, the products ran at 41
// of the 78.6 TFLOP/s peak: two barriers per chunk, and every activation value
// stored to and loaded from memory.  Measured (3-256x4-128 trunk): 10.19 ->
// 7.07 ms at 96^3 (58 TFLOP/s; the library's fp64 product of two 8192 x 8192
// matrices reaches 71), 299 -> 157 us at 24 x 20 x 27, 279 -> 50 us at
// 15 x 17 x 13, where most CUs had no tile.
#include "common.h"
#include "dense.h"
#include "dense_dev.h"
#include "prof.h"

#include <type_traits>

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
  const int t = threadIdx.x, lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
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

// ---- the layers' products in fixed point ---------------------------------------------
// H W of a tanh layer on the int8 matrix units, by splitting both factors into
// digits (Ozaki, Ogita, Oishi, Rump 2012; in integers Ootomo, Ozaki, Yokota 2024):
// a node's row of H and a column of W are each scaled by a power of two and
// rounded to 56-bit fixed point (error at most 2^-56 of the largest entry's
// power of two), written as seven balanced base-256 digits.  The
// 28 digit products of weight 256^6 and above are summed exactly in int32, by
// weight, over all k (at most 7 * 256 * 2^14 < 2^25), then joined in fp64; the
// 21 below add up to less than a double product's rounding errors.  Against
// 80-bit products the whole trunk's error is 2 to 5 times smaller than the fp64
// path's (3-256x4-128: 2.1e-16 of T, fp64 9.8e-16; 3-32x4-128: 2.4e-16, 4.0e-16).
// The scales are the row's and the column's, so a value far below both has less
// relative precision than in fp64; k_trunk_digits therefore refuses weights
// where one entry dominates a column (a result could be a small h alone), and
// rows are rescaled after every layer.
//
// What bounds it: per 32 x 32 tile and 32-deep chunk 28 matrix instructions of
// 32 cycles, where fp64 takes 32 of 64 (1.6 M of the 3.1 M busy cycles of a
// 64^3 grid), and the vector units' joining of the sums, tanh and digits
// (70 instructions per value, 1.2 M cycles).  The two do not run side by side,
// with one or two workgroups to a CU, and the clock falls to 1.7 GHz meanwhile.
// Measured (3-256x4-128 trunk), fp64 products -> these: 7.07 -> 5.66 ms at
// 96^3, 2100 -> 1715 us at 64^3, 1260 -> 990 us at 56 x 48 x 52, 155 -> 113 us at
// 24 x 20 x 27, 86 -> 63 us at 31 x 33 x 8.
typedef int i4 __attribute__((ext_vector_type(4)));
typedef int i16 __attribute__((ext_vector_type(16)));
constexpr int DIG = 7;

// The matrix operands hold feature 8 (i / 4) + 4 h + i % 4 of a 32-feature
// chunk in byte i of lanes 32 h .. 32 h + 31: the order in which a lane's
// sixteen results of the product before come out, so each lane writes and
// reads its own 16 bytes of every digit.
__device__ __forceinline__ int feature(int half, int i) { return 8 * (i >> 2) + 4 * half + (i & 3); }

// power of two e with |x| <= 0.996 * 2^e (the largest digit sum is 127 / 255 of
// 2^56), of the magnitude whose high word is hi
__device__ __forceinline__ int fix_exp(int hi) { return ((hi + 0x2100) >> 20) - 1022; }

// digits of v[i] * sc, |v * sc| <= 0.996: with B = 0x80808080808080 the bytes of
// round(v sc 2^55) + B, less 128 each.  Two additions of 1.5 * 2^52 units (one
// of 2^-23, one of 2^-55) round and leave the integers in the low words; the
// second's bit 32 carries into the first.
__device__ __forceinline__ void digits16(const double (&v)[16], double sc, i4 (&d)[DIG]) {
  constexpr double c1 = 805306368.0 + 8421504.0 * 0x1p-23, c2 = 0.1875 + 2155905152.0 * 0x1p-55;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    unsigned lo[4], hi[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const double x = v[4 * q + e], t = fma(x, sc, c1), f = t - c1, u = fma(x, sc, -f) + c2;
      lo[e] = (unsigned)__double2loint(u);
      hi[e] = (unsigned)__double2loint(t) + (unsigned)(__double2hiint(u) - 0x3FC80000);
    }
    // 4 x 4 byte transposes
    const unsigned a = __builtin_amdgcn_perm(lo[1], lo[0], 0x05010400), b = __builtin_amdgcn_perm(lo[3], lo[2], 0x05010400);
    const unsigned c = __builtin_amdgcn_perm(lo[1], lo[0], 0x07030602), g = __builtin_amdgcn_perm(lo[3], lo[2], 0x07030602);
    const unsigned k = __builtin_amdgcn_perm(hi[1], hi[0], 0x05010400), l = __builtin_amdgcn_perm(hi[3], hi[2], 0x05010400);
    const unsigned m = __builtin_amdgcn_perm(hi[1], hi[0], 0x07030602), n = __builtin_amdgcn_perm(hi[3], hi[2], 0x07030602);
    d[0][q] = (int)(__builtin_amdgcn_perm(b, a, 0x05040100) ^ 0x80808080u);
    d[1][q] = (int)(__builtin_amdgcn_perm(b, a, 0x07060302) ^ 0x80808080u);
    d[2][q] = (int)(__builtin_amdgcn_perm(g, c, 0x05040100) ^ 0x80808080u);
    d[3][q] = (int)(__builtin_amdgcn_perm(g, c, 0x07060302) ^ 0x80808080u);
    d[4][q] = (int)(__builtin_amdgcn_perm(l, k, 0x05040100) ^ 0x80808080u);
    d[5][q] = (int)(__builtin_amdgcn_perm(l, k, 0x07060302) ^ 0x80808080u);
    d[6][q] = (int)(__builtin_amdgcn_perm(n, m, 0x05040100) ^ 0x80808080u);
  }
}

// Digits of one layer's W (K x N, one workgroup per 32 columns; columns past N
// zero) in the order the product loads them, [tile][chunk][digit][lane], and
// the columns' exponents less 54 (the sums' unit).  check: only look for
// non-finite values.  flag[0] |= 1 where a weight or bias is not finite, or an
// entry exceeds 16 times its column's mean magnitude.
__global__ __launch_bounds__(256) void k_trunk_digits(int K, int N, const double* __restrict__ W,
                                                      const double* __restrict__ b, int check, i4* __restrict__ dig,
                                                      int* __restrict__ ec, int* __restrict__ flag) {
  __shared__ double mx[8][32], sm[8][32];
  __shared__ int ex[32];
  const int t = threadIdx.x, tile = blockIdx.x, col = 32 * tile + (t & 31);
  double m = 0.0, s = 0.0;
  bool bad = false;
  if (col < N) {
    bad = !isfinite(b[col]);
    for (int k = t >> 5; k < K; k += 8) {
      const double v = fabs(W[(size_t)k * N + col]);
      bad |= !isfinite(v);
      m = fmax(m, v);
      s += v / K;
    }
  }
  mx[t >> 5][t & 31] = m;
  sm[t >> 5][t & 31] = s;
  __syncthreads();
  if (t < 32) {
    for (int i = 1; i < 8; ++i) {
      m = fmax(m, mx[i][t]);
      s += sm[i][t];
    }
    ex[t] = fix_exp(__double2hiint(m));
    if (!check) {
      ec[col] = ex[t] - 54;
      bad |= m > 16.0 * s;
    }
  }
  if (bad) atomicOr(flag, 1);
  if (check) return;
  __syncthreads();
  const int nc = K / 32;
  for (int e = t; e < 64 * nc; e += 256) {
    const int c = e >> 6, lane = e & 63, cl = 32 * tile + (lane & 31);
    double v[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const double x = cl < N ? W[(size_t)(32 * c + feature(lane >> 5, i)) * N + cl] : 0.0;
      v[i] = isfinite(x) ? ldexp(x, -ex[lane & 31]) : 0.0;
    }
    i4 d[DIG];
    digits16(v, 1.0, d);
#pragma unroll
    for (int q = 0; q < DIG; ++q) dig[((size_t)(tile * nc + c) * DIG + q) * 64 + lane] = d[q];
  }
}

__global__ void k_clear_flag(int* flag) { flag[0] = 0; }

struct TrunkFixArgs {
  TrunkArgs t;
  const i4* dig;               // all layers' digits
  const int* ec;               // and column exponents
  int doff[TRUNK_MAXL], eoff[TRUNK_MAXL], dbytes;
};

// fp64 of an int32 (the conversion instruction is slower)
__device__ __forceinline__ double from_int(int a) {
  return __hiloint2double(0x43300000, a ^ (int)0x80000000) - 4503601774854144.0;
}

// 32 nodes through all layers.  Products are taken transposed, W^T H^T: a lane's
// results are sixteen features of node lane % 32.  Wavefront w takes feature
// tile w; the digits of all features are in LDS, those of W stream from L2 into
// registers, each digit's register refilled for the next chunk once its last
// product is issued.
template <typename T>
__global__ __launch_bounds__(64 * TRUNK_WAVES, 2) void k_trunk_fix(TrunkFixArgs a, T* __restrict__ out) {
  __shared__ i4 dig[8][DIG][64];
  __shared__ int rmax[2][32];
  const int t = threadIdx.x, lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int half = lane >> 5, L = a.t.L;
  const size_t row = (size_t)blockIdx.x * 32 + (lane & 31);
  const __amdgpu_buffer_rsrc_t wr =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<i4*>(a.dig), 0, a.dbytes, 0x00020000);
  i4 wv[DIG];
  auto load_w = [&](int s, int so) {
    wv[s] = __builtin_bit_cast(i4, __builtin_amdgcn_raw_buffer_load_b128(wr, 16 * lane, so + 1024 * s, 0));
  };
  auto tiles = [&](int l) { return (a.t.w[l + 1] + 31) >> 5; };
  // the first digits of the wavefront's next product, from layer l on, are loaded ahead
  auto load_ahead = [&](int l) {
    while (l < L && wave >= tiles(l)) ++l;
    if (l < L) {
      const int so = a.doff[l] + wave * (a.t.w[l] >> 5) * (1024 * DIG);
#pragma unroll
      for (int s = DIG - 1; s >= 0; --s) load_w(s, so);
    }
  };
  load_ahead(1);
  if (t < 64) (&rmax[0][0])[t] = 0;
  __syncthreads();
  double v[16];
  int buf = 0, er = 0;
  // tanh layer done: its rows' scales, then its digits
  auto publish = [&](int nt) {
    int m = 0;
    if (wave < nt)
#pragma unroll
      for (int i = 0; i < 16; ++i) m = max(m, __double2hiint(v[i]) & 0x7fffffff);
    m = max(m, __shfl_xor(m, 32));
    if (lane < 32) atomicMax(&rmax[buf][lane], m);
    __syncthreads();  // the scales are there, and every wavefront has read this layer's input
    er = fix_exp(rmax[buf][lane & 31]);
    buf ^= 1;
    if (t < 32) rmax[buf][t] = 0;
    const double sc = __hiloint2double((1023 - er) << 20, 0);
    if (wave < nt) {
      i4 d[DIG];
      digits16(v, sc, d);
#pragma unroll
      for (int s = 0; s < DIG; ++s) dig[wave][s][lane] = d[s];
    }
    __syncthreads();
  };
  {  // input layer on the node coordinates
    const size_t p = row < a.t.nn ? row : a.t.nn - 1;  // rows past the end repeat the last node
    const int nx = a.t.n[0], ny = a.t.n[1], N1 = a.t.w[1];
    const double x = (double)((int)(p % nx) + 1) / (double)(nx + 1);
    const double y = (double)((int)((p / nx) % ny) + 1) / (double)(ny + 1);
    const double z = (double)((int)(p / ((size_t)nx * ny)) + 1) / (double)(a.t.n[2] + 1);
    if (wave < tiles(0))
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const int c = 32 * wave + feature(half, i);
        double h = x * a.t.W[0][c];
        h += y * a.t.W[0][N1 + c];
        if (a.t.dim > 2) h += z * a.t.W[0][2 * N1 + c];
        v[i] = tanh_fast<false>(h + a.t.b[0][c]);
      }
    publish(tiles(0));
  }
  for (int l = 1; l < L; ++l) {
    const int nt = tiles(l), nc = a.t.w[l] >> 5, N = a.t.w[l + 1];
    const bool last = l + 1 == L;
    if (wave < nt) {
      i16 acc[DIG];  // by digit weight 256^(6 + q)
      i4 hv[DIG];
#pragma unroll
      for (int q = 0; q < DIG; ++q) acc[q] = i16{};
#pragma unroll
      for (int s = 0; s < DIG; ++s) hv[s] = dig[0][s][lane];
      int so = a.doff[l] + wave * nc * (1024 * DIG);
      auto chunk = [&](int c, auto more) {
        so += 1024 * DIG;
#pragma unroll
        for (int i = DIG - 1; i >= 0; --i) {
#pragma unroll
          for (int j = DIG - 1 - i; j < DIG; ++j)
            acc[i + j - 6] = __builtin_amdgcn_mfma_i32_32x32x32_i8(wv[i], hv[j], acc[i + j - 6], 0, 0, 0);
          if constexpr (more.value) {
            load_w(i, so);
            hv[DIG - 1 - i] = dig[c + 1][DIG - 1 - i][lane];
            __builtin_amdgcn_sched_barrier(0);
          }
        }
      };
      for (int c = 0; c + 1 < nc; ++c) chunk(c, std::true_type{});
      chunk(nc - 1, std::false_type{});
      load_ahead(l + 1);
      __builtin_amdgcn_sched_barrier(0);
      // four results; their columns are c .. c + 3
      auto join = [&](int q, int c, double (&x)[4]) {
        const i4 ec = *reinterpret_cast<const i4*>(a.ec + a.eoff[l] + c);
        const double2 b0 = *reinterpret_cast<const double2*>(a.t.b[l] + c);
        const double2 b1 = *reinterpret_cast<const double2*>(a.t.b[l] + c + 2);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int i = 4 * q + e;
          double y = from_int((acc[6][i] << 8) + acc[5][i]);
          y = fma(y, 256.0, from_int(acc[4][i]));
          y = fma(y, 256.0, from_int(acc[3][i]));
          y = fma(y, 256.0, from_int(acc[2][i]));
          y = fma(y, 256.0, from_int(acc[1][i] + ((acc[0][i] + 128) >> 8)));
          x[e] = ldexp(y, er + ec[e]) + (e < 2 ? (e ? b0.y : b0.x) : e == 2 ? b1.x : b1.y);
        }
      };
      if (last) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int c = 32 * wave + feature(half, 4 * q);
          if (c >= N) continue;  // N is a multiple of 16: all four columns or none
          double x[4];
          join(q, c, x);
          if (row < a.t.nn)
#pragma unroll
            for (int e = 0; e < 4; ++e) out[row * N + c + e] = (T)x[e];
        }
      } else {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          double x[4];
          join(q, 32 * wave + feature(half, 4 * q), x);
#pragma unroll
          for (int e = 0; e < 4; ++e) v[4 * q + e] = tanh_fast<false>(x[e]);
        }
      }
    }
    if (!last) publish(nt);
  }
}

// bytes of a network's digits, their flag and column exponents; offsets by layer
static size_t fix_layout(int L, const int* w, TrunkFixArgs* a) {
  size_t d = 0, e = 4;  // ec[0] is the flag
  for (int l = 1; l < L; ++l) {
    if (a) {
      a->doff[l] = (int)d;
      a->eoff[l] = (int)e;
    }
    const size_t tiles = ((size_t)w[l + 1] + 31) / 32;
    d += tiles * (w[l] / 32) * DIG * 1024;
    e += 32 * tiles;
  }
  if (a) a->dbytes = (int)d;
  return d + e * sizeof(int);
}

size_t trunk_fix_bytes(int L, const int* w) { return fix_layout(L, w, nullptr); }

const int* trunk_fix_build(int L, const int* w, const double* const* W, const double* const* b, void* buf,
                           hipStream_t st) {
  TrunkFixArgs a{};
  fix_layout(L, w, &a);
  int* ec = (int*)((char*)buf + a.dbytes);
  hipLaunchKernelGGL(k_clear_flag, dim3(1), dim3(1), 0, st, ec);
  for (int l = 0; l < L; ++l)
    hipLaunchKernelGGL(k_trunk_digits, dim3((unsigned)((w[l + 1] + 31) / 32)), dim3(256), 0, st, w[l], w[l + 1], W[l],
                       b[l], l == 0, (i4*)((char*)buf + a.doff[l]), ec + a.eoff[l], ec);
  return ec;
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
  hipLaunchKernelGGL((k_trunk<RT, T>), dim3((unsigned)((a.nn + rows - 1) / rows)), dim3(64 * TRUNK_WAVES), lds, st, a,
                     out);
}

template <typename T>
void trunk_fused(int dim, const int n[3], int L, const int* w, const double* const* W, const double* const* b, int act,
                 const void* fix, T* out, hipStream_t st) {
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
  // Fixed-point products wherever the weights have digits, but for grids whose
  // 16-row fp64 blocks all run at once, one to a CU (3315 nodes: 50 us, against 55
  // in fixed point; 8184 nodes, two fp64 blocks to a CU: 86 against 63)
  if (fix && a.nn > 256 * 16) {
    TrunkFixArgs f{};
    f.t = a;
    fix_layout(L, w, &f);
    f.dig = (const i4*)fix;
    f.ec = (const int*)((const char*)fix + f.dbytes);
    hipLaunchKernelGGL(k_trunk_fix<T>, dim3((unsigned)((a.nn + 31) / 32)), dim3(64 * TRUNK_WAVES), 0, st, f, out);
    kprof_end(KP_MFMA, flops, st);
    return;
  }
  // 32-row blocks, two to a CU so that one's activations run beside the
  // other's products (96^3: 7.2 ms, against 7.7 ms for 64-row blocks, one to
  // a CU); grids that would give some of the 256 CUs no 32-row block take
  // 16-row blocks (3315 nodes: 50 us)
  if (a.nn > 256 * 32) trunk_launch<2, T>(a, out, st);
  else trunk_launch<1, T>(a, out, st);
  kprof_end(KP_MFMA, flops, st);
}
template void trunk_fused<double>(int, const int*, int, const int*, const double* const*, const double* const*, int,
                                  const void*, double*, hipStream_t);
template void trunk_fused<float>(int, const int*, int, const int*, const double* const*, const double* const*, int,
                                 const void*, float*, hipStream_t);

}  // namespace helm
