// Stencil kernels of the discrete Helmholtz operator (§2 eq. 1) and of the
// point relaxations of eq. 2 (damped Jacobi, red-black Gauss-Seidel).
//
// Mapping: a workgroup is 64 x ty threads (ty = 4, or 8 on large grids),
// lanes along x (a wavefront reads
// one contiguous 1 KiB (complex128) row segment per load), 4 rows in y, and
// each thread marches over `zb` consecutive z-planes keeping the z-1, z, z+1
// values of its column in registers, so every node is loaded from HBM once;
// x/y neighbours are re-read from L1/L2.  Masks enter through one neighbour
// code byte per node, so all loads of a node are independent and issued
// together.  Logical blocks are laid out x-, y-,
// then z-fastest and remapped so that each XCD owns one contiguous range of
// them (one z-slab), keeping halo re-reads inside that XCD's L2.
//
// Per-node arithmetic is fixed (independent of the tiling): the axis terms
// ((c - x_minus) + (c - x_plus)) / h_a^2 are accumulated x, y, z in turn and
// s_p c is subtracted last, in fp64 for both storage precisions.
#include "common.h"

#include <type_traits>
#include "internal.h"
#include "prof.h"
#include "stencil_dev.h"

namespace helm {

__global__ void k_build_codes(int dim, int nx, int ny, int nz, const uint8_t* __restrict__ mask,
                              uint8_t* __restrict__ code) {
  const size_t n = (size_t)nx * ny * nz, plane = (size_t)nx * ny;
  for (size_t p = blockIdx.x * (size_t)blockDim.x + threadIdx.x; p < n; p += (size_t)gridDim.x * blockDim.x) {
    const int i = (int)(p % nx), j = (int)((p / nx) % ny), l = (int)(p / plane);
    uint8_t c = mask[p] ? NB_SELF : 0;
    if (i == 0 || mask[p - 1]) c |= NB_XM;
    if (i + 1 == nx || mask[p + 1]) c |= NB_XP;
    if (j == 0 || mask[p - nx]) c |= NB_YM;
    if (j + 1 == ny || mask[p + nx]) c |= NB_YP;
    if (dim == 3) {
      if (l == 0 || mask[p - plane]) c |= NB_ZM;
      if (l + 1 == nz || mask[p + plane]) c |= NB_ZP;
    }
    code[p] = c;
  }
}

static int stencil_blocks(const StencilGeom& g) {
  const int rows = g.ty * g.rows;
  const int nbx = (g.nx + 63) / 64, nby = (g.ny + rows - 1) / rows, nbz = (g.nz + g.zb - 1) / g.zb;
  return nbx * nby * nbz;
}

template <typename S, int DIM, int MODE, int R>
__global__ __launch_bounds__(512) void k_stencil(StencilGeom g, const cplx_t<S>* __restrict__ sc,
                                                 const uint8_t* __restrict__ code, const cplx_t<S>* x,
                                                 const cplx_t<S>* __restrict__ f, cplx_t<S>* y,
                                                 double omega, int color, double* __restrict__ partials) {
  const unsigned lb = xcd_remap(blockIdx.x, gridDim.x);
  stencil_tile<S, DIM, MODE, R>(g, lb, sc, code, x, f, y, omega, color, MODE == ST_RESID ? partials + lb : nullptr);
}

template <typename S, int DIM, int R>
__global__ __launch_bounds__(512) void k_jacobi2z(StencilGeom g, const cplx_t<S>* __restrict__ sc,
                                                  const uint8_t* __restrict__ code, const cplx_t<S>* __restrict__ f,
                                                  cplx_t<S>* __restrict__ y, double omega,
                                                  const double* __restrict__ fscale, cplx_t<S>* __restrict__ fout) {
  jacobi2z_tile<S, DIM, R>(g, xcd_remap(blockIdx.x, gridDim.x), sc, code, f, y, omega, fscale, fout);
}

// One red-black Gauss-Seidel sweep in a single pass, out of place (uin -> uout):
// red nodes ((i + j + z) even) get the relaxation update from uin; black nodes
// get it from the red values just computed at their six neighbours.  Every
// thread keeps the new red values of its own column at z - 1, z and z + 1 in
// registers; the in-plane ones are exchanged through LDS, and threads on the
// tile's rim recompute the red value of the neighbouring tile's node (from uin,
// so no other workgroup's output is ever read).  The per-node arithmetic is that
// of the two colour passes of k_stencil<RBGS>, so the result is the same; HBM
// sees one pass (uin, f, s and the code byte read, uout written).
// the relaxation update at node (i, j, z) from the values of x alone (a red
// node), rounded to the storage precision: the black updates read red values
// as if the two colours were separate passes through memory
template <typename S, int DIM>
__device__ __forceinline__ double2 red_at(const StencilGeom& g, const cplx_t<S>* __restrict__ sc,
                                          const uint8_t* __restrict__ code, const cplx_t<S>* __restrict__ x,
                                          const cplx_t<S>* __restrict__ f, int i, int j, int z, double omega) {
  const size_t plane = (size_t)g.nx * g.ny;
  const size_t p = (size_t)i + (size_t)g.nx * ((size_t)j + (size_t)g.ny * z);
  const unsigned cd = code[p];
  const ptrdiff_t oxm = i > 0 ? -1 : 0, oxp = i + 1 < g.nx ? 1 : 0;
  const ptrdiff_t oym = j > 0 ? -(ptrdiff_t)g.nx : 0, oyp = j + 1 < g.ny ? (ptrdiff_t)g.nx : 0;
  double2 q = czero(), w = czero();
  if (DIM == 3) {
    if (z > 0) q = ldc(x, p - plane);
    if (z + 1 < g.nz) w = ldc(x, p + plane);
  }
  return rnd_store<S>(relax_upd<S>(g, cd, ldc(x, p), ldc(x, p + oxm), ldc(x, p + oxp), ldc(x, p + oym),
                                   ldc(x, p + oyp), q, w, ldc(sc, p), ldc(f, p), omega, DIM == 3));
}

// Thread (tx, ty) owns the node pair x = 2 tx, 2 tx + 1 of row j in a 128 x ty
// tile: in every plane one of the pair is red and the other black, so every
// lane does one red and one black update (no checkerboard divergence).  The
// black node's red neighbours: along x its own red node and the neighbouring
// lane's (a wavefront is one row; the tile's outer neighbours are recomputed by
// lanes 0 and 63), along y the red nodes of the rows above and below (LDS; the
// tile's outer rows recomputed by the first and last row), along z the red
// values of its own column below and above (the one above is also the red node
// of the next plane, computed once).
template <typename S, int DIM>
__global__ __launch_bounds__(512) void k_rbgs_fused(StencilGeom g, const cplx_t<S>* __restrict__ sc,
                                                    const uint8_t* __restrict__ code, const cplx_t<S>* __restrict__ uin,
                                                    const cplx_t<S>* __restrict__ f, cplx_t<S>* __restrict__ uout,
                                                    double omega) {
  __shared__ double2 red[8][128];  // new red values of the current plane (ty <= 8)
  const unsigned lb = xcd_remap(blockIdx.x, gridDim.x);
  const unsigned nbx = (g.nx + 127) / 128, nby = (g.ny + g.ty - 1) / g.ty;
  const unsigned bx = lb % nbx, by = (lb / nbx) % nby, bz = lb / (nbx * nby);
  const int tx = threadIdx.x, tyi = threadIdx.y;
  const int x0 = bx * 128 + 2 * tx;
  const int j = by * g.ty + tyi;
  const int z0 = bz * g.zb;
  const int z1 = min(g.nz, z0 + g.zb);
  const bool rowin = j < g.ny;
  // the pair's red node sits at x0 + ((x0 + j + z) & 1); its black node at the other
  auto xr = [&](int z) { return x0 + ((x0 + j + z) & 1); };
  auto xb = [&](int z) { return x0 + 1 - ((x0 + j + z) & 1); };
  auto in = [&](int x) { return rowin && x < g.nx; };
  // red value of this plane's red node, and of the red node below this plane's black node
  double2 rcur = czero(), rbelow = czero();
  if (z0 < z1) {
    if (in(xr(z0))) rcur = red_at<S, DIM>(g, sc, code, uin, f, xr(z0), j, z0, omega);
    if (DIM == 3 && z0 > 0 && in(xb(z0))) rbelow = red_at<S, DIM>(g, sc, code, uin, f, xb(z0), j, z0 - 1, omega);
  }
  for (int z = z0; z < z1; ++z) {
    const int r_x = xr(z), b_x = xb(z);
    // the black node's own inputs, issued first
    const bool bin = in(b_x);
    const size_t pb = (size_t)b_x + (size_t)g.nx * ((size_t)j + (size_t)g.ny * z);
    unsigned cdb = 0;
    double2 ub = czero(), sb = czero(), fb = czero();
    if (bin) {
      cdb = code[pb];
      ub = ldc(uin, pb);
      sb = ldc(sc, pb);
      fb = ldc(f, pb);
    }
    // red of the column above the black node: next plane's red node of this pair
    double2 rabove = czero();
    if (DIM == 3 && z + 1 < g.nz && in(b_x)) rabove = red_at<S, DIM>(g, sc, code, uin, f, b_x, j, z + 1, omega);
    // x neighbours of the black node: its own pair's red node and the adjacent lane's
    const bool red_left = r_x < b_x;  // red at x0, black at x0 + 1: the right neighbour is lane tx + 1's red
    const double2 nb = make_double2(__shfl(rcur.x, red_left ? (tx + 1) & 63 : (tx + 63) & 63, 64),
                                    __shfl(rcur.y, red_left ? (tx + 1) & 63 : (tx + 63) & 63, 64));
    double2 xo = nb;  // the red node on the far side of the black node
    if (red_left && tx == 63 && in(b_x + 1)) xo = red_at<S, DIM>(g, sc, code, uin, f, b_x + 1, j, z, omega);
    if (!red_left && tx == 0 && b_x > 0 && rowin) xo = red_at<S, DIM>(g, sc, code, uin, f, b_x - 1, j, z, omega);
    // y neighbours (same x as the black node) through LDS; the tile's outer rows recomputed
    red[tyi][r_x - bx * 128] = rcur;
    double2 ym = czero(), yp = czero();
    if (tyi == 0 && j > 0 && in(b_x)) ym = red_at<S, DIM>(g, sc, code, uin, f, b_x, j - 1, z, omega);
    if (tyi == g.ty - 1 && j + 1 < g.ny && in(b_x)) yp = red_at<S, DIM>(g, sc, code, uin, f, b_x, j + 1, z, omega);
    __syncthreads();
    if (tyi > 0) ym = red[tyi - 1][b_x - bx * 128];
    if (tyi < g.ty - 1) yp = red[tyi + 1][b_x - bx * 128];
    if (in(r_x)) {
      const size_t pr = (size_t)r_x + (size_t)g.nx * ((size_t)j + (size_t)g.ny * z);
      stc_out(uout, pr, rcur, g.nt);
    }
    if (bin) {
      const double2 a = red_left ? rcur : xo;   // x - 1
      const double2 b = red_left ? xo : rcur;   // x + 1
      const double2 out = relax_upd<S>(g, cdb, ub, a, b, ym, yp, rbelow, rabove, sb, fb, omega, DIM == 3);
      stc_out(uout, pb, out, g.nt);
    }
    __syncthreads();
    // next plane: this plane's red node is below the next black node (same x), and
    // the red node above this black node is the next plane's red node
    rbelow = rcur;
    rcur = rabove;
  }
}

// ---- red-black sweep through an LDS ring of planes (3D) -------------------------
// A workgroup owns a 64 x 8 column tile and marches over zb planes.  Each plane
// of uin is staged once in LDS with a two-node rim (68 x 12 values); a ring of
// six staged planes is kept.  In step z the red half-sweep of plane z + 1 runs
// on the tile and a one-node rim (the rim's red values are the neighbouring
// tile's, recomputed here from uin, so no other workgroup's output is read) and
// overwrites the red positions of the staged plane; then the black half-sweep
// of plane z reads its six red neighbours (planes z - 1, z, z + 1) and its own
// old value from LDS.  Black positions in LDS always keep their uin values, which
// is what the red updates read.  Plane z + 4 is loaded into registers one step
// ahead and the node data (code byte, s, f) of the next step's updates as well;
// one barrier per step.  Stores go through the caches: a colour's stores fill
// every other 16-byte slot of a line, and the other colour's stores of the same
// line follow a step later, so they merge in L2 (non-temporal stores of these
// half lines cost 8% at 256^3 and 13% at 384^3).  Every global access is a buffer load or store whose
// offset is pushed past the end of the buffer where the node is absent (loads
// give 0, stores are dropped), so a step issues the same memory operations on
// every path and waiting for the prefetched data never waits for the step's
// stores.  Red values are rounded to the storage precision before the black
// updates read them, as if the two colours were separate passes through
// memory; the per-node arithmetic is relax_upd's.  Buffers must be under 2 GiB.
constexpr int RB_TX = 64, RB_TY = 8, RB_LX = RB_TX + 4, RB_LY = RB_TY + 4, RB_PL = RB_LX * RB_LY, RB_NS = 6;
constexpr int RB_RROW = (RB_TX + 2) / 2, RB_NRED = RB_RROW * (RB_TY + 2);  // red nodes of the tile and its rim (330)
// 384 threads: one red update per thread and step (330 on the tile and its
// rim), one black update on the first 256 (the tile's 256 black nodes), the
// staged plane three positions per thread
constexpr int RB_NT = 384, RB_NB = RB_TX * RB_TY / 2;
constexpr int RB_QP = (RB_PL + RB_NT - 1) / RB_NT;
static_assert(RB_NB <= RB_NT && RB_NRED <= RB_NT, "ring tile sizes");

// A node's data for one relaxation update: the aligned 32-bit word that holds
// its code byte (a word, not the byte, so that a value carried into the next
// loop iteration needs no conversion, which would make the step wait for its
// own prefetches), s and f.  Code buffers are padded to a multiple of 4 bytes.
struct NodeIn {
  unsigned cw;
  double2 s, f;
};

template <typename S, int DEPTH>
__global__ __launch_bounds__(RB_NT) void k_rbgs_ring(StencilGeom g, int zb, const cplx_t<S>* __restrict__ sc,
                                                   const uint8_t* __restrict__ code,
                                                   const cplx_t<S>* __restrict__ uin, const cplx_t<S>* __restrict__ f,
                                                   cplx_t<S>* __restrict__ uout, double omega) {
  using C = cplx_t<S>;
  __shared__ double2 ring[RB_NS][RB_PL];
  const unsigned lb = xcd_remap(blockIdx.x, gridDim.x);
  const unsigned nbx = (g.nx + RB_TX - 1) / RB_TX, nby = (g.ny + RB_TY - 1) / RB_TY;
  const int bx = lb % nbx, by = (lb / nbx) % nby, bz = lb / (nbx * nby);
  const int gx0 = bx * RB_TX - 2, gy0 = by * RB_TY - 2;  // global (x, y) of LDS position (0, 0)
  const int z0 = bz * zb, z1 = min(g.nz, z0 + zb);
  const int t = threadIdx.x;
  const unsigned nxy = (unsigned)g.nx * g.ny, nn = nxy * g.nz;
  constexpr unsigned ESZ = sizeof(C), ABSENT = RB_OOB / ESZ;  // ABSENT >= nn, as ESZ nn < 2^31
  // A plane: its first node and a mask of the fields' sizes.  For one that is not
  // there or not to be stored both are 0: the fields are empty (loads give 0,
  // stores are dropped), and the scalar part of the address stays below the
  // buffer's size.  The mask goes through readfirstlane, so that a step has no
  // branches on it (they made it wait for its own prefetches).
  struct Plane {
    unsigned ok, n0;
  };
  auto plane = [&](int k, bool on = true) -> Plane {
    const unsigned ok = __builtin_amdgcn_readfirstlane(on && k >= 0 && k < g.nz ? ~0u : 0u);
    return {ok, ok & ((unsigned)k * nxy)};
  };
  auto slot = [](int k) { return (k + RB_NS) % RB_NS; };  // k >= -RB_NS
  // LDS position e's node within its plane
  auto node = [&](int e) -> unsigned {
    const int gx = gx0 + e % RB_LX, gy = gy0 + e / RB_LX;
    return gx >= 0 && gx < g.nx && gy >= 0 && gy < g.ny ? (unsigned)(gx + g.nx * gy) : ABSENT;
  };
  // Everything about a thread's nodes but their plane is formed once: the
  // staged positions' offsets, and for planes of either parity its red and its
  // black node's LDS position, node within the plane and store offset.  Formed
  // anew each step, the addresses were a third of a step's instructions (157 x
  // 142 x 131 in fp32: 70 -> 63 us a sweep).
  unsigned pv[RB_QP];
#pragma unroll
  for (int q = 0; q < RB_QP; ++q) pv[q] = t + RB_NT * q < RB_PL ? node(t + RB_NT * q) * ESZ : RB_OOB;
  const bool bact = t < RB_NB;  // a black node of the tile (32 per row, 8 rows)
  int re[2], be[2];
  unsigned rv[2], bv[2], ro[2];
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    const int r = t < RB_NRED ? t : RB_NRED - 1;
    const int ly = 1 + r / RB_RROW, lx = 1 + ((gx0 + 1 + gy0 + ly + k) & 1) + 2 * (r % RB_RROW);
    re[k] = ly * RB_LX + lx;
    rv[k] = t < RB_NRED ? node(re[k]) : ABSENT;
    const bool tile = lx >= 2 && lx < RB_TX + 2 && ly >= 2 && ly < RB_TY + 2;
    ro[k] = tile ? rv[k] * ESZ : RB_OOB;  // the rim's values are the neighbouring tile's to store
    const int tb = bact ? t : t - RB_NB;
    const int my = 2 + tb / (RB_TX / 2), mx = 3 - ((gx0 + gy0 + my + k) & 1) + 2 * (tb % (RB_TX / 2));
    be[k] = my * RB_LX + mx;
    bv[k] = bact ? node(be[k]) : ABSENT;
  }
  // staged plane k: thread t holds LDS positions t + RB_NT q (zero where there is no node)
  auto load_plane = [&](int k, double2 (&pre)[RB_QP]) {
    const Plane l = plane(k);
    const __amdgpu_buffer_rsrc_t r_u = rb_rsrc(uin, nn * ESZ & l.ok);
#pragma unroll
    for (int q = 0; q < RB_QP; ++q) pre[q] = rb_ld(r_u, pv[q], l.n0 * ESZ, (const C*)nullptr);
  };
  auto store_plane = [&](int k, const double2 (&pre)[RB_QP]) {
    double2* P = ring[slot(k)];
#pragma unroll
    for (int q = 0; q < RB_QP; ++q)
      if (t + RB_NT * q < RB_PL) P[t + RB_NT * q] = pre[q];
  };
  auto load_node = [&](unsigned v, int k, NodeIn& in) {
    const Plane l = plane(k);
    in.cw = __builtin_amdgcn_raw_buffer_load_b32(rb_rsrc(code, (nn + 3) & ~3u & l.ok), (v + l.n0) & ~3u, 0, 0);
    in.s = rb_ld(rb_rsrc(sc, nn * ESZ & l.ok), v * ESZ, l.n0 * ESZ, (const C*)nullptr);
    in.f = rb_ld(rb_rsrc(f, nn * ESZ & l.ok), v * ESZ, l.n0 * ESZ, (const C*)nullptr);
  };
  // the code byte of node v of plane k in its word
  auto code_of = [&](unsigned cw, unsigned v, int k) { return __builtin_amdgcn_ubfe(cw, 8 * ((v + plane(k).n0) & 3), 8); };
  // node data of a step's red update (plane kr) and black update (plane kb), of parities pr and pb
  auto load_next = [&](int kr, int pr, int kb, int pb, NodeIn& rn, NodeIn& bn) {
    load_node(rv[pr], kr, rn);
    load_node(bv[pb], kb, bn);
  };
  // red half-sweep of plane k (parity pk); the tile's values go to uout when `own`
  auto red = [&](int k, int pk, const NodeIn& in, bool own) {
    double2* P = ring[slot(k)];
    const int e = re[pk];
    const double2 v = rnd_store<S>(relax_upd<S>(g, code_of(in.cw, rv[pk], k), P[e], P[e - 1], P[e + 1], P[e - RB_LX],
                                                P[e + RB_LX], ring[slot(k - 1)][e], ring[slot(k + 1)][e], in.s, in.f,
                                                omega, true));
    if (rv[pk] != ABSENT) P[e] = v;  // a plane that is not there holds no neighbour of a node's
    const Plane l = plane(k, own);
    rb_st_cached(rb_rsrc(uout, nn * ESZ & l.ok), ro[pk], l.n0 * ESZ, v, (C*)nullptr);
  };
  // prologue: planes z0 - 2 .. z0 + 2 staged, plane z0 + 3 in flight, red of z0 - 1 and z0
  // Prefetch depth DEPTH: step z reads the register set loaded DEPTH - 1 steps
  // earlier (plane z + 3, node data of its updates) and loads the set of step
  // z + DEPTH - 1 into the set step z - 1 used.  The loop is unrolled by DEPTH so
  // that every set keeps its registers (a set carried into differently named
  // registers at the loop's back-edge would make each step wait for its own
  // loads).  The kernel runs with DEPTH = 2; depths 3 and 4 measured no faster.
  struct Pre {
    double2 pl[RB_QP];
    NodeIn rn, bn;
  };
  Pre S_[DEPTH];
  NodeIn r0, r1;
  // march(P): z0 has parity P, so that a step's parities are constants (the
  // loop is unrolled by an even DEPTH)
  static_assert(DEPTH % 2 == 0, "a step's parity follows its place in the unrolled loop");
  auto march = [&](auto par) {
    constexpr int P0 = decltype(par)::value;
    for (int k = z0 - 2; k <= z0 + 2; ++k) {
      load_plane(k, S_[0].pl);
      store_plane(k, S_[0].pl);
    }
    load_node(rv[1 - P0], z0 - 1, r0);
    load_node(rv[P0], z0, r1);
#pragma unroll
    for (int j = 0; j < DEPTH - 1; ++j) {
      load_plane(z0 + 3 + j, S_[j].pl);
      load_next(z0 + 1 + j, (P0 + 1 + j) & 1, z0 + j, (P0 + j) & 1, S_[j].rn, S_[j].bn);
    }
    __syncthreads();
    red(z0 - 1, 1 - P0, r0, false);
    red(z0, P0, r1, true);
    auto step = [&](int z, int pz, const Pre& cur, Pre& nxt) {
      store_plane(z + 3, cur.pl);  // its slot last held plane z - 3
      load_plane(z + DEPTH + 2, nxt.pl);
      load_next(z + DEPTH, pz, z + DEPTH - 1, 1 - pz, nxt.rn, nxt.bn);
      red(z + 1, 1 - pz, cur.rn, z + 1 < z1);
      __syncthreads();
      // black half-sweep of plane z on the tile (wavefronts of the first 256 threads)
      if (bact) {
        const int e = be[pz];
        const double2* P = ring[slot(z)];
        const double2 v = relax_upd<S>(g, code_of(cur.bn.cw, bv[pz], z), P[e], P[e - 1], P[e + 1], P[e - RB_LX],
                                       P[e + RB_LX], ring[slot(z - 1)][e], ring[slot(z + 1)][e], cur.bn.s, cur.bn.f,
                                       omega, true);
        const Plane l = plane(z, z < z1);
        rb_st_cached(rb_rsrc(uout, nn * ESZ & l.ok), bv[pz] * ESZ, l.n0 * ESZ, v, (C*)nullptr);
      }
    };
    // the march is rounded up to a multiple of DEPTH steps: the steps past z1
    // store nothing (no branches around them, so the register sets stay put)
    for (int z = z0; z < z1; z += DEPTH) {
#pragma unroll
      for (int i = 0; i < DEPTH; ++i) step(z + i, (P0 + i) & 1, S_[i], S_[(i + DEPTH - 1) % DEPTH]);
    }
  };
  if (z0 & 1) march(std::integral_constant<int, 1>{});
  else march(std::integral_constant<int, 0>{});
}

template <typename S>
void jacobi2_from_zero(const StencilGeom& g, const void* sc, const uint8_t* code, const void* f, void* z, double omega,
                       hipStream_t st, const double* fscale, void* fout) {
  using C = cplx_t<S>;
  const int nb = stencil_blocks(g);
  const double n = (double)g.nx * g.ny * g.nz, esz = 2.0 * sizeof(S);
  kprof_begin(KP_STENCIL, st);
  if (g.dim == 3 && g.rows == 2)
    hipLaunchKernelGGL((k_jacobi2z<S, 3, 2>), dim3(nb), dim3(64, g.ty), 0, st, g, (const C*)sc, code, (const C*)f,
                       (C*)z, omega, fscale, (C*)fout);
  else if (g.dim == 3)
    hipLaunchKernelGGL((k_jacobi2z<S, 3, 1>), dim3(nb), dim3(64, g.ty), 0, st, g, (const C*)sc, code, (const C*)f,
                       (C*)z, omega, fscale, (C*)fout);
  else
    hipLaunchKernelGGL((k_jacobi2z<S, 2, 1>), dim3(nb), dim3(64, g.ty), 0, st, g, (const C*)sc, code, (const C*)f,
                       (C*)z, omega, fscale, (C*)fout);
  kprof_end(KP_STENCIL, n * ((fout ? 4 : 3) * esz + 1), st);
}

// z = omega D^{-1} f: a Jacobi sweep started from z = 0 (no stencil needed).
template <typename S>
__global__ __launch_bounds__(256) void k_jacobi0(size_t n, double dsum, const cplx_t<S>* __restrict__ sc,
                                                 const uint8_t* __restrict__ mask,
                                                 const cplx_t<S>* __restrict__ f, cplx_t<S>* __restrict__ z,
                                                 double omega) {
  for (size_t p = blockIdx.x * (size_t)blockDim.x + threadIdx.x; p < n; p += (size_t)gridDim.x * blockDim.x) {
    const double2 r = ldc(f, p);
    double2 d = make_double2(1.0, 0.0);
    if (!mask[p]) {
      const double2 sp = ldc(sc, p);
      d = make_double2(dsum - sp.x, -sp.y);
    }
    const double2 q = ddiv(r, d);
    stc(z, p, make_double2(omega * q.x, omega * q.y));
  }
}

// s = ksq (1 + i alpha), stored in the op's precision.
template <typename S>
__global__ void k_build_s(size_t n, const double* __restrict__ ksq, const double* __restrict__ alpha,
                          cplx_t<S>* __restrict__ sc) {
  for (size_t p = blockIdx.x * (size_t)blockDim.x + threadIdx.x; p < n; p += (size_t)gridDim.x * blockDim.x)
    stc(sc, p, make_double2(ksq[p], ksq[p] * alpha[p]));
}


StencilGeom make_geom(int dim, const int n[3], int zb) {
  StencilGeom g;
  g.nx = n[0];
  g.ny = n[1];
  g.nz = dim == 3 ? n[2] : 1;
  g.dim = dim;
  g.rb = 0;
  g.dsum = 0.0;
  for (int a = 0; a < 3; ++a) g.ih2[a] = 0.0;
  for (int a = 0; a < dim; ++a) {
    const double h = 1.0 / (n[a] + 1);
    g.ih2[a] = 1.0 / (h * h);
    g.dsum += 2.0 * g.ih2[a];
  }
  // taller tiles (fewer y-halo re-reads) on large grids; 64 x 4 keeps enough
  // workgroups on small ones
  const size_t nn = (size_t)g.nx * g.ny * g.nz;
  g.ty = (g.ny >= 128 && nn >= ((size_t)1 << 22)) ? 8 : 4;
  // two rows per thread on large 3D grids (64 x 16 tiles: fewer re-read halo
  // rows; 5.8 against 4.9 TB/s for y = A x at 256^3); small grids keep one row
  // per thread for the block count
  g.rows = (dim == 3 && g.ty == 8) ? 2 : 1;
  g.nt = nn >= ((size_t)1 << 23);
  if (zb <= 0) {
    // enough blocks to fill 256 CUs several times over, long z-marches otherwise
    const long nxy = (long)((g.nx + 63) / 64) * ((g.ny + g.ty * g.rows - 1) / (g.ty * g.rows));
    long target = 2048;
    zb = (int)((nxy * g.nz) / target);
    if (zb < 1) zb = 1;
    if (zb > 16) zb = 16;
  }
  g.zb = dim == 3 ? zb : 1;
  return g;
}

int stencil_nblocks(const StencilGeom& g) { return stencil_blocks(g); }

void build_codes(const StencilGeom& g, const uint8_t* mask, uint8_t* code, hipStream_t st) {
  size_t n = (size_t)g.nx * g.ny * g.nz;
  size_t nb = (n + 255) / 256;
  if (nb > 8192) nb = 8192;
  hipLaunchKernelGGL(k_build_codes, dim3((unsigned)nb), dim3(256), 0, st, g.dim, g.nx, g.ny, g.nz, mask, code);
}

template <typename S, int MODE>
static void launch_mode(const StencilGeom& g, const void* sc, const uint8_t* code, const void* x, const void* f,
                        void* y, double omega, int color, double* part, hipStream_t st) {
  using C = cplx_t<S>;
  dim3 blk(64, g.ty);
  const int nb = stencil_blocks(g);
  const double n = (double)g.nx * g.ny * g.nz, esz = 2.0 * sizeof(S);
  // algorithmic bytes: x, s, the code byte, y (+ f); a red-black colour pass is half a sweep
  const double bytes = MODE == ST_APPLY ? n * (3 * esz + 1) : MODE == ST_RBGS ? n * (4 * esz + 1) / 2 : n * (4 * esz + 1);
  kprof_begin(KP_STENCIL, st);
  if (g.dim == 3 && g.rows == 2)
    hipLaunchKernelGGL((k_stencil<S, 3, MODE, 2>), dim3(nb), blk, 0, st, g, (const C*)sc, code, (const C*)x,
                       (const C*)f, (C*)y, omega, color, part);
  else if (g.dim == 3)
    hipLaunchKernelGGL((k_stencil<S, 3, MODE, 1>), dim3(nb), blk, 0, st, g, (const C*)sc, code, (const C*)x,
                       (const C*)f, (C*)y, omega, color, part);
  else
    hipLaunchKernelGGL((k_stencil<S, 2, MODE, 1>), dim3(nb), blk, 0, st, g, (const C*)sc, code, (const C*)x,
                       (const C*)f, (C*)y, omega, color, part);
  kprof_end(KP_STENCIL, bytes, st);
}

template <typename S>
void stencil_apply(const StencilGeom& g, const void* sc, const uint8_t* code, const void* x, void* y,
                   hipStream_t st) {
  launch_mode<S, ST_APPLY>(g, sc, code, x, nullptr, y, 0.0, 0, nullptr, st);
}
template <typename S>
void stencil_resid(const StencilGeom& g, const void* sc, const uint8_t* code, const void* f, const void* u,
                   void* r, double* part, hipStream_t st) {
  launch_mode<S, ST_RESID>(g, sc, code, u, f, r, 0.0, 0, part, st);
}
template <typename S>
void stencil_jacobi(const StencilGeom& g, const void* sc, const uint8_t* code, const void* f, const void* u,
                    void* unew, double omega, hipStream_t st) {
  launch_mode<S, ST_JACOBI>(g, sc, code, u, f, unew, omega, 0, nullptr, st);
}
template <typename S>
void stencil_rbgs_fused(const StencilGeom& g0, const void* sc, const uint8_t* code, const void* f, const void* uin,
                        void* uout, double omega, hipStream_t st) {
  using C = cplx_t<S>;
  // 128 x 8 tiles: the recomputed rim rows are a quarter of the tile's rows
  StencilGeom g = g0;
  g.ty = g.ny >= 8 ? 8 : g0.ty;
  const int nb = ((g.nx + 127) / 128) * ((g.ny + g.ty - 1) / g.ty) * ((g.nz + g.zb - 1) / g.zb);
  const double n = (double)g.nx * g.ny * g.nz, esz = 2.0 * sizeof(S);
  kprof_begin(KP_STENCIL, st);
  // the ring kernel addresses each buffer with 32-bit offsets (fields under 2 GiB)
  const bool small = n * esz < 2147483648.0;
  const bool ring = g.dim == 3 && (g.rb == 1 || (g.rb == 0 && small));
  if (ring) {
    // planes per workgroup: the march length (2 .. 64) with the fewest steps,
    // counting a march's prologue as three and rounds of the 512 workgroups that run
    // at once (two per CU, by their LDS).  Measured in us a sweep: 157 x 142 x 131 in
    // fp32 15 planes (one round) 46, 6 planes (three rounds) 57; fp64 200 x 180 x 160
    // 32 planes 104, 15 planes 114; 320^3 64 planes 521, 32 planes 531; 352^3 733 and
    // 765; 384^3 55 planes 890, 64 planes 903, 32 planes 943.  Where one round does it
    // all, a length from 32 on within 5% (256^3 32 planes 260, 64 planes 282, 40-55
    // 283-303).  From five rounds of 64-plane marches on HBM is the bound, a last
    // round that is not full costs less than more prologues, and 64 planes are best:
    // 448^3 64 planes 1476, 32-56 planes 1544-1577; 500^3 2064 and 2111-2139; fp32
    // 512^3 1233 and 1343.
    const long tiles = (long)((g.nx + RB_TX - 1) / RB_TX) * ((g.ny + RB_TY - 1) / RB_TY);
    auto steps = [&](int c) { return (tiles * ((g.nz + c - 1) / c) + 511) / 512 * (c + 3); };
    int zb = 2;
    for (int c = 3; c <= 64; ++c)
      if (steps(c) < steps(zb)) zb = c;
    if (steps(zb) == zb + 3)
      for (int c = 32; c < zb; ++c)
        if (20 * steps(c) <= 21 * steps(zb)) zb = c;
    if (tiles * g.nz >= 64L * 2560) zb = 64;
    const long nbr = tiles * ((g.nz + zb - 1) / zb);
    hipLaunchKernelGGL((k_rbgs_ring<S, 2>), dim3((unsigned)nbr), dim3(RB_NT), 0, st, g, zb, (const C*)sc, code,
                       (const C*)uin, (const C*)f, (C*)uout, omega);
  } else if (g.dim == 3)
    hipLaunchKernelGGL((k_rbgs_fused<S, 3>), dim3(nb), dim3(64, g.ty), 0, st, g, (const C*)sc, code, (const C*)uin,
                       (const C*)f, (C*)uout, omega);
  else
    hipLaunchKernelGGL((k_rbgs_fused<S, 2>), dim3(nb), dim3(64, g.ty), 0, st, g, (const C*)sc, code, (const C*)uin,
                       (const C*)f, (C*)uout, omega);
  kprof_end(KP_STENCIL, n * (4 * esz + 1), st);
}
template <typename S>
void jacobi_from_zero(size_t n, double dsum, const void* sc, const uint8_t* mask, const void* f, void* z,
                      double omega, hipStream_t st) {
  using C = cplx_t<S>;
  int nb = (int)((n + 255) / 256);
  if (nb > 8192) nb = 8192;
  hipLaunchKernelGGL((k_jacobi0<S>), dim3(nb), dim3(256), 0, st, n, dsum, (const C*)sc, mask, (const C*)f, (C*)z,
                     omega);
}
template <typename S>
void build_s(size_t n, const double* ksq, const double* alpha, void* sc, hipStream_t st) {
  int nb = (int)((n + 255) / 256);
  if (nb > 8192) nb = 8192;
  hipLaunchKernelGGL((k_build_s<S>), dim3(nb), dim3(256), 0, st, n, ksq, alpha, (cplx_t<S>*)sc);
}

#define HELM_INST(S)                                                                                        \
  template void stencil_apply<S>(const StencilGeom&, const void*, const uint8_t*, const void*, void*,        \
                                 hipStream_t);                                                              \
  template void stencil_resid<S>(const StencilGeom&, const void*, const uint8_t*, const void*, const void*,  \
                                 void*, double*, hipStream_t);                                              \
  template void stencil_jacobi<S>(const StencilGeom&, const void*, const uint8_t*, const void*, const void*, \
                                  void*, double, hipStream_t);                                              \
  template void stencil_rbgs_fused<S>(const StencilGeom&, const void*, const uint8_t*, const void*, const void*, \
                                      void*, double, hipStream_t);                                          \
  template void jacobi_from_zero<S>(size_t, double, const void*, const uint8_t*, const void*, void*, double,  \
                                    hipStream_t);                                                           \
  template void jacobi2_from_zero<S>(const StencilGeom&, const void*, const uint8_t*, const void*, void*,     \
                                     double, hipStream_t, const double*, void*);                            \
  template void build_s<S>(size_t, const double*, const double*, void*, hipStream_t);
HELM_INST(double)
HELM_INST(float)
#undef HELM_INST

}  // namespace helm
