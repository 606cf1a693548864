// Several damped Jacobi sweeps of eq. 2 per launch (§3.1.1).
//
// A sweep alone reads u, f, s and the code byte and writes u: 65 bytes a node
// (complex128) for about 40 fp64 instructions, so large grids are bound by
// HBM and small ones by the launch (3.8 us for 64 x 64 nodes).  Sweeps taken
// together on a tile with a rim (one node more on each side per sweep, its
// values recomputed by the tile that needs them, from the launch's input) cost
// one read and one write of the field, and one launch.  Every sweep's values
// are rounded to the storage precision, and the per-node arithmetic is
// relax_upd's, so the result is that of single sweeps, bit for bit.
#include "common.h"
#include "internal.h"
#include "prof.h"
#include "stencil_dev.h"


namespace helm {

// ---- 2D: several sweeps, the tile in LDS -------------------------------------------
// A workgroup holds a 32 x 32 region (512 threads, two nodes each: f, s, the
// code and the reciprocal diagonal stay in registers over the sweeps, u
// ping-pongs through LDS) and stores the part that t sweeps leave valid:
// 32 - 2 t nodes on an axis, all of them on an axis of at most 32 nodes, where
// the region needs no rim.  Eight sweeps leave a 16 x 16 tile of the 32 x 32:
// four times the arithmetic, in a sixth of the launches (25 sweeps: 96 -> 27 us
// at 64 x 64); five leave 22 x 22.  Where the tiles do not all run at once the
// arithmetic counts (complex64 at 2000 x 2000, a sweep: 33 us by eights, 19 by
// fours, 25 alone).
constexpr int JT = 32, JT_FEW = 512, JT_NT = 512, JT_N = JT * JT / JT_NT, JT_LD = JT + 2;

template <typename S>
__global__ __launch_bounds__(JT_NT) void k_jacobi_tile(StencilGeom g, int sweeps, int tx, int ty, int nbx,
                                                       const cplx_t<S>* __restrict__ sc,
                                                       const uint8_t* __restrict__ code, const cplx_t<S>* uin,
                                                       const cplx_t<S>* __restrict__ f, cplx_t<S>* uout,
                                                       double omega) {
  __shared__ cplx_t<S> buf[2][JT_LD * JT_LD];
  const int lx = threadIdx.x, ly0 = threadIdx.y, t = lx + JT * ly0;
  const int bx = blockIdx.x % nbx, by = blockIdx.x / nbx;
  // an axis covered by one region has no rim
  const int rx = tx == JT ? 0 : sweeps, ry = ty == JT ? 0 : sweeps;
  const int x = bx * tx - rx + lx;
  for (int e = t; e < 2 * JT_LD * JT_LD; e += JT_NT) stc(&buf[0][0], e, czero());
  double2 u[JT_N], fp[JT_N], sp[JT_N], d[JT_N];
  double inv[JT_N];
  unsigned cd[JT_N];
  size_t p[JT_N];
  bool in[JT_N], own[JT_N];
#pragma unroll
  for (int q = 0; q < JT_N; ++q) {
    const int ly = ly0 + q * (JT_NT / JT), y = by * ty - ry + ly;
    in[q] = x >= 0 && x < g.nx && y >= 0 && y < g.ny;
    own[q] = in[q] && lx >= rx && lx < rx + tx && ly >= ry && ly < ry + ty;
    p[q] = in[q] ? (size_t)y * g.nx + x : 0;
    cd[q] = in[q] ? code[p[q]] : 0;
    u[q] = in[q] ? ldc(uin, p[q]) : czero();
    fp[q] = in[q] ? ldc(f, p[q]) : czero();
    sp[q] = in[q] ? ldc(sc, p[q]) : czero();
  }
  __syncthreads();
#pragma unroll
  for (int q = 0; q < JT_N; ++q) {
    d[q] = (cd[q] & NB_SELF) ? make_double2(1.0, 0.0) : make_double2(g.dsum - sp[q].x, -sp[q].y);
    inv[q] = 1.0 / (d[q].x * d[q].x + d[q].y * d[q].y);
    stc(buf[0], (ly0 + q * (JT_NT / JT) + 1) * JT_LD + lx + 1, u[q]);
  }
  for (int k = 0; k < sweeps; ++k) {
    __syncthreads();
    const cplx_t<S>* src = buf[k & 1];
    cplx_t<S>* dst = buf[(k + 1) & 1];
#pragma unroll
    for (int q = 0; q < JT_N; ++q) {
      const int e = (ly0 + q * (JT_NT / JT) + 1) * JT_LD + lx + 1;
      const double2 c = u[q];
      const double2 r = csub(fp[q], stencil_row2<S>(g, cd[q], c, ldc(src, e - 1), ldc(src, e + 1),
                                                    ldc(src, e - JT_LD), ldc(src, e + JT_LD), sp[q]));
      const double2 qq = ddiv_inv(r, d[q], inv[q]);
      u[q] = rnd_store<S>(make_double2(c.x + omega * qq.x, c.y + omega * qq.y));
      stc(dst, e, u[q]);
    }
  }
#pragma unroll
  for (int q = 0; q < JT_N; ++q)
    if (own[q]) stc(uout, p[q], u[q]);
}

// ---- 3D: two sweeps in one march --------------------------------------------------
// A workgroup of 64 x 16 threads marches a 64 x 16 column region along z, one
// node of each plane per thread.  Step z forms the first sweep's values v on
// plane z + 1 and the second sweep's on plane z: a column's values at the
// three planes of each sweep stay in its thread's registers, the planes'
// x and y neighbours meet in LDS (u of plane z + 1 and v of plane z,
// double-buffered: one barrier per step), and f, s, the code and the
// reciprocal diagonal of a node are formed once, a step ahead, and kept for the
// second sweep.  The inner 60 x 12 nodes are stored; a march starts two steps
// early.  The vector arithmetic (two sweeps of 1024 nodes for every 720 stored)
// weighs as much as the traffic, so a node is published to its neighbours as 0
// where it is absent to them (masked, or outside the grid) and no neighbour has
// to be selected by its code bit (303 -> 275 us at 256^3 complex128), LDS holds
// fp64 in complex64 too (no conversion per read: 238 -> 225 us), and buffer
// loads (fields under 2 GiB) take a fixed lane offset and the plane's in a
// scalar.  Two sweeps at 256^3: 383 us as single ones (5.7 TB/s of 65 bytes a
// node each), 275 us together (4.0 TB/s of one read and write); complex64 335
// and 225 us.  Loads issued two steps ahead were slower (330 us: register
// copies).
constexpr int JM_X = 64, JM_Y = 16, JM_TX = JM_X - 4, JM_TY = JM_Y - 4, JM_LX = JM_X + 2, JM_PL = JM_LX * (JM_Y + 2);

// relax_upd with absent neighbours already 0 and inv = 1 / |d|^2 given
__device__ __forceinline__ double2 march_diag(const StencilGeom& g, bool self, double2 sp) {
  return self ? make_double2(1.0, 0.0) : make_double2(g.dsum - sp.x, -sp.y);
}
__device__ __forceinline__ double2 march_upd(const StencilGeom& g, bool self, double2 c, double2 a, double2 b, double2 e,
                                             double2 h, double2 q, double2 w, double2 sp, double2 fp, double inv,
                                             double omega) {
  double2 acc;
  acc.x = ((c.x - a.x) + (c.x - b.x)) * g.ih2[0];
  acc.y = ((c.y - a.y) + (c.y - b.y)) * g.ih2[0];
  acc.x = acc.x + ((c.x - e.x) + (c.x - h.x)) * g.ih2[1];
  acc.y = acc.y + ((c.y - e.y) + (c.y - h.y)) * g.ih2[1];
  acc.x = acc.x + ((c.x - q.x) + (c.x - w.x)) * g.ih2[2];
  acc.y = acc.y + ((c.y - q.y) + (c.y - w.y)) * g.ih2[2];
  double2 ax = csub(acc, cmul(sp, c));
  if (self) ax = c;
  const double2 qq = ddiv_inv(csub(fp, ax), march_diag(g, self, sp), inv);
  return make_double2(c.x + omega * qq.x, c.y + omega * qq.y);
}

template <typename S>
__global__ __launch_bounds__(JM_X* JM_Y) void k_jacobi_march2(StencilGeom g, int zb,
                                                              const cplx_t<S>* __restrict__ sc,
                                                              const uint8_t* __restrict__ code,
                                                              const cplx_t<S>* __restrict__ uin,
                                                              const cplx_t<S>* __restrict__ f,
                                                              cplx_t<S>* __restrict__ uout, double omega) {
  using C = cplx_t<S>;
  __shared__ double2 U[2][JM_PL], V[2][JM_PL];
  const unsigned lb = xcd_remap(blockIdx.x, gridDim.x);
  const unsigned nbx = (g.nx + JM_TX - 1) / JM_TX, nby = (g.ny + JM_TY - 1) / JM_TY;
  const int bx = lb % nbx, by = (lb / nbx) % nby, bz = lb / (nbx * nby);
  const int lx = threadIdx.x, ly = threadIdx.y;
  const int x = bx * JM_TX - 2 + lx, y = by * JM_TY - 2 + ly;
  const int z0 = bz * zb, z1 = min(g.nz, z0 + zb);
  const size_t nxy = (size_t)g.nx * g.ny, nn = nxy * g.nz;
  const __amdgpu_buffer_rsrc_t r_u = rb_rsrc(uin, nn * sizeof(C)), r_f = rb_rsrc(f, nn * sizeof(C)),
                               r_s = rb_rsrc(sc, nn * sizeof(C)), r_c = rb_rsrc(code, nn),
                               r_o = rb_rsrc(uout, nn * sizeof(C));
  const bool in = x >= 0 && x < g.nx && y >= 0 && y < g.ny;
  const bool own = in && lx >= 2 && lx < JM_X - 2 && ly >= 2 && ly < JM_Y - 2;
  const unsigned col = in ? (unsigned)y * g.nx + x : 0u;
  const unsigned co = in ? col * (unsigned)sizeof(C) : RB_OOB, cc = in ? col : RB_OOB;
  const unsigned oo = own ? co : RB_OOB;
  const unsigned pb = (unsigned)(nxy * sizeof(C));
  auto has = [&](int k) { return k >= 0 && k < g.nz; };  // uniform
  auto ld = [&](const __amdgpu_buffer_rsrc_t& r, int k) {
    return rb_ld(r, has(k) ? co : RB_OOB, has(k) ? pb * (unsigned)k : 0u, (const C*)nullptr);
  };
  auto ldcd = [&](int k) -> unsigned {
    return __builtin_amdgcn_raw_buffer_load_b8(r_c, has(k) ? cc : RB_OOB, has(k) ? (unsigned)nxy * k : 0u, 0);
  };
  // a node outside the grid counts as masked: 0 to its neighbours
  auto masked = [&](unsigned c, int k) { return !in || !has(k) || (c & NB_SELF); };
  const int e = (ly + 1) * JM_LX + lx + 1;
  // the region's rim: read by edge threads, whose values are not used
  for (int k = ly * JM_X + lx; k < JM_PL; k += JM_X * JM_Y) {
    stc(U[0], k, czero());
    stc(U[1], k, czero());
    stc(V[0], k, czero());
    stc(V[1], k, czero());
  }
  // at step z: u of the node on planes z + 1 (u1) and z + 2 (u2), as published
  // on plane z (q0); v on planes z - 1 (published, m0) and z (v0); node data
  // of planes z (0) and z + 1 (1); whether it is masked on planes z .. z + 2.
  // A step's loads land in the next one.
  struct Pre {
    double2 u, f, s;  // u of plane z + 3, node data of plane z + 2
    unsigned c;       // code of plane z + 3
  };
  auto fetch = [&](Pre& pre, int zz) {
    pre.u = ld(r_u, zz + 3);
    pre.f = ld(r_f, zz + 2);
    pre.s = ld(r_s, zz + 2);
    pre.c = ldcd(zz + 3);
  };
  int z = z0 - 2;
  double2 q0 = ld(r_u, z), u1 = ld(r_u, z + 1), u2 = ld(r_u, z + 2);
  double2 f0 = czero(), s0 = czero(), f1 = ld(r_f, z + 1), s1 = ld(r_s, z + 1);
  unsigned c_0 = ldcd(z), c_1 = ldcd(z + 1), c_2 = ldcd(z + 2);
  Pre pre;
  fetch(pre, z);
  double2 m0 = czero(), v0 = czero();
  double i0 = 1.0;
  if (masked(c_0, z)) q0 = czero();
  bool m_0 = true, m_1 = masked(c_1, z + 1);
  __syncthreads();
  stc(U[0], e, m_1 ? czero() : u1);
  auto step = [&](int zz, int buf) {
    const Pre now = pre;
    fetch(pre, zz + 1);
    const bool m_2 = masked(c_2, zz + 2);
    const double2 d1 = march_diag(g, m_1, s1);
    const double i1 = 1.0 / (d1.x * d1.x + d1.y * d1.y);
    __syncthreads();
    const double2* P = U[buf];
    const double2* R = V[buf];
    const double2 p2 = m_2 ? czero() : u2;  // u of plane z + 2 as its neighbours see it
    const double2 v1 = rnd_store<S>(march_upd(g, m_1, u1, ldc(P, e - 1), ldc(P, e + 1), ldc(P, e - JM_LX),
                                              ldc(P, e + JM_LX), q0, p2, s1, f1, i1, omega));
    const double2 n1 = m_1 ? czero() : v1, n0 = m_0 ? czero() : v0;
    const double2 w = march_upd(g, m_0, v0, ldc(R, e - 1), ldc(R, e + 1), ldc(R, e - JM_LX), ldc(R, e + JM_LX), m0, n1,
                                s0, f0, i0, omega);
    const bool out = zz >= z0 && zz < z1;  // uniform
    rb_st(r_o, out ? oo : RB_OOB, out ? pb * (unsigned)zz : 0u, w, (C*)nullptr);
    stc(U[1 - buf], e, p2);
    stc(V[1 - buf], e, n1);
    q0 = m_1 ? czero() : u1;
    u1 = u2;
    u2 = now.u;
    m0 = n0;
    v0 = v1;
    f0 = f1;
    s0 = s1;
    i0 = i1;
    m_0 = m_1;
    f1 = now.f;
    s1 = now.s;
    m_1 = m_2;
    c_2 = now.c;
  };
  for (; z < z1; z += 2) {  // a step past z1 stores nothing
    step(z, 0);
    step(z + 1, 1);
  }
}

// planes per march: the fewest rounds of the chip's 256 workgroups (one to a
// CU) times the steps of one, two of which only start the march
static int march_planes(long tiles, int nz) {
  int best = nz;
  long cost = -1;
  for (int c = 1; c <= nz; ++c) {
    const int zb = (nz + c - 1) / c;
    const long rounds = (tiles * ((nz + zb - 1) / zb) + 255) / 256;
    const long t = rounds * (zb + 3);
    if (cost < 0 || t < cost) {
      cost = t;
      best = zb;
    }
    if (zb <= 2) break;
  }
  return best;
}

template <typename S>
static void jacobi_march2(const StencilGeom& g, const void* sc, const uint8_t* code, const void* f, const void* u,
                          void* unew, double omega, hipStream_t st) {
  using C = cplx_t<S>;
  const long tiles = (long)((g.nx + JM_TX - 1) / JM_TX) * ((g.ny + JM_TY - 1) / JM_TY);
  const int zb = march_planes(tiles, g.nz);
  const double n = (double)g.nx * g.ny * g.nz, esz = 2.0 * sizeof(S);
  kprof_begin(KP_STENCIL, st);
  hipLaunchKernelGGL((k_jacobi_march2<S>), dim3((unsigned)(tiles * ((g.nz + zb - 1) / zb))), dim3(JM_X, JM_Y), 0, st,
                     g, zb, (const C*)sc, code, (const C*)u, (const C*)f, (C*)unew, omega);
  kprof_end(KP_STENCIL, n * (4 * esz + 1), st);
}

template <typename S>
static void jacobi_tile(const StencilGeom& g, const void* sc, const uint8_t* code, const void* f, const void* u,
                        void* unew, double omega, int sweeps, hipStream_t st) {
  using C = cplx_t<S>;
  const int tx = g.nx <= JT ? JT : JT - 2 * sweeps, ty = g.ny <= JT ? JT : JT - 2 * sweeps;
  const int nbx = (g.nx + tx - 1) / tx, nby = (g.ny + ty - 1) / ty;
  const double n = (double)g.nx * g.ny, esz = 2.0 * sizeof(S);
  kprof_begin(KP_STENCIL, st);
  hipLaunchKernelGGL((k_jacobi_tile<S>), dim3(nbx * nby), dim3(JT, JT_NT / JT), 0, st, g, sweeps, tx, ty, nbx, (const C*)sc,
                     code, (const C*)u, (const C*)f, (C*)unew, omega);
  kprof_end(KP_STENCIL, n * (4 * esz + 1), st);
}

// Whether the paired march is faster than two single sweeps: grids of at least
// 0.8 Mi nodes (64^3: 13.5 us a pair against 9.7 for two sweeps, 80^3: 16 and 17,
// 96^3: 18.4 and 22.5) whose columns fill the 60 x 12 tiles to three quarters
// (128^3 fills 0.69 of them: 39 us against 36 in complex64), and buffer offsets.
template <typename S>
static bool march_pays(const StencilGeom& g) {
  const size_t nxy = (size_t)g.nx * g.ny, n = nxy * g.nz;
  const size_t tiles = (size_t)((g.nx + JM_TX - 1) / JM_TX) * ((g.ny + JM_TY - 1) / JM_TY);
  return g.dim == 3 && n >= 800000 && 4 * nxy >= 3 * tiles * JM_TX * JM_TY && n * 2 * sizeof(S) < ((size_t)1 << 31);
}

template <typename S>
void relax_sweeps(const StencilGeom& g, const void* sc, const uint8_t* code, bool rbgs, double omega, int sweeps,
                  const void* f, void* u, void* tmp, hipStream_t st) {
  const size_t n = (size_t)g.nx * g.ny * g.nz;
  int left = sweeps;
  if (!rbgs && g.dim == 2 && g.nx <= JT && g.ny <= JT) {
    // one workgroup holds the grid: any count in place (0.5 us a sweep), at most 1024 per launch
    for (; left > 0; left -= 1024) jacobi_tile<S>(g, sc, code, f, u, u, omega, left < 1024 ? left : 1024, st);
    return;
  }
  void* a = u;
  void* b = tmp;
  auto swap = [&] {
    void* t = a;
    a = b;
    b = t;
  };
  if (!rbgs && g.dim == 2 && sweeps >= 2) {
    // Up to eight sweeps a launch on grids of at most JT_FEW tiles of 16 x 16, two to
    // a CU (300 x 311: 1.5 us a sweep by fours and by eights), five on larger ones
    // (500 x 500 by fours and by eights: 2.2 and 2.4 us, complex64 2.4 and 2.8; 4096
    // x 4096: 73 and 114); a launch of one sweep is the untiled one (two sweeps at
    // 1000 x 1000: 21 us, 30 as tiles).  An even number of launches, so that the last
    // lands in u.
    const int most = (size_t)((g.nx + 15) / 16) * ((g.ny + 15) / 16) <= JT_FEW ? 8 : 5;
    for (int launches = 2 * ((sweeps - 1) / (2 * most) + 1); launches > 0; --launches, swap()) {
      const int k = (left - 1) / launches + 1;
      if (k > 1) jacobi_tile<S>(g, sc, code, f, a, b, omega, k, st);
      else stencil_jacobi<S>(g, sc, code, f, a, b, omega, st);
      left -= k;
    }
    return;
  }
  // pairs, then single sweeps.  An odd number of passes ends in a copy, which on
  // grids below 4 Mi nodes costs what one pair saves (157 x 142 x 131: 63 us for
  // a pair and the copy, 63 for two sweeps): an even count of sweeps then keeps
  // two of them single.
  int pairs = !rbgs && march_pays<S>(g) ? sweeps / 2 : 0;
  if ((pairs & 1) && sweeps % 2 == 0 && n < ((size_t)1 << 22)) --pairs;
  for (; pairs > 0; --pairs, left -= 2, swap()) jacobi_march2<S>(g, sc, code, f, a, b, omega, st);
  for (; left > 0; --left, swap()) {
    if (rbgs) stencil_rbgs_fused<S>(g, sc, code, f, a, b, omega, st);
    else stencil_jacobi<S>(g, sc, code, f, a, b, omega, st);
  }
  if (a != u) copy_vec<S>(n, a, u, st);
}
template void relax_sweeps<double>(const StencilGeom&, const void*, const uint8_t*, bool, double, int, const void*,
                                   void*, void*, hipStream_t);
template void relax_sweeps<float>(const StencilGeom&, const void*, const uint8_t*, bool, double, int, const void*,
                                  void*, void*, hipStream_t);

}  // namespace helm
