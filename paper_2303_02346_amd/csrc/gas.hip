// The gas step (include/gas.h): incompressible advection-projection on a
// staggered grid (FluidLab section 3.2, after Stam 1999) and its adjoint.
//
// Forward step, three launches plus the pressure solve:
//   k_gas_advect   every grid point of u, v, w and the cells: the velocity
//                  at the point from its stencils, back-trace, trilinear
//                  sample, emitter blend (one launch for the four grids); the
//                  scalars are final then
//   k_gas_div      per cell: divergence of the advected velocity with the
//                  buoyancy of the y-faces added on the fly and the walls
//                  closed; right-hand side of the pressure equation
//   pressure       A psi = div (A: 7-point Neumann Laplacian in cell units;
//                  psi = pressure * dt / h), by default exactly: DCT-II
//                  transforms along z, y and x on the matrix cores (k_axis),
//                  division by the eigenvalue sums, inverse transforms; or
//                  multigrid V-cycles (mg_solve: red-black half-sweeps on
//                  the finest level, tiled full sweeps on the coarser grid
//                  levels, the levels of at most 4096 cells in one workgroup)
//   k_gas_final    u = u* - grad psi on the interior faces, walls zero
// Adjoint step: the projection of the adjoint (the same divergence without
// buoyancy, pressure solve and subtraction; the projector is self-adjoint on
// wall-closed fields), then k_gas_adj_advect, which recomputes the
// back-traces, applies the buoyancy and emitter adjoints and scatters the
// advection adjoint at the back-traced points with float atomics (samples
// merge the corners they share first), and k_gas_adj_ugather, which gathers
// the adjoint of the grid-point velocities over their stencils; the
// emitter's pose partials are reduced per wavefront into 128 FP64
// accumulator copies.
#include <hip/hip_runtime.h>
#include <math.h>
#include <string.h>
#include <algorithm>
#include <type_traits>
#include <new>
#include <vector>

#include "../../include/gas.h"
#include "mpm_internal.h"

namespace mpm {
namespace {

constexpr int MAXK = 4;
constexpr int SLOTS = 128;
constexpr int POSE_PARTIALS = 6;          // c (3), a = R e_y (3)
constexpr int BOTTOM_CELLS = 4096;        // levels this small run inside one workgroup, in LDS
constexpr int BOTTOM_LDS = 4800;          // >= 4096 * 8 / 7
#ifndef GAS_BOTTOM_THREADS
#define GAS_BOTTOM_THREADS 1024
#endif
constexpr int BOTTOM_THREADS = GAS_BOTTOM_THREADS;
constexpr int MAX_LEVELS = 12;
#ifndef GAS_COARSE_SWEEPS
#define GAS_COARSE_SWEEPS 4
#endif
constexpr int COARSE_SWEEPS = GAS_COARSE_SWEEPS;
#ifndef GAS_HALF_LEVELS
#define GAS_HALF_LEVELS 1
#endif
constexpr int HALF_LEVELS = GAS_HALF_LEVELS;   // finest levels smoothed by separate half-sweeps
#ifndef GAS_NU0_PRE
#define GAS_NU0_PRE 2
#endif
#ifndef GAS_NU0_POST
#define GAS_NU0_POST 1
#endif
#ifndef GAS_NU_POST
#define GAS_NU_POST 2
#endif
#ifndef GAS_NU_BOTTOM
#define GAS_NU_BOTTOM 2
#endif
// sweeps before / after the coarse correction on the finest level, after it
// on the coarser grid levels, and before and after it inside the bottom solve
constexpr int NU0_PRE = GAS_NU0_PRE, NU0_POST = GAS_NU0_POST, NU_POST = GAS_NU_POST, NU_BOTTOM = GAS_NU_BOTTOM;
// smoother tiles: TX x TY x TZ cells per workgroup; psi staged with a 2-cell
// halo, f with a 1-cell halo
#ifndef GAS_TILE_X
#define GAS_TILE_X 8
#endif
#ifndef GAS_TILE_Y
#define GAS_TILE_Y 8
#endif
#ifndef GAS_TILE_Z
#define GAS_TILE_Z 8
#endif
constexpr int TX = GAS_TILE_X, TY = GAS_TILE_Y, TZ = GAS_TILE_Z;
constexpr int PX = TX + 4, PY = TY + 4, PZ = TZ + 4;
constexpr int FX = TX + 2, FY = TY + 2, FZ = TZ + 2;

inline size_t al256(size_t x) { return (x + 255) & ~(size_t)255; }
inline unsigned nblk(size_t n, unsigned b) {
  size_t g = (n + b - 1) / b;
  return (unsigned)(g < 65536 * 16 ? g : 65536 * 16);
}

// Workgroups are dispatched round-robin over the 8 XCDs, each with its own
// L2.  The advection reads its neighbours' rows (stencils and samples), so
// its workgroup order is permuted to give every XCD one contiguous eighth of
// the points: workgroup b takes block start(b % 8) + b / 8 of the range (a
// bijection of [0, gridDim.x)).  At 128^3 this cuts the advection's fetched
// bytes by 40% (the kernel's time is set by its VALU issue, not by them).
__device__ inline unsigned xcd_block() {
  const unsigned nb = gridDim.x, b = blockIdx.x, x = b & 7u, per = nb >> 3, rem = nb & 7u;
  return x * per + min(x, rem) + (b >> 3);
}

struct Dims {
  int x, y, z;
  __host__ __device__ size_t cells() const { return (size_t)x * y * z; }
};

struct GP {
  int nx, ny, nz, K;
  float h, inv_h, dt, beta, t_amb;
  float s2inv;          // 1 / (2 sigma^2)
  float kappa, speed;
  float src[MAXK];
  size_t nu, nv, nw, nc;
  uint32_t mz, mz1;     // multipliers of row_of for rows of nz and nz + 1 points
  int big;              // an array of 4 GB or more: samples need 64-bit offsets
  int* err;             // device error word (MPM_ERR_NONFINITE)
};

// Point kernels run one workgroup on 256 U consecutive points of one x plane of
// one grid, so that the grid, the plane and every array's plane are uniform
// over the workgroup: a point costs one multiplication for its row instead of
// three divisions by run-time sizes, and the stencil loads are 32-bit offsets
// from scalar bases.  U points a thread share the uniform part, about 100
// scalar instructions (U = 1, and the planes' number by division: k_gas_final
// 21.8 us at 128^3 against 13.1).  The workgroups go plane by plane (u, v, w,
// cells of a plane in turn), in xcd_block's order.
struct PointGrid {
  uint32_t nb[4], per, mper;   // workgroups of a plane of each grid, of all, and its multiplier for division
  uint32_t blocks;
};
__host__ __device__ inline int plane_points(int q, int ny, int nz) { return q == 1 ? (ny + 1) * nz : (q == 2 ? ny * (nz + 1) : ny * nz); }
inline PointGrid point_grid(const GP& P, int nq, int u) {
  PointGrid G = {};
  for (int q = 0; q < nq; q++) {
    G.nb[q] = ((uint32_t)plane_points(q, P.ny, P.nz) + 256u * u - 1) / (256u * u);
    G.per += G.nb[q];
  }
  G.blocks = G.per * (uint32_t)(P.nx + 1);
  G.mper = (uint32_t)((0x100000000ull + G.per - 1) / G.per);
  return G;
}
struct PlaneBlock {
  int q, i, r0, n;   // grid, plane, first point in the plane, points of the plane (n = 0: past the grid's last plane)
};
template <int U>
__device__ __forceinline__ PlaneBlock plane_block(const GP& P, const PointGrid& G) {
  uint32_t b = xcd_block();
  PlaneBlock o;
  o.i = G.per == 1u ? (int)b : (int)__umulhi(b, G.mper);
  if ((uint32_t)o.i * G.per > b) o.i--;   // (the multiplier rounds up)
  b -= (uint32_t)o.i * G.per;
  o.q = 0;
#pragma unroll
  for (int q = 0; q < 3; q++)
    if (o.q == q && b >= G.nb[q]) { b -= G.nb[q]; o.q = q + 1; }
  o.n = (o.q == 0 || o.i < P.nx) ? plane_points(o.q, P.ny, P.nz) : 0;
  o.r0 = (int)b * 256 * U;
  return o;
}
// row of point r in rows of d values, m = ceil(2^32 / d) (exact for r d < 2^32)
__device__ __forceinline__ int row_of(int r, uint32_t m) { return (int)__umulhi((uint32_t)r, m); }

// grid q: 0 = u (x-faces), 1 = v, 2 = w, 3 = cells
__device__ inline void gdims(const GP& P, int q, int& d0, int& d1, int& d2) {
  d0 = P.nx + (q == 0);
  d1 = P.ny + (q == 1);
  d2 = P.nz + (q == 2);
}
__device__ inline float gorigin(int q, int a) { return (q == a) ? 0.f : 0.5f; }

// trilinear sample of grid q at a point: base node, fractions, clamped axes
struct Lerp {
  int i0, j0, k0;
  float f[3];
  bool cl[3];
};

// The sample of grid q at the back-traced point x - dt U of its point (i, j, k).
// (Here and below the roundings are written out.  A sample's fraction has lost
// the digits of its coordinate, so what the compiler contracts, which differs
// from kernel to kernel, changed the velocities' distance from a 64-bit run by
// a factor of two.)
__device__ __forceinline__ Lerp lerp_setup(const GP& P, int q, int i, int j, int k, const float* U) {
#pragma clang fp contract(off)
  int d[3];
  gdims(P, q, d[0], d[1], d[2]);
  const int n[3] = {i, j, k};
  Lerp L;
  int b[3];
#pragma unroll
  for (int a = 0; a < 3; a++) {
    const float o = gorigin(q, a), no = (float)n[a] + o;
    const float xb = fmaf(no, P.h, -(P.dt * U[a]));
    float g = fmaf(xb, P.inv_h, -o);
    const float hi = (float)(d[a] - 1);
    L.cl[a] = !(g >= 0.f && g <= hi);        // (also NaN)
    g = fminf(fmaxf(g, 0.f), hi);
    const float fl = fminf(floorf(g), hi - 1.f);
    b[a] = (int)fl;
    L.f[a] = g - fl;
  }
  L.i0 = b[0]; L.j0 = b[1]; L.k0 = b[2];
  return L;
}

// flat index in one grid array (every array has fewer than 2^32 values:
// 32-bit arithmetic, widened for the address)
__device__ inline size_t gidx(int i, int j, int k, int d1, int d2) {
  return (size_t)(((uint32_t)i * (uint32_t)d1 + (uint32_t)j) * (uint32_t)d2 + (uint32_t)k);
}

__device__ inline void cell_of(const Dims& D, size_t g, int& i, int& j, int& k) {
  const uint32_t g32 = (uint32_t)g, r = g32 / (uint32_t)D.z;
  k = (int)(g32 - r * (uint32_t)D.z);
  i = (int)(r / (uint32_t)D.y);
  j = (int)(r - (uint32_t)i * (uint32_t)D.y);
}

// d(sample)/d(fraction) per axis
__device__ inline void lerp_grad(const float* c, const Lerp& L, float* g) {
  const float fx = L.f[0], fy = L.f[1], fz = L.f[2];
  g[0] = (1 - fy) * (1 - fz) * (c[4] - c[0]) + (1 - fy) * fz * (c[5] - c[1]) + fy * (1 - fz) * (c[6] - c[2]) +
         fy * fz * (c[7] - c[3]);
  g[1] = (1 - fx) * (1 - fz) * (c[2] - c[0]) + (1 - fx) * fz * (c[3] - c[1]) + fx * (1 - fz) * (c[6] - c[4]) +
         fx * fz * (c[7] - c[5]);
  g[2] = (1 - fx) * (1 - fy) * (c[1] - c[0]) + (1 - fx) * fy * (c[3] - c[2]) + fx * (1 - fy) * (c[5] - c[4]) +
         fx * fy * (c[7] - c[6]);
}

struct VelPtrs {
  const float* u;
  const float* v;
  const float* w;
};

// The velocity at a grid point: the trilinear sample of each component grid
// there reduces to the point's own value on its own grid and to averages of 2
// or 4 neighbours on the others (sample fractions 0 or 1/2, clamped at the walls
// like every sample).  Point (j, k) on plane i of grid Q: the planes' bases are
// uniform, the offsets in a plane 32-bit.
__device__ __forceinline__ float ld32(const float* __restrict__ p, uint32_t off) {
  return *reinterpret_cast<const float*>(reinterpret_cast<const char*>(p) + 4u * off);
}
template <int Q>
__device__ __forceinline__ void plane_velocity(const GP& P, const VelPtrs& vel, int i, int j, int k, float* U) {
  const int ny = P.ny, nz = P.nz;
  const size_t pu = (size_t)ny * nz, pv = (size_t)(ny + 1) * nz, pw = (size_t)ny * (nz + 1);
  const uint32_t z = (uint32_t)nz, o = (uint32_t)(j * nz + k), ow = o + (uint32_t)j;   // rows of nz and of nz + 1
  if (Q == 3) {
    const float *u0 = vel.u + i * pu, *v0 = vel.v + i * pv, *w0 = vel.w + i * pw;
    U[0] = 0.5f * (ld32(u0, o) + ld32(u0 + pu, o));
    U[1] = 0.5f * (ld32(v0, o) + ld32(v0, o + z));
    U[2] = 0.5f * (ld32(w0, ow) + ld32(w0, ow + 1));
  } else if (Q == 0) {
    const int ia = max(i - 1, 0), ib = min(i, P.nx - 1);
    const float *va = vel.v + ia * pv, *vb = vel.v + ib * pv, *wa = vel.w + ia * pw, *wb = vel.w + ib * pw;
    U[0] = ld32(vel.u + i * pu, o);
    U[1] = 0.25f * ((ld32(va, o) + ld32(vb, o)) + (ld32(va, o + z) + ld32(vb, o + z)));
    U[2] = 0.25f * ((ld32(wa, ow) + ld32(wb, ow)) + (ld32(wa, ow + 1) + ld32(wb, ow + 1)));
  } else if (Q == 1) {
    const uint32_t ja = (uint32_t)max(j - 1, 0), jb = (uint32_t)min(j, ny - 1), uk = (uint32_t)k;
    const float *u0 = vel.u + i * pu, *u1 = u0 + pu, *w0 = vel.w + i * pw;
    const uint32_t oa = ja * z + uk, ob = jb * z + uk, wa = oa + ja, wb = ob + jb;
    U[0] = 0.25f * ((ld32(u0, oa) + ld32(u0, ob)) + (ld32(u1, oa) + ld32(u1, ob)));
    U[1] = ld32(vel.v + i * pv, o);
    U[2] = 0.25f * ((ld32(w0, wa) + ld32(w0, wb)) + (ld32(w0, wa + 1) + ld32(w0, wb + 1)));
  } else {
    const uint32_t oa = (uint32_t)(j * nz + max(k - 1, 0)), ob = (uint32_t)(j * nz + min(k, nz - 1));
    const float *u0 = vel.u + i * pu, *u1 = u0 + pu, *v0 = vel.v + i * pv;
    U[0] = 0.25f * ((ld32(u0, oa) + ld32(u0, ob)) + (ld32(u1, oa) + ld32(u1, ob)));
    U[1] = 0.25f * ((ld32(v0, oa) + ld32(v0, ob)) + (ld32(v0, oa + z) + ld32(v0, ob + z)));
    U[2] = ld32(vel.w + i * pw, ow);
  }
}

// the eight corner values as four z pairs (two adjacent values, 4-byte aligned)
struct __attribute__((packed, aligned(4))) ZPair {
  float a, b;
};
__device__ __forceinline__ void lerp_pairs(int big, const float* __restrict__ F, const Lerp& L, uint32_t d1, uint32_t d2,
                                           ZPair* c) {
  const uint32_t b = ((uint32_t)L.i0 * d1 + (uint32_t)L.j0) * d2 + (uint32_t)L.k0, sx = d1 * d2;
  const float* row[4] = {F, F + d2, F + sx, F + (size_t)sx + d2};
  if (big) {
#pragma unroll
    for (int n = 0; n < 4; n++) c[n] = *reinterpret_cast<const ZPair*>(row[n] + b);
  } else {
#pragma unroll
    for (int n = 0; n < 4; n++) c[n] = *reinterpret_cast<const ZPair*>(reinterpret_cast<const char*>(row[n]) + 4u * b);
  }
}
__device__ __forceinline__ float lerp_pairs_eval(const ZPair* c, const Lerp& L) {
#pragma clang fp contract(off)
  const float fx[2] = {1.f - L.f[0], L.f[0]}, fy[2] = {1.f - L.f[1], L.f[1]}, fz[2] = {1.f - L.f[2], L.f[2]};
  float s = 0.f;
#pragma unroll
  for (int n = 0; n < 4; n++) {
    const float w = fx[n >> 1] * fy[n & 1];
    s = fmaf(w * fz[0], c[n].a, s);
    s = fmaf(w * fz[1], c[n].b, s);
  }
  return s;
}

struct Pose {
  float c[3], a[3];   // centre and outflow axis R e_y
};
__device__ inline Pose load_pose(const double* p) {
  Pose o;
#pragma unroll
  for (int k = 0; k < 3; k++) { o.c[k] = (float)p[k]; o.a[k] = (float)p[3 + k * 3 + 1]; }
  return o;
}
// offset d of point (i, j, k) of grid Q from the emitter, and its blend
template <int Q>
__device__ __forceinline__ float emitter_chi(const GP& P, const Pose& E, int i, int j, int k, float* d) {
#pragma clang fp contract(off)
  const int n[3] = {i, j, k};
#pragma unroll
  for (int a = 0; a < 3; a++) {
    const float no = (float)n[a] + gorigin(Q, a);
    d[a] = fmaf(no, P.h, -E.c[a]);
  }
  const float r2 = fmaf(d[2], d[2], fmaf(d[0], d[0], d[1] * d[1]));
  return P.kappa * expf(-r2 * P.s2inv);
}

// ---------------------------------------------------------------------------
// forward
// ---------------------------------------------------------------------------
// One point of grid Q in plane i.  The scalars go straight to the step's output.
template <int Q>
__device__ __forceinline__ void advect_point(const GP& P, const VelPtrs& vel, const float* __restrict__ s,
                                             float* __restrict__ o, const Pose& E, int i, int r) {
  constexpr bool Z1 = Q == 2;
  const uint32_t d1 = (uint32_t)(P.ny + (Q == 1)), d2 = (uint32_t)(P.nz + (Q == 2));
  const int j = row_of(r, Z1 ? P.mz1 : P.mz), k = r - j * (int)d2;
  float d[3], U[3];
  plane_velocity<Q>(P, vel, i, j, k, U);
  const Lerp L = lerp_setup(P, Q, i, j, k, U);
  const size_t g = (size_t)i * d1 * d2;   // (uniform)
  if (Q < 3) {
    ZPair c[4];
    lerp_pairs(P.big, Q == 0 ? vel.u : (Q == 1 ? vel.v : vel.w), L, d1, d2, c);
    const float chi = emitter_chi<Q>(P, E, i, j, k, d);
    const float val = lerp_pairs_eval(c, L);
    (o + g)[(uint32_t)r] = fmaf(chi, fmaf(P.speed, E.a[Q < 3 ? Q : 0], -val), val);
  } else {
    ZPair c[MAXK][4];
#pragma unroll
    for (int kk = 0; kk < MAXK; kk++)
      if (kk < P.K) lerp_pairs(P.big, s + kk * P.nc, L, d1, d2, c[kk]);
    const float chi = emitter_chi<Q>(P, E, i, j, k, d);
    bool fin = true;
#pragma unroll
    for (int kk = 0; kk < MAXK; kk++) {
      if (kk >= P.K) break;
      const float vs = lerp_pairs_eval(c[kk], L), val = fmaf(chi, P.src[kk] - vs, vs);
      fin = fin && isfinite(val);
      (o + kk * P.nc + g)[(uint32_t)r] = val;
    }
    if (!fin) atomicOr(P.err, ERR_NONFINITE);
  }
}

constexpr int ADV_U = 4, DIV_U = 1, FIN_U = 4;
// (bound by VALU issue: the plane-wise points and the loads of whole z pairs
// took it from 70.4 to 42 us at 128^3 with two scalars; the
// arrays it has to read and write take 16)
__global__ __launch_bounds__(256) void k_gas_advect(GP P, VelPtrs vel, const float* __restrict__ s,
                                                    float* __restrict__ u1, float* __restrict__ v1,
                                                    float* __restrict__ w1, float* __restrict__ s1,
                                                    const double* __restrict__ pose, PointGrid G) {
  const PlaneBlock b = plane_block<ADV_U>(P, G);
  const Pose E = load_pose(pose);
  auto points = [&](auto q, float* o) {
#pragma unroll 1
    for (int r = b.r0 + (int)threadIdx.x, u = 0; u < ADV_U && r < b.n; u++, r += 256)
      advect_point<decltype(q)::value>(P, vel, s, o, E, b.i, r);
  };
  if (b.q == 0) points(std::integral_constant<int, 0>{}, u1);
  else if (b.q == 1) points(std::integral_constant<int, 1>{}, v1);
  else if (b.q == 2) points(std::integral_constant<int, 2>{}, w1);
  else points(std::integral_constant<int, 3>{}, s1);
}

// divergence (sum of face differences, walls closed) of (u1, v1, w1), with BUOY
// the buoyancy of the temperature T1 added to the y-faces (the adjoint's
// velocity takes none); psi (the multigrid's first guess) is cleared where it
// is given
template <bool BUOY>
__global__ __launch_bounds__(256) void k_gas_div(GP P, const float* __restrict__ u1, const float* __restrict__ v1,
                                                 const float* __restrict__ w1, const float* __restrict__ T1,
                                                 float* __restrict__ f, float* __restrict__ psi, PointGrid G) {
  const PlaneBlock b = plane_block<DIV_U>(P, G);
  if (b.i >= P.nx) return;
  const int i = b.i;
  const uint32_t z = (uint32_t)P.nz;
  const size_t pu = (size_t)P.ny * P.nz, pv = pu + P.nz, pw = pu + P.ny;
  const float *u0 = u1 + i * pu, *v0 = v1 + i * pv, *w0 = w1 + i * pw, *T0 = BUOY ? T1 + i * pu : nullptr;
  const float bd = P.dt * P.beta;
#pragma unroll
  for (int u = 0; u < DIV_U; u++) {
    const int r = b.r0 + 256 * u + (int)threadIdx.x;
    if (r >= b.n) break;
    const int j = row_of(r, P.mz), k = r - j * P.nz;
    const uint32_t o = (uint32_t)r, ow = o + (uint32_t)j;
    const float ur = (i + 1 < P.nx) ? ld32(u0 + pu, o) : 0.f;
    const float ul = (i > 0) ? ld32(u0, o) : 0.f;
    const float tc = BUOY ? ld32(T0, o) : 0.f;
    float vt = (j + 1 < P.ny) ? ld32(v0, o + z) : 0.f, vb = (j > 0) ? ld32(v0, o) : 0.f;
    if (BUOY) {
      if (j + 1 < P.ny) vt += bd * (0.5f * (tc + ld32(T0, o + z)) - P.t_amb);
      if (j > 0) vb += bd * (0.5f * (ld32(T0, o - z) + tc) - P.t_amb);
    }
    const float wf = (k + 1 < P.nz) ? ld32(w0, ow + 1) : 0.f;
    const float wb = (k > 0) ? ld32(w0, ow) : 0.f;
    (f + i * pu)[o] = (ur - ul) + (vt - vb) + (wf - wb);
    if (psi) (psi + i * pu)[o] = 0.f;
  }
}

// u = u* - grad psi on the interior faces (with BUOY, v with its buoyancy), walls zero
template <bool BUOY>
__global__ __launch_bounds__(256) void k_gas_final(GP P, const float* __restrict__ u1, const float* __restrict__ v1,
                                                   const float* __restrict__ w1, const float* __restrict__ s1,
                                                   const float* __restrict__ psi, float* __restrict__ u,
                                                   float* __restrict__ v, float* __restrict__ w, PointGrid G) {
  const PlaneBlock b = plane_block<FIN_U>(P, G);
  const int i = b.i;
  const uint32_t z = (uint32_t)P.nz;
  const size_t pc = (size_t)P.ny * P.nz, pv = pc + P.nz, pw = pc + P.ny;
  bool fin = true;
  auto points = [&](float* O, auto&& value) {
#pragma unroll
    for (int t = 0; t < FIN_U; t++) {
      const int r = b.r0 + 256 * t + (int)threadIdx.x;
      if (r >= b.n) break;
      const float val = value(r, (uint32_t)r);
      fin = fin && isfinite(val);
      O[(uint32_t)r] = val;
    }
  };
  if (b.q == 0) {
    const bool in = i > 0 && i < P.nx;
    const float *p0 = psi + (in ? i : 1) * pc, *u0 = u1 + i * pc;
    points(u + i * pc, [&](int, uint32_t o) { return in ? ld32(u0, o) - (ld32(p0, o) - ld32(p0 - pc, o)) : 0.f; });
  } else if (b.q == 1) {
    const float *p0 = psi + i * pc, *T0 = BUOY ? s1 + i * pc : nullptr, *v0 = v1 + i * pv;
    points(v + i * pv, [&](int r, uint32_t o) {
      const int j = row_of(r, P.mz);
      if (!(j > 0 && j < P.ny)) return 0.f;
      float val = ld32(v0, o);
      if (BUOY) val += P.dt * P.beta * (0.5f * (ld32(T0, o - z) + ld32(T0, o)) - P.t_amb);
      return val - (ld32(p0, o) - ld32(p0, o - z));
    });
  } else {
    const float *p0 = psi + i * pc, *w0 = w1 + i * pw;
    points(w + i * pw, [&](int r, uint32_t o) {
      const int j = row_of(r, P.mz1), k = r - j * (P.nz + 1);
      if (!(k > 0 && k < P.nz)) return 0.f;
      const uint32_t c = o - (uint32_t)j;
      return ld32(w0, o) - (ld32(p0, c) - ld32(p0, c - 1));
    });
  }
  if (!fin) atomicOr(P.err, ERR_NONFINITE);
}

// ---------------------------------------------------------------------------
// multigrid for A psi = f, A the 7-point Neumann Laplacian in cell units
// (A psi)_c = sum over in-domain neighbours (psi_n - psi_c).  Red-black
// Gauss-Seidel smoothing, residual restriction f_c = (1/2) sum of the 8
// children's residuals (the coarse operator is A again at twice the
// spacing), cell-centred trilinear prolongation.
// ---------------------------------------------------------------------------

// sum of the in-domain neighbours and their number
__device__ inline float nb_sum(const float* psi, const Dims& D, int i, int j, int k, int& cnt) {
  float s = 0.f;
  cnt = 0;
  const size_t c = gidx(i, j, k, D.y, D.z);
  if (i > 0) { s += psi[c - (size_t)D.y * D.z]; cnt++; }
  if (i + 1 < D.x) { s += psi[c + (size_t)D.y * D.z]; cnt++; }
  if (j > 0) { s += psi[c - D.z]; cnt++; }
  if (j + 1 < D.y) { s += psi[c + D.z]; cnt++; }
  if (k > 0) { s += psi[c - 1]; cnt++; }
  if (k + 1 < D.z) { s += psi[c + 1]; cnt++; }
  return s;
}

// 1 / cnt for a neighbour count of 1..6 (a division would cost a long sequence)
__device__ inline float inv_count(int cnt) {
  return cnt == 6 ? (1.f / 6.f) : (cnt == 5 ? 0.2f : (cnt == 4 ? 0.25f : (cnt == 3 ? (1.f / 3.f) : (cnt == 2 ? 0.5f : 1.f))));
}

__device__ inline bool inside(const Dims& D, int i, int j, int k) {
  return i >= 0 && j >= 0 && k >= 0 && i < D.x && j < D.y && k < D.z;
}
__device__ inline float prolong_at(const float* psi_c, const Dims& Dc, int i, int j, int k);

// One full red-black Gauss-Seidel sweep (colour c1, then the other colour)
// per tile.  The tile's colour-c1 cells are updated on the tile and its
// 1-cell halo (the halo values are the ones the neighbouring tiles compute
// from the same old values), then the other colour on the tile itself, so
// the result equals two separate half-sweeps over the whole grid.  With
// psi_c, the prolonged coarse correction is added to every staged value
// first (the correction step fused into the sweep that follows it).
__global__ __launch_bounds__(256) void k_rb_sweep(float* __restrict__ psi, const float* __restrict__ f, Dims D, int c1,
                                                  const float* __restrict__ psi_c, Dims Dc) {
  constexpr int NP = PX * PY * PZ, NF = FX * FY * FZ;
  constexpr int RP = (NP + 255) / 256, RF = (NF + 255) / 256;
  __shared__ float sP[NP], sF[NF];
  const int tid = threadIdx.x;
  const int i0 = blockIdx.x * TX, j0 = blockIdx.y * TY, k0 = blockIdx.z * TZ;
  // staging: every load of the thread is issued before the first is used
  // (a loop that stored each value to LDS as it arrived would wait out one
  // memory latency per iteration)
  float vp[RP], vf[RF];
#pragma unroll
  for (int r = 0; r < RP; r++) {
    const int q = tid + r * 256;
    const int a = q / (PY * PZ), b = (q / PZ) % PY, c = q % PZ;
    const int i = i0 - 2 + a, j = j0 - 2 + b, k = k0 - 2 + c;
    vp[r] = (q < NP && inside(D, i, j, k)) ? psi[gidx(i, j, k, D.y, D.z)] : 0.f;
  }
#pragma unroll
  for (int r = 0; r < RF; r++) {
    const int q = tid + r * 256;
    const int a = q / (FY * FZ), b = (q / FZ) % FY, c = q % FZ;
    const int i = i0 - 1 + a, j = j0 - 1 + b, k = k0 - 1 + c;
    vf[r] = (q < NF && inside(D, i, j, k)) ? f[gidx(i, j, k, D.y, D.z)] : 0.f;
  }
  if (psi_c) {
#pragma unroll
    for (int r = 0; r < RP; r++) {
      const int q = tid + r * 256;
      const int a = q / (PY * PZ), b = (q / PZ) % PY, c = q % PZ;
      const int i = i0 - 2 + a, j = j0 - 2 + b, k = k0 - 2 + c;
      if (q < NP && inside(D, i, j, k)) vp[r] += prolong_at(psi_c, Dc, i, j, k);
    }
  }
#pragma unroll
  for (int r = 0; r < RP; r++) {
    const int q = tid + r * 256;
    if (q < NP) sP[q] = vp[r];
  }
#pragma unroll
  for (int r = 0; r < RF; r++) {
    const int q = tid + r * 256;
    if (q < NF) sF[q] = vf[r];
  }
  __syncthreads();
  auto update = [&](int i, int j, int k, int pq, int fq) {
    float s = 0.f;
    int cnt = 0;
    if (i > 0) { s += sP[pq - PY * PZ]; cnt++; }
    if (i + 1 < D.x) { s += sP[pq + PY * PZ]; cnt++; }
    if (j > 0) { s += sP[pq - PZ]; cnt++; }
    if (j + 1 < D.y) { s += sP[pq + PZ]; cnt++; }
    if (k > 0) { s += sP[pq - 1]; cnt++; }
    if (k + 1 < D.z) { s += sP[pq + 1]; cnt++; }
    sP[pq] = (s - sF[fq]) * inv_count(cnt);
  };
  for (int q = tid; q < FX * FY * FZ; q += 256) {
    const int a = q / (FY * FZ), b = (q / FZ) % FY, c = q % FZ;
    const int i = i0 - 1 + a, j = j0 - 1 + b, k = k0 - 1 + c;
    if (inside(D, i, j, k) && ((i + j + k) & 1) == c1) update(i, j, k, ((a + 1) * PY + b + 1) * PZ + c + 1, q);
  }
  __syncthreads();
  for (int q = tid; q < TX * TY * TZ; q += 256) {
    const int a = q / (TY * TZ), b = (q / TZ) % TY, c = q % TZ;
    const int i = i0 + a, j = j0 + b, k = k0 + c;
    if (inside(D, i, j, k) && ((i + j + k) & 1) != c1)
      update(i, j, k, ((a + 2) * PY + b + 2) * PZ + c + 2, ((a + 1) * FY + b + 1) * FZ + c + 1);
  }
  __syncthreads();
  for (int q = tid; q < TX * TY * TZ; q += 256) {
    const int a = q / (TY * TZ), b = (q / TZ) % TY, c = q % TZ;
    const int i = i0 + a, j = j0 + b, k = k0 + c;
    if (inside(D, i, j, k)) psi[gidx(i, j, k, D.y, D.z)] = sP[((a + 2) * PY + b + 2) * PZ + c + 2];
  }
}

__device__ inline float residual_at(const float* psi, const float* f, const Dims& D, int i, int j, int k) {
  int cnt;
  const float s = nb_sum(psi, D, i, j, k, cnt);
  const size_t c = gidx(i, j, k, D.y, D.z);
  return f[c] - (s - (float)cnt * psi[c]);
}

// One red-black half-sweep (the cells of one colour), one thread per pair of
// z-neighbours (one cell of each colour), for the finest levels.
__global__ __launch_bounds__(256) void k_rb_half(float* __restrict__ psi, const float* __restrict__ f, Dims D,
                                                 int color) {
  const uint32_t nzp = (uint32_t)D.z >> 1;
  const uint32_t n = (uint32_t)D.x * (uint32_t)D.y * nzp;
  for (uint32_t g = blockIdx.x * blockDim.x + threadIdx.x; g < n; g += gridDim.x * blockDim.x) {
    const uint32_t r = g / nzp, kp = g - r * nzp;
    const int i = (int)(r / (uint32_t)D.y), j = (int)(r - (uint32_t)i * (uint32_t)D.y);
    const int k = 2 * (int)kp + ((color + i + j) & 1);
    int cnt;
    const float sn = nb_sum(psi, D, i, j, k, cnt);
    const size_t c = gidx(i, j, k, D.y, D.z);
    psi[c] = (sn - f[c]) * inv_count(cnt);
  }
}

__global__ __launch_bounds__(256) void k_prolong(const float* __restrict__ psi_c, Dims Dc, float* __restrict__ psi,
                                                 Dims Df) {
  const size_t n = Df.cells();
  for (size_t g = blockIdx.x * (size_t)blockDim.x + threadIdx.x; g < n; g += (size_t)gridDim.x * blockDim.x) {
    int i, j, k;
    cell_of(Df, g, i, j, k);
    psi[g] += prolong_at(psi_c, Dc, i, j, k);
  }
}

__global__ __launch_bounds__(256) void k_restrict(const float* __restrict__ psi, const float* __restrict__ f, Dims Df,
                                                  float* __restrict__ psi_c, float* __restrict__ f_c, Dims Dc) {
  const size_t n = Dc.cells();
  for (size_t g = blockIdx.x * (size_t)blockDim.x + threadIdx.x; g < n; g += (size_t)gridDim.x * blockDim.x) {
    int I, J, K;
    cell_of(Dc, g, I, J, K);
    float r = 0.f;
#pragma unroll
    for (int c = 0; c < 8; c++) r += residual_at(psi, f, Df, 2 * I + (c >> 2), 2 * J + ((c >> 1) & 1), 2 * K + (c & 1));
    f_c[g] = 0.5f * r;
    psi_c[g] = 0.f;
  }
}

// trilinear interpolation from the coarse cell centres at fine cell (i, j, k)
__device__ inline float prolong_at(const float* psi_c, const Dims& Dc, int i, int j, int k) {
  const int I = i >> 1, J = j >> 1, K = k >> 1;
  const int I2 = min(max(I + ((i & 1) ? 1 : -1), 0), Dc.x - 1);
  const int J2 = min(max(J + ((j & 1) ? 1 : -1), 0), Dc.y - 1);
  const int K2 = min(max(K + ((k & 1) ? 1 : -1), 0), Dc.z - 1);
  const int ii[2] = {I, I2}, jj[2] = {J, J2}, kk[2] = {K, K2};
  const float wt[2] = {0.75f, 0.25f};
  float s = 0.f;
#pragma unroll
  for (int a = 0; a < 2; a++)
#pragma unroll
    for (int b = 0; b < 2; b++)
#pragma unroll
      for (int c = 0; c < 2; c++) s += wt[a] * wt[b] * wt[c] * psi_c[gidx(ii[a], jj[b], kk[c], Dc.y, Dc.z)];
  return s;
}


struct BottomArgs {
  int n_levels;              // levels handled here (the first is the entry level)
  Dims D[MAX_LEVELS];
  float* psi;                // entry level's psi (global): initial guess in, solution out
  const float* f;            // entry level's right-hand side (global)
};

// The V-cycle below the entry level, in one workgroup with every level in LDS.
__global__ __launch_bounds__(BOTTOM_THREADS) void k_bottom(BottomArgs B) {
  __shared__ float s_psi[BOTTOM_LDS], s_f[BOTTOM_LDS];
  __shared__ int s_ijk[BOTTOM_LDS];   // packed i | j << 10 | k << 20 of every cell of every level
  const int tid = threadIdx.x, NT = blockDim.x;
  int off[MAX_LEVELS];
  {
    int o = 0;
    for (int l = 0; l < B.n_levels; l++) { off[l] = o; o += (int)B.D[l].cells(); }
  }
  const int n0 = (int)B.D[0].cells();
  for (int c = tid; c < n0; c += NT) { s_psi[c] = B.psi[c]; s_f[c] = B.f[c]; }
  // the cell coordinates, decoded once (the phases below only read them)
  for (int l = 0; l < B.n_levels; l++)
    for (int c = tid; c < (int)B.D[l].cells(); c += NT) {
      int i, j, k;
      cell_of(B.D[l], c, i, j, k);
      s_ijk[off[l] + c] = i | (j << 10) | (k << 20);
    }
  __syncthreads();
  auto sweep = [&](int l, int color) {
    const Dims D = B.D[l];
    float* p = s_psi + off[l];
    const float* fl = s_f + off[l];
    const int* ijk = s_ijk + off[l];
    for (int c = tid; c < (int)D.cells(); c += NT) {
      const int e = ijk[c];
      const int i = e & 1023, j = (e >> 10) & 1023, k = e >> 20;
      if (((i + j + k) & 1) != color) continue;
      int cnt;
      const float s = nb_sum(p, D, i, j, k, cnt);
      p[c] = (s - fl[c]) / (float)cnt;
    }
    __syncthreads();
  };
  const int L = B.n_levels;
  for (int l = 0; l + 1 < L; l++) {
    for (int sw = 0; sw < NU_BOTTOM; sw++) { sweep(l, 0); sweep(l, 1); }
    const Dims Df = B.D[l], Dc = B.D[l + 1];
    for (int c = tid; c < (int)Dc.cells(); c += NT) {
      const int e = s_ijk[off[l + 1] + c];
      const int I = e & 1023, J = (e >> 10) & 1023, K = e >> 20;
      float r = 0.f;
      for (int q = 0; q < 8; q++)
        r += residual_at(s_psi + off[l], s_f + off[l], Df, 2 * I + (q >> 2), 2 * J + ((q >> 1) & 1), 2 * K + (q & 1));
      s_f[off[l + 1] + c] = 0.5f * r;
      s_psi[off[l + 1] + c] = 0.f;
    }
    __syncthreads();
  }
  for (int it = 0; it < COARSE_SWEEPS; it++) { sweep(L - 1, 0); sweep(L - 1, 1); }
  for (int l = L - 2; l >= 0; l--) {
    const Dims Df = B.D[l], Dc = B.D[l + 1];
    for (int c = tid; c < (int)Df.cells(); c += NT) {
      const int e = s_ijk[off[l] + c];
      const int i = e & 1023, j = (e >> 10) & 1023, k = e >> 20;
      s_psi[off[l] + c] += prolong_at(s_psi + off[l + 1], Dc, i, j, k);
    }
    __syncthreads();
    for (int sw = 0; sw < NU_BOTTOM; sw++) { sweep(l, 1); sweep(l, 0); }
  }
  for (int c = tid; c < n0; c += NT) B.psi[c] = s_psi[c];
}

// ---------------------------------------------------------------------------
// Spectral pressure solve.  With closed walls on a box of uniform cells the
// 7-point Neumann Laplacian is the Kronecker sum of 1-D Neumann Laplacians,
// each diagonalised by the DCT-II basis cos(pi k (i + 1/2) / n) with
// eigenvalues -4 sin^2(pi k / 2n).  So A psi = f is solved exactly by three
// axis transforms, a division by lambda_x + lambda_y + lambda_z (the
// constant mode, lambda = 0, set to zero: the gauge), and three inverse
// transforms.  Each axis transform is a dense contraction with an n x n
// matrix: out[k] = sum_i M[i][k] in[i] along the axis.
// ---------------------------------------------------------------------------
// The contractions run on the matrix cores in FP32 (v_mfma_f32_16x16x4f32),
// 16 outputs x 16 lines a tile, two accumulators over alternate steps of four
// terms, added at the end.  A wavefront takes 16 C lines and AXIS_MT tiles of
// outputs at a time; the wavefronts of a workgroup share the lines.  Nothing
// goes through LDS on the way in: the matrix is laid out once in the order in
// which lanes hold it; along y and x a lane loads its C adjacent lines at once,
// along z four adjacent terms, exchanged over the lanes that hold a line (with
// 4-byte loads of the terms as they are needed 18.7 and 22.4 us).  The last forward pass (x), the division by the eigenvalues and the first
// inverse pass are one launch, the coefficients in LDS between them.  At 128^3:
// 10.6 and 14.1 us forward and back along z, 9.7 and 9.6 along y and 17.5 for both
// along x (a pass's floor: 16.8 MB at the rate of a large copy, 3.2 us, and 537
// MFLOP, 3.5 us on all matrix cores; at two wavefronts per SIMD the latency of the
// loads ahead of each 32 products is the rest); 14 us each when 16 lines x 16
// outputs a wavefront went through LDS and every line chunk was read eight times.
// One output tile at a time takes 12 us along y and 20 along x, four 12 and 25.
// Half-length contractions by the parity of the basis (sums and differences of the
// two halves of a line) took 48 us a solve, not 61, but round differently:
// gradients that hang on the far tail of the emitter moved by their own error, now
// and then to twice it.  Here every sum is taken in the order of the terms, and
// the results are the bits of the contractions staged through LDS.
typedef float floatx4 __attribute__((ext_vector_type(4)));

struct AxisArgs {
  const float* in;
  float* out;
  const float4* M;       // the pass's matrix, in fragments (see gas_create)
  const float4* M2;      // AXIS_BOTH: the inverse's
  int n;                 // length of the transformed axis
  int A, B;              // layout [A][n][B]; inner transform (B == 1): A lines of n contiguous values
  // division of the outputs by the 3-D eigenvalue (along x; NULL: none); output index k = kx, line index b = ky * nz + kz
  const float* lx;
  const float* ly;
  const float* lz;
  int nz;
};

enum { AXIS_ONE = 0, AXIS_BOTH = 1 };

// 16-term steps, and 16-output tiles, of an axis of n values
__host__ __device__ inline int axis_steps(int n) { return (n + 15) / 16; }
constexpr int AXIS_MT = 2;   // output tiles a wavefront takes together

template <int C> struct AxisVec;
template <> struct AxisVec<2> { using T = float2; };
template <int C> __device__ __forceinline__ float axis_get(const typename AxisVec<C>::T& v, int c) {
  return reinterpret_cast<const float*>(&v)[c];
}

// 4 x 4 transpose over the four rows of 16 lanes: lane (lr, lc) gives v[t] to
// element lr of lane (t, lc)
__device__ __forceinline__ float4 axis_transpose(float4 v) {
  typedef uint32_t u2 __attribute__((ext_vector_type(2)));
  const uint32_t x = __float_as_uint(v.x), y = __float_as_uint(v.y), z = __float_as_uint(v.z), w = __float_as_uint(v.w);
  const u2 xz = __builtin_amdgcn_permlane32_swap(x, z, false, false);   // rows 2, 3 of x with rows 0, 1 of z
  const u2 yw = __builtin_amdgcn_permlane32_swap(y, w, false, false);
  const u2 xy = __builtin_amdgcn_permlane16_swap(xz[0], yw[0], false, false);   // rows 1, 3 of x with rows 0, 2 of y
  const u2 zw = __builtin_amdgcn_permlane16_swap(xz[1], yw[1], false, false);
  return make_float4(__uint_as_float(xy[0]), __uint_as_float(xy[1]), __uint_as_float(zw[0]), __uint_as_float(zw[1]));
}

// Output tiles m0 .. m0 + AXIS_MT - 1: res[q][c] = 16 outputs x 16 lines (line
// tile c).  load(s, e): the C values of each of the terms 16 s + 4 t + lr, t < 4.
template <int C, class Load>
__device__ __forceinline__ void axis_contract(const float4* __restrict__ M, int S, int m0, int lane, Load&& load,
                                              floatx4 (&res)[AXIS_MT][C]) {
  floatx4 acc[2][AXIS_MT][C];
  const float4* Mq[AXIS_MT];
#pragma unroll
  for (int q = 0; q < AXIS_MT; q++) {
    Mq[q] = M + (size_t)min(m0 + q, S - 1) * S * 64 + lane;   // (a tile past the last is not stored)
#pragma unroll
    for (int u = 0; u < 2; u++)
#pragma unroll
      for (int c = 0; c < C; c++) acc[u][q][c] = floatx4{0.f, 0.f, 0.f, 0.f};
  }
#pragma unroll 2
  for (int s = 0; s < S; s++) {
    float4 f[AXIS_MT];
#pragma unroll
    for (int q = 0; q < AXIS_MT; q++) f[q] = Mq[q][s * 64];
    float e[4][C];
    load(s, e);
#pragma unroll
    for (int t = 0; t < 4; t++)
#pragma unroll
      for (int q = 0; q < AXIS_MT; q++)
#pragma unroll
        for (int c = 0; c < C; c++)
          acc[t & 1][q][c] =
              __builtin_amdgcn_mfma_f32_16x16x4f32(reinterpret_cast<const float*>(&f[q])[t], e[t][c], acc[t & 1][q][c], 0, 0, 0);
  }
#pragma unroll
  for (int q = 0; q < AXIS_MT; q++)
#pragma unroll
    for (int c = 0; c < C; c++) res[q][c] = acc[0][q][c] + acc[1][q][c];
}

template <bool INNER, int KIND, int C>
__global__ __launch_bounds__(256) void k_axis(AxisArgs X) {
  using V = typename AxisVec<C>::T;
  extern __shared__ __align__(16) float s_coef[];   // AXIS_BOTH: [k][16 C lines]
  constexpr int LINES = 16 * C;
  const int lane = threadIdx.x & 63, lr = lane >> 4, lc = lane & 15;
  const int wv = threadIdx.x >> 6, nw = blockDim.x >> 6;
  const int n = X.n, S = axis_steps(n);
  const int line0 = blockIdx.x * LINES;
  // output tiles: every wavefront of the line's workgroups (blockIdx.z) in turn
  const int m_first = AXIS_MT * (wv + nw * (int)blockIdx.z), m_step = AXIS_MT * nw * (int)gridDim.z;
  floatx4 res[AXIS_MT][C];
  if (INNER) {
    // line tile c of the lane: row line0 + 16 c + lc
    const float* in[C];
    bool on[C];
#pragma unroll
    for (int c = 0; c < C; c++) {
      const int line = line0 + 16 * c + lc;
      on[c] = line < X.A;
      in[c] = X.in + (size_t)(on[c] ? line : 0) * n;
    }
    for (int m0 = m_first; m0 < S; m0 += m_step) {
      axis_contract<C>(X.M, S, m0, lane, [&](int s, float (&e)[4][C]) {
        const int i = min(16 * s + 4 * lr, n - 4);   // (past n the matrix is zero)
#pragma unroll
        for (int c = 0; c < C; c++) {
          const float4 a = axis_transpose(*(const float4*)(in[c] + i));
          e[0][c] = a.x; e[1][c] = a.y; e[2][c] = a.z; e[3][c] = a.w;
        }
      }, res);
#pragma unroll
      for (int q = 0; q < AXIS_MT; q++) {
        const int k = 16 * (m0 + q) + 4 * lr;   // (n is a multiple of 4)
        if (k >= n) continue;
#pragma unroll
        for (int c = 0; c < C; c++)
          if (on[c])
            *(float4*)(X.out + (size_t)(line0 + 16 * c + lc) * n + k) =
                make_float4(res[q][c][0], res[q][c][1], res[q][c][2], res[q][c][3]);
      }
    }
    return;
  }
  // line tile c of the lane: column line + c of the [n][B] plane
  const int line = line0 + C * lc;
  const bool on = line < X.B;
  const size_t plane = (size_t)blockIdx.y * n * X.B;
  // (a lane past the last line reads its workgroup's first one: in place, the others' lines may be being written)
  const float* in = X.in + plane + (on ? line : line0);
  float* out = X.out + plane + line;
  const uint32_t B = (uint32_t)X.B;
  float lyz[C];
  const bool divide = X.lx != nullptr;
  if (divide) {
    const int l = on ? line : 0, ky = l / X.nz, kz = l - ky * X.nz;   // (C divides nz: the lines share ky)
#pragma unroll
    for (int c = 0; c < C; c++) { lyz[c] = X.lz[kz + c]; }
    const float ly = X.ly[ky];
    for (int m0 = m_first; m0 < S; m0 += m_step) {
      axis_contract<C>(X.M, S, m0, lane, [&](int s, float (&e)[4][C]) {
#pragma unroll
        for (int t = 0; t < 4; t++) {
          const V a = *(const V*)(in + (uint32_t)min(16 * s + 4 * t + lr, n - 1) * B);
#pragma unroll
          for (int c = 0; c < C; c++) e[t][c] = axis_get<C>(a, c);
        }
      }, res);
#pragma unroll
      for (int q = 0; q < AXIS_MT; q++)
#pragma unroll
        for (int r = 0; r < 4; r++) {
          const int k = 16 * (m0 + q) + 4 * lr + r;
          if (k >= n) continue;
          V v;
          float* f = reinterpret_cast<float*>(&v);
#pragma unroll
          for (int c = 0; c < C; c++) {
            const float lam = X.lx[k] + ly + lyz[c];
            f[c] = lam != 0.f ? res[q][c][r] / lam : 0.f;
          }
          if (KIND == AXIS_BOTH) *(V*)(s_coef + k * LINES + C * lc) = v;
          else if (on) *(V*)(out + (uint32_t)k * B) = v;
        }
    }
    if (KIND != AXIS_BOTH) return;
    __syncthreads();
  }
  const float4* Mi = KIND == AXIS_BOTH ? X.M2 : X.M;
  for (int m0 = m_first; m0 < S; m0 += m_step) {
    axis_contract<C>(Mi, S, m0, lane, [&](int s, float (&e)[4][C]) {
#pragma unroll
      for (int t = 0; t < 4; t++) {
        const int i = min(16 * s + 4 * t + lr, n - 1);
        const V a = KIND == AXIS_BOTH ? *(const V*)(s_coef + i * LINES + C * lc) : *(const V*)(in + (uint32_t)i * B);
#pragma unroll
        for (int c = 0; c < C; c++) e[t][c] = axis_get<C>(a, c);
      }
    }, res);
    if (!on) continue;
#pragma unroll
    for (int q = 0; q < AXIS_MT; q++)
#pragma unroll
      for (int r = 0; r < 4; r++) {
        const int k = 16 * (m0 + q) + 4 * lr + r;
        if (k >= n) continue;
        V v;
#pragma unroll
        for (int c = 0; c < C; c++) reinterpret_cast<float*>(&v)[c] = res[q][c][r];
        *(V*)(out + (uint32_t)k * B) = v;
      }
  }
}

// |f - A psi|^2 and |f|^2 per block into part[2 * block]; the last step sums
__global__ __launch_bounds__(256) void k_resnorm(const float* __restrict__ psi, const float* __restrict__ f, Dims D,
                                                 double* __restrict__ part) {
  __shared__ double s_r[256], s_b[256];
  double r2 = 0.0, b2 = 0.0;
  const size_t n = D.cells();
  for (size_t g = blockIdx.x * (size_t)blockDim.x + threadIdx.x; g < n; g += (size_t)gridDim.x * blockDim.x) {
    int i, j, k;
    cell_of(D, g, i, j, k);
    const double r = residual_at(psi, f, D, i, j, k);
    r2 += r * r;
    b2 += (double)f[g] * f[g];
  }
  s_r[threadIdx.x] = r2;
  s_b[threadIdx.x] = b2;
  __syncthreads();
  for (int o = 128; o > 0; o >>= 1) {
    if ((int)threadIdx.x < o) { s_r[threadIdx.x] += s_r[threadIdx.x + o]; s_b[threadIdx.x] += s_b[threadIdx.x + o]; }
    __syncthreads();
  }
  if (threadIdx.x == 0) { part[2 * blockIdx.x] = s_r[0]; part[2 * blockIdx.x + 1] = s_b[0]; }
}
__global__ void k_resnorm_final(const double* __restrict__ part, int nb, double* __restrict__ out) {
  if (threadIdx.x != 0 || blockIdx.x != 0) return;
  double r = 0.0, b = 0.0;
  for (int q = 0; q < nb; q++) { r += part[2 * q]; b += part[2 * q + 1]; }
  out[0] = b > 0.0 ? sqrt(r / b) : 0.0;
}

// ---------------------------------------------------------------------------
// adjoint
// ---------------------------------------------------------------------------
struct AdjOut {
  float* u;
  float* v;
  float* w;
  float* s;
};

// Adjoint of advection + emitter + buoyancy for every grid point of state s_t.
// ub1/vb1/wb1: adjoint of the blended velocities (already projected, walls
// zero); sb: adjoint of the output scalars; out: adjoint of s_t (cleared
// before; accumulated with atomics); slots: pose partials.
//
// The atomics of the scatter at the back-traced points were 215 of its 392 us at
// 128^3 (two scalars; four to eight a sample), and what they cost goes with the
// cache lines they touch, so samples that share corners are merged first.
// Neighbouring points' samples usually lie in neighbouring cells: a wavefront
// holds 64 columns consecutive along z, whose lanes hand their k0 + 1 corners to
// the next lane; a thread walks ADJ_J points along y and carries its j0 + 1
// corners to the next one; and the workgroup's ADJ_I wavefronts hold consecutive
// planes, each handing its i0 + 1 corners to the next through LDS.  The corners
// at k0 + 1 that no lane took (mostly the last lane's) are carried and handed on
// in the same way.  Each merge is taken only where the cells do adjoin (the
// cell's packed index says so).  With an adjoint that is non-zero everywhere 506 ->
// 240 us; over the eight steps back from a loss of 27 cells, where much of it is
// still zero, 392 -> 197 on average (113 in the first, 215 in the last), 65 of them
// the atomics, and there 261 with the last lane's corners issued as they come, 205
// and 210 with 4 x 4 and 4 x 8 planes x points, 222 and 244 with 2 x 4 and 8 x 2.
// (Columns, not points, are dealt to the lanes, so that rows of any length fill the
// wavefronts.)
//
// ADJ_J points one after the other are a chain, which sets the time of a small
// grid (12 x 20 x 28, four scalars: 63 us); there a thread takes one point.  The
// line is at three workgroups a CU with one point a thread: backward of four steps
// at 40^3 469 us against 534 with ADJ_J points, 48^3 505 and 540, 64^3 700 and 675,
// 8 x 1024 x 8 1000 and 950.
constexpr int ADJ_J = 8, ADJ_I = 8;   // points a thread (or one), planes (wavefronts) a workgroup
constexpr uint32_t ADJ_SHORT_BLOCKS = 3 * 256;

__device__ __forceinline__ int lane_prev(int x) { return __builtin_amdgcn_update_dpp(0, x, 0x138, 0xF, 0xF, false); }   // wave_shr:1
__device__ __forceinline__ int lane_next(int x) { return __builtin_amdgcn_update_dpp(0, x, 0x130, 0xF, 0xF, false); }   // wave_shl:1
__device__ __forceinline__ float lane_prev(float x) { return __int_as_float(lane_prev(__float_as_int(x))); }

// blocks of 64 columns (j group, k) of each grid, and groups of ADJ_I planes
inline PointGrid column_grid(const GP& P, int J) {
  PointGrid G = {};
  for (int q = 0; q < 4; q++) {
    const uint32_t groups = (uint32_t)(P.ny + (q == 1) + J - 1) / J;
    G.nb[q] = (groups * (uint32_t)(P.nz + (q == 2)) + 63u) / 64u;
    G.per += G.nb[q];
  }
  G.blocks = G.per * (uint32_t)((P.nx + ADJ_I) / ADJ_I);
  G.mper = (uint32_t)((0x100000000ull + G.per - 1) / G.per);
  return G;
}

constexpr uint32_t CELL_I = 1u << 22, CELL_J = 1u << 11, NO_CELL = 0xffffffffu;   // packed cell: i0, j0, k0

struct AdjLds {
  uint32_t cell[2][ADJ_I][64];
  float e[2][ADJ_I][MAXK][64], h[2][ADJ_I][MAXK][64];   // the rows at k0 and (where the next lane did not take it) k0 + 1
};

template <int Q, int J>
__device__ __forceinline__ void adj_columns(const GP& P, const VelPtrs& vel, const float* __restrict__ s,
                                            const float* __restrict__ ab_in, const float* __restrict__ vb1,
                                            float* __restrict__ tgt, const Pose& E, float* __restrict__ ub, size_t total,
                                            int i, int col0, AdjLds& S, double* part) {
  constexpr int NV = Q < 3 ? 1 : MAXK;
  const int K = Q < 3 ? 1 : P.K;
  const int lane = (int)__lane_id(), wv = (int)(threadIdx.x >> 6);
  const int d0 = P.nx + (Q == 0), d1 = P.ny + (Q == 1), d2 = P.nz + (Q == 2);
  const int groups = (d1 + J - 1) / J;
  const int col = col0 + lane, jg = row_of(col, Q == 2 ? P.mz1 : P.mz), k = col - jg * d2;
  const bool lane_on = i < d0 && jg < groups;
  const size_t sx = (size_t)d1 * d2;
  const size_t plane = (size_t)i * sx;   // (uniform)
  auto flush = [&](uint32_t c, int off1, int kk, float v) {   // v into corner off1 (x) of cell c, if any
    if (v == 0.f) return;
    const uint32_t at = ((c >> 22) * (uint32_t)d1 + ((c >> 11) & 2047u)) * (uint32_t)d2 + (c & 2047u);
    atomicAdd(tgt + (Q < 3 ? 0 : kk * P.nc) + (off1 ? sx : 0) + at, v);
  };
  uint32_t pcell = NO_CELL;   // carried row: the cell whose (i0, j0, k0) and (i0 + 1, j0, k0) corners it holds
  float pend[NV][2] = {}, hpend[NV][2] = {};
#pragma unroll 1
  for (int t = 0; t <= J; t++) {
    const int j = jg * J + t;
    const bool on = lane_on && t < J && j < d1;
    uint32_t cell = NO_CELL;
    Lerp L = {};
    float sval[NV] = {};
    if (on) {
      const uint32_t r = (uint32_t)(j * d2 + k);
      float d[3], U[3], xbb[3] = {0.f, 0.f, 0.f};   // xbb: adjoint of the back-traced point
      plane_velocity<Q>(P, vel, i, j, k, U);
      L = lerp_setup(P, Q, i, j, k, U);
      cell = ((uint32_t)L.i0 << 22) | ((uint32_t)L.j0 << 11) | (uint32_t)L.k0;
      const float chi = emitter_chi<Q>(P, E, i, j, k, d);
      const float dchi[3] = {chi * d[0] * 2.f * P.s2inv, chi * d[1] * 2.f * P.s2inv, chi * d[2] * 2.f * P.s2inv};
      auto sample = [&](const float* F, float ab, float target, int kk) {
        ZPair z[4];
        lerp_pairs(P.big, F, L, (uint32_t)d1, (uint32_t)d2, z);
        const float val = lerp_pairs_eval(z, L);
        // emitter: out = val + chi (target - val)
#pragma unroll
        for (int a = 0; a < 3; a++) part[a] += (double)(ab * (target - val) * dchi[a]);
        const float vbar = (1.f - chi) * ab;
        sval[kk] = vbar;
        const float c[8] = {z[0].a, z[0].b, z[1].a, z[1].b, z[2].a, z[2].b, z[3].a, z[3].b};
        float gr[3];
        lerp_grad(c, L, gr);
#pragma unroll
        for (int a = 0; a < 3; a++) xbb[a] += L.cl[a] ? 0.f : vbar * gr[a] * P.inv_h;
      };
      if (Q < 3) {
        const float ab = (ab_in + plane)[r];
        if (ab != 0.f) {
          part[3 + (Q < 3 ? Q : 0)] += (double)(ab * chi * P.speed);
          sample(Q == 0 ? vel.u : (Q == 1 ? vel.v : vel.w), ab, P.speed * E.a[Q < 3 ? Q : 0], 0);
        }
      } else {
#pragma unroll
        for (int kk = 0; kk < NV; kk++) {
          if (kk >= K) break;
          float ab = (ab_in + kk * P.nc + plane)[r];
          if (kk == 0) {
            // buoyancy: each interior y-face of this cell took dt beta T / 2
            const float* v0 = vb1 + (size_t)i * (sx + P.nz);
            float vs = 0.f;
            if (j > 0) vs += ld32(v0, r);
            if (j + 1 < P.ny) vs += ld32(v0, r + (uint32_t)P.nz);
            ab += 0.5f * P.dt * P.beta * vs;
          }
          if (ab != 0.f) sample(s + kk * P.nc, ab, P.src[kk], kk);
        }
      }
      // back-trace xb = x - dt U(x): U's adjoint -dt xbb is kept per point;
      // k_gas_adj_ugather spreads it over the velocity grids
#pragma unroll
      for (int a = 0; a < 3; a++) (ub + (size_t)a * total + plane)[r] = -P.dt * xbb[a];
    }
    // along z: the previous lane's cell adjoins this one's, or the next lane's this one's
    // (the lane moves run with every lane active: not behind a condition)
    const uint32_t cell_p = (uint32_t)lane_prev((int)cell);
    const bool take = lane > 0 && cell_p + 1u == cell;
    const int take_n = lane_next(take ? 1 : 0);
    const bool given = lane < 63 && take_n != 0;
    // along y: the carried row is this cell's
    const bool carried = pcell == cell;
    const uint32_t ecell = t < J ? cell : pcell;   // the row emitted now (after the last point, the carried one)
    float e0[NV], e1[NV], h0[NV], h1[NV];
#pragma unroll
    for (int kk = 0; kk < NV; kk++) {
      e0[kk] = e1[kk] = h0[kk] = h1[kk] = 0.f;
      if (kk >= K) continue;
      if (t == J) {
        e0[kk] = pend[kk][0]; e1[kk] = pend[kk][1];
        h0[kk] = hpend[kk][0]; h1[kk] = hpend[kk][1];
        continue;
      }
      const float gz = (1.f - L.f[2]) * sval[kk], fz = L.f[2] * sval[kk];
      float lo[2][2], hi[2][2];
#pragma unroll
      for (int cx = 0; cx < 2; cx++)
#pragma unroll
        for (int cy = 0; cy < 2; cy++) {
          const float wxy = (cx ? L.f[0] : 1.f - L.f[0]) * (cy ? L.f[1] : 1.f - L.f[1]);
          hi[cx][cy] = wxy * fz;
          const float hp = lane_prev(hi[cx][cy]);
          lo[cx][cy] = wxy * gz + (take ? hp : 0.f);
          if (given) hi[cx][cy] = 0.f;
        }
      if (carried) {
        lo[0][0] += pend[kk][0];
        lo[1][0] += pend[kk][1];
        hi[0][0] += hpend[kk][0];
        hi[1][0] += hpend[kk][1];
      } else if (pcell != NO_CELL) {
        flush(pcell, 0, kk, pend[kk][0]);
        flush(pcell, 1, kk, pend[kk][1]);
        flush(pcell + 1u, 0, kk, hpend[kk][0]);
        flush(pcell + 1u, 1, kk, hpend[kk][1]);
      }
      e0[kk] = lo[0][0];
      e1[kk] = lo[1][0];
      pend[kk][0] = lo[0][1];
      pend[kk][1] = lo[1][1];
      h0[kk] = hi[0][0];
      h1[kk] = hi[1][0];
      hpend[kk][0] = hi[0][1];
      hpend[kk][1] = hi[1][1];
    }
    pcell = cell == NO_CELL ? NO_CELL : cell + CELL_J;
    // along x: the next wavefront's cell adjoins this one's
    const int buf = t & 1;
    S.cell[buf][wv][lane] = ecell;
#pragma unroll
    for (int kk = 0; kk < NV; kk++)
      if (kk < K) {
        S.e[buf][wv][kk][lane] = e1[kk];
        S.h[buf][wv][kk][lane] = h1[kk];
      }
    __syncthreads();
    const uint32_t cp = wv > 0 ? S.cell[buf][wv - 1][lane] : NO_CELL, cn = wv < ADJ_I - 1 ? S.cell[buf][wv + 1][lane] : NO_CELL;
    const bool xtake = ecell != NO_CELL && ecell >= CELL_I && cp + CELL_I == ecell;
    const bool xgiven = ecell != NO_CELL && cn != NO_CELL && cn >= CELL_I && ecell + CELL_I == cn;
    if (ecell != NO_CELL) {
#pragma unroll
      for (int kk = 0; kk < NV; kk++) {
        if (kk >= K) break;
        flush(ecell, 0, kk, e0[kk] + (xtake ? S.e[buf][wv - 1][kk][lane] : 0.f));
        flush(ecell + 1u, 0, kk, h0[kk] + (xtake ? S.h[buf][wv - 1][kk][lane] : 0.f));
        if (!xgiven) {
          flush(ecell, 1, kk, e1[kk]);
          flush(ecell + 1u, 1, kk, h1[kk]);
        }
      }
    }
  }
}

template <int J>
__global__ __launch_bounds__(64 * ADJ_I) void k_gas_adj_advect(GP P, VelPtrs vel, const float* __restrict__ s,
                                                        const float* __restrict__ ub1, const float* __restrict__ vb1,
                                                        const float* __restrict__ wb1, const float* __restrict__ sb,
                                                        AdjOut out, const double* __restrict__ pose,
                                                        double* __restrict__ slots, float* __restrict__ ub, PointGrid G) {
  __shared__ AdjLds S;
  const size_t total = P.nu + P.nv + P.nw + P.nc;
  const Pose E = load_pose(pose);
  double part[POSE_PARTIALS] = {0, 0, 0, 0, 0, 0};
  uint32_t b = xcd_block();
  int ig = G.per == 1u ? (int)b : (int)__umulhi(b, G.mper);
  if ((uint32_t)ig * G.per > b) ig--;
  b -= (uint32_t)ig * G.per;
  int q = 0;
#pragma unroll
  for (int n = 0; n < 3; n++)
    if (q == n && b >= G.nb[n]) { b -= G.nb[n]; q = n + 1; }
  const int i = ADJ_I * ig + __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)), col0 = 64 * (int)b;
  if (q == 0) adj_columns<0, J>(P, vel, s, ub1, nullptr, out.u, E, ub, total, i, col0, S, part);
  else if (q == 1) adj_columns<1, J>(P, vel, s, vb1, nullptr, out.v, E, ub + P.nu, total, i, col0, S, part);
  else if (q == 2) adj_columns<2, J>(P, vel, s, wb1, nullptr, out.w, E, ub + P.nu + P.nv, total, i, col0, S, part);
  else adj_columns<3, J>(P, vel, s, sb, vb1, out.s, E, ub + P.nu + P.nv + P.nw, total, i, col0, S, part);
  // pose partials: wave sums, one FP64 atomic per component into the
  // wavefront's accumulator copy
  const int wave = blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6);
  double* dst = slots + (size_t)(wave % SLOTS) * POSE_PARTIALS;
#pragma unroll
  for (int qn = 0; qn < POSE_PARTIALS; qn++) {
    double v = part[qn];
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
    if (__lane_id() == 0 && v != 0.0) atomicAdd(dst + qn, v);
  }
}

// Adjoint of the velocity at every grid point (U of the back-traces, from
// the stencils of plane_velocity) as a gather: each velocity node of grid A
// sums the U_A adjoints (ub, from k_gas_adj_advect) of the points whose
// stencil holds it, with the stencil's weights: its own point (1), the two
// cells beside it along A (1/2 each), and on each other face grid B the points
// beside it along A (1/2) whose clamped pair along B holds it (1/2 per hit: the
// lower of the two is hit twice at the first node, the upper at the last).
template <int A>
__device__ __forceinline__ float ugather_point(const GP& P, const float* __restrict__ Uu, const float* __restrict__ Uv,
                                               const float* __restrict__ Uw, const float* __restrict__ Uc, int i, int r) {
  const int ny = P.ny, nz = P.nz;
  const size_t pu = (size_t)ny * nz, pv = pu + nz, pw = pu + ny;
  const uint32_t z = (uint32_t)nz;
  const int j = row_of(r, A == 2 ? P.mz1 : P.mz), k = r - j * (nz + (A == 2));
  auto hit = [](bool edge) { return edge ? 2.f : 1.f; };
  float cs = 0.f, f0 = 0.f, f1 = 0.f;
  if (A == 0) {
    const uint32_t o = (uint32_t)r, ow = o + (uint32_t)j;
    const float a0 = hit(j == 0), a1 = hit(j == ny - 1), b0 = hit(k == 0), b1 = hit(k == nz - 1);
#pragma unroll
    for (int ta = 0; ta < 2; ta++) {
      const int pi = i - 1 + ta;
      if (pi < 0 || pi >= P.nx) continue;   // (uniform)
      const float *c = Uc + pi * pu, *v = Uv + pi * pv, *w = Uw + pi * pw;
      cs += ld32(c, o);
      f0 += a0 * ld32(v, o) + a1 * ld32(v, o + z);
      f1 += b0 * ld32(w, ow) + b1 * ld32(w, ow + 1);
    }
    return ld32(Uu + i * pu, o) + 0.5f * cs + 0.25f * f0 + 0.25f * f1;
  }
  if (A == 1) {
    const float a0 = hit(i == 0), a1 = hit(i == P.nx - 1), b0 = hit(k == 0), b1 = hit(k == nz - 1);
    const float *c = Uc + i * pu, *u0 = Uu + i * pu, *u1 = u0 + pu, *w = Uw + i * pw;
#pragma unroll
    for (int ta = 0; ta < 2; ta++) {
      const int pj = j - 1 + ta;
      if (pj < 0 || pj >= ny) continue;
      const uint32_t o = (uint32_t)(pj * nz + k), ow = o + (uint32_t)pj;
      cs += ld32(c, o);
      f0 += a0 * ld32(u0, o) + a1 * ld32(u1, o);
      f1 += b0 * ld32(w, ow) + b1 * ld32(w, ow + 1);
    }
    return ld32(Uv + i * pv, (uint32_t)r) + 0.5f * cs + 0.25f * f0 + 0.25f * f1;
  }
  const float a0 = hit(i == 0), a1 = hit(i == P.nx - 1), b0 = hit(j == 0), b1 = hit(j == ny - 1);
  const float *c = Uc + i * pu, *u0 = Uu + i * pu, *u1 = u0 + pu, *v = Uv + i * pv;
#pragma unroll
  for (int ta = 0; ta < 2; ta++) {
    const int pk = k - 1 + ta;
    if (pk < 0 || pk >= nz) continue;
    const uint32_t o = (uint32_t)(j * nz + pk);
    cs += ld32(c, o);
    f0 += a0 * ld32(u0, o) + a1 * ld32(u1, o);
    f1 += b0 * ld32(v, o) + b1 * ld32(v, o + z);
  }
  return ld32(Uw + i * pw, (uint32_t)r) + 0.5f * cs + 0.25f * f0 + 0.25f * f1;
}

constexpr int UG_U = 2;
__global__ __launch_bounds__(256) void k_gas_adj_ugather(GP P, const float* __restrict__ ub, AdjOut out, PointGrid G) {
  const size_t total = P.nu + P.nv + P.nw + P.nc;
  const PlaneBlock b = plane_block<UG_U>(P, G);
  auto points = [&](auto a, float* O) {
    constexpr int A = decltype(a)::value;
    const float *Uu = ub + A * total, *Uv = Uu + P.nu, *Uw = Uv + P.nv, *Uc = Uw + P.nw;
    O += (size_t)b.i * plane_points(A, P.ny, P.nz);
#pragma unroll
    for (int t = 0; t < UG_U; t++) {
      const int r = b.r0 + 256 * t + (int)threadIdx.x;
      if (r < b.n) O[(uint32_t)r] += ugather_point<A>(P, Uu, Uv, Uw, Uc, b.i, r);
    }
  };
  if (b.q == 0) points(std::integral_constant<int, 0>{}, out.u);
  else if (b.q == 1) points(std::integral_constant<int, 1>{}, out.v);
  else points(std::integral_constant<int, 2>{}, out.w);
}

// sum of the accumulator copies into the step's pose partials (c at 6..8 and
// the axis a = R e_y at 9..11 of the ACC_DOUBLES layout); copies cleared
__global__ __launch_bounds__(64) void k_gas_pose_acc(double* __restrict__ slots, double* __restrict__ acc_t) {
  const int lane = threadIdx.x;
  double tot[POSE_PARTIALS];
#pragma unroll
  for (int qn = 0; qn < POSE_PARTIALS; qn++) tot[qn] = 0.0;
  for (int sl = lane; sl < SLOTS; sl += 64) {
#pragma unroll
    for (int qn = 0; qn < POSE_PARTIALS; qn++) { tot[qn] += slots[sl * POSE_PARTIALS + qn]; slots[sl * POSE_PARTIALS + qn] = 0.0; }
  }
#pragma unroll
  for (int qn = 0; qn < POSE_PARTIALS; qn++)
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) tot[qn] += __shfl_xor(tot[qn], o);
  if (lane == 0) {
#pragma unroll
    for (int qn = 0; qn < POSE_PARTIALS; qn++) acc_t[6 + qn] += tot[qn];
  }
}

// sensor loss: one workgroup
__global__ __launch_bounds__(256) void k_gas_sensors(const float* __restrict__ T, size_t nc, int n,
                                                     const int* __restrict__ cells, const float* __restrict__ targets,
                                                     float* __restrict__ loss, float* __restrict__ gT) {
  __shared__ double s_l[256];
  double l = 0.0;
  for (int m = threadIdx.x; m < n; m += blockDim.x) {
    const int c = cells[m];
    if (c < 0 || (size_t)c >= nc) continue;
    const float e = T[c] - targets[m];
    l += fabs((double)e);
    if (gT) atomicAdd(&gT[c], e > 0.f ? 1.f : (e < 0.f ? -1.f : 0.f));
  }
  s_l[threadIdx.x] = l;
  __syncthreads();
  for (int o = 128; o > 0; o >>= 1) {
    if ((int)threadIdx.x < o) s_l[threadIdx.x] += s_l[threadIdx.x + o];
    __syncthreads();
  }
  if (threadIdx.x == 0) loss[0] = (float)s_l[0];
}

// ---------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------
struct Layout {
  size_t tmp, pose, act, acc, slots, resp, resout, err, ckpt, seg, adj0, adj1, ub;
  size_t spec_tmp, dct[3], idct[3], lam[3];   // spectral solve: a cell array, per-axis matrices and eigenvalues
  size_t psi[MAX_LEVELS], f[MAX_LEVELS];
  size_t total;
  size_t state_floats;
  int n_levels, n_grid_levels, n_ckpt;
  Dims D[MAX_LEVELS];
};

bool desc_ok(const gas_desc* d) {
  if (!d) return false;
  const int n[3] = {d->nx, d->ny, d->nz};
  for (int a = 0; a < 3; a++)
    if (n[a] < 8 || n[a] > 1024 || (n[a] % 4) != 0) return false;
  if (!(d->h > 0.f) || !(d->dt > 0.f)) return false;
  if (d->n_scalars < 1 || d->n_scalars > MAXK || !d->src) return false;
  if (!(d->emit_sigma > 0.f) || !(d->emit_kappa >= 0.f && d->emit_kappa <= 1.f)) return false;
  if (d->horizon < 1 || d->mg_cycles < 1 || d->mg_cycles > 64) return false;
  if (d->pressure_solver != 0 && d->pressure_solver != 1) return false;
  if (d->requires_grad && (d->ckpt_every < 1 || d->ckpt_every > 4096)) return false;
  return true;
}

Layout plan(const gas_desc* d);

// (the coarsest level must fit the one-workgroup bottom solve)
bool levels_ok(const gas_desc* d);

Layout plan(const gas_desc* d) {
  Layout L;
  const size_t nx = d->nx, ny = d->ny, nz = d->nz, K = d->n_scalars, T = d->horizon;
  const size_t nc = nx * ny * nz;
  L.state_floats = (nx + 1) * ny * nz + nx * (ny + 1) * nz + nx * ny * (nz + 1) + K * nc;
  // levels: halve while every dimension stays even and at least 2
  L.D[0] = Dims{d->nx, d->ny, d->nz};
  L.n_levels = 1;
  while (L.n_levels < MAX_LEVELS) {
    const Dims p = L.D[L.n_levels - 1];
    if ((p.x & 1) || (p.y & 1) || (p.z & 1) || p.x < 4 || p.y < 4 || p.z < 4) break;
    L.D[L.n_levels++] = Dims{p.x / 2, p.y / 2, p.z / 2};
  }
  // the grid levels end where the levels fit one workgroup's LDS
  L.n_grid_levels = 0;
  while (L.n_grid_levels < L.n_levels && L.D[L.n_grid_levels].cells() > (size_t)BOTTOM_CELLS) L.n_grid_levels++;
  size_t o = 0;
  auto take = [&](size_t b) { size_t r = o; o += al256(b); return r; };
  L.tmp = take(L.state_floats * 4);
  {
    const int nn[3] = {d->nx, d->ny, d->nz};
    L.spec_tmp = take(nc * 4);
    for (int a = 0; a < 3; a++) {
      const size_t st = axis_steps(nn[a]);
      L.dct[a] = take(st * st * 64 * sizeof(float4));
      L.idct[a] = take(st * st * 64 * sizeof(float4));
      L.lam[a] = take((size_t)nn[a] * 4);
    }
  }
  for (int l = 0; l < L.n_levels; l++) { L.psi[l] = take(L.D[l].cells() * 4); L.f[l] = take(L.D[l].cells() * 4); }
  L.pose = take((T + 1) * POSE_DOUBLES * sizeof(double));
  L.act = take(T * 6 * sizeof(float));
  L.slots = take(SLOTS * POSE_PARTIALS * sizeof(double));
  L.resp = take(2 * 4096 * sizeof(double));
  L.resout = take(64);
  L.err = take(64);
  if (d->requires_grad) {
    const int k = d->ckpt_every;
    L.n_ckpt = (int)((T + k - 1) / k) + 1;
    L.acc = take(T * ACC_DOUBLES * sizeof(double));
    L.ckpt = take(al256(L.state_floats * 4) * L.n_ckpt);
    L.seg = take(al256(L.state_floats * 4) * (size_t)k);
    L.adj0 = take(L.state_floats * 4);
    L.adj1 = take(L.state_floats * 4);
    L.ub = take(3 * (nc + (nx + 1) * ny * nz + nx * (ny + 1) * nz + nx * ny * (nz + 1)) * 4);
  } else {
    L.n_ckpt = 0;
    L.acc = L.ckpt = L.seg = L.adj0 = L.adj1 = L.ub = 0;
  }
  L.total = o;
  return L;
}

bool levels_ok(const gas_desc* d) {
  if (d->pressure_solver == 0) return true;   // (the spectral solve has no hierarchy)
  const Layout L = plan(d);
  return L.n_grid_levels < L.n_levels;
}

}  // namespace
}  // namespace mpm

using namespace mpm;

struct gas_ctx {
  gas_desc d;
  Layout L;
  GP P;
  hipStream_t stream;
  char* ws;
  std::vector<float> src;
  std::vector<char> act_set;
  gas_state user;
  bool has_state;
  int t;
  bool stats;
  double last_res;
  int last_err_bits;
  HostWord err_host;
  KernelTimer t_adv, t_smooth;
};

namespace {

// a packed state: u, v, w, s consecutive
gas_state packed(gas_ctx* c, char* base) {
  const GP& P = c->P;
  gas_state s;
  s.u = (float*)base;
  s.v = s.u + P.nu;
  s.w = s.v + P.nv;
  s.s = s.w + P.nw;
  return s;
}
size_t state_stride(gas_ctx* c) { return al256(c->L.state_floats * 4); }
const double* pose_at(gas_ctx* c, int t) { return (const double*)(c->ws + c->L.pose) + (size_t)t * POSE_DOUBLES; }

void copy_state(gas_ctx* c, const gas_state& a, const gas_state& b) {
  const GP& P = c->P;
  hipMemcpyAsync(b.u, a.u, P.nu * 4, hipMemcpyDeviceToDevice, c->stream);
  hipMemcpyAsync(b.v, a.v, P.nv * 4, hipMemcpyDeviceToDevice, c->stream);
  hipMemcpyAsync(b.w, a.w, P.nw * 4, hipMemcpyDeviceToDevice, c->stream);
  hipMemcpyAsync(b.s, a.s, (size_t)P.K * P.nc * 4, hipMemcpyDeviceToDevice, c->stream);
}

// A psi = f on level 0 (psi0 holds the initial guess)
void mg_solve(gas_ctx* c, float* psi0, float* f0) {
  const Layout& L = c->L;
  hipStream_t s = c->stream;
  auto psi = [&](int l) { return l == 0 ? psi0 : (float*)(c->ws + L.psi[l]); };
  auto fl = [&](int l) { return l == 0 ? f0 : (float*)(c->ws + L.f[l]); };
  const int G = L.n_grid_levels;
  BottomArgs B;
  B.n_levels = L.n_levels - G;
  for (int l = 0; l < B.n_levels; l++) B.D[l] = L.D[G + l];
  B.psi = psi(G);
  B.f = fl(G);
  auto tiles = [&](int l) {
    const Dims& D = L.D[l];
    return dim3((D.x + TX - 1) / TX, (D.y + TY - 1) / TY, (D.z + TZ - 1) / TZ);
  };
  // V(2,2): red-black sweeps before each restriction, black-red sweeps after
  // each correction (the first of them adds the correction as it stages)
  for (int cyc = 0; cyc < c->d.mg_cycles; cyc++) {
    for (int l = 0; l < G; l++) {
      for (int sw = 0; sw < (l == 0 ? NU0_PRE : 2); sw++) {
        if (l < HALF_LEVELS) {
          for (int color = 0; color < 2; color++) {
            if (l == 0) c->t_smooth.begin(s);
            k_rb_half<<<nblk(L.D[l].cells() / 2, 256), 256, 0, s>>>(psi(l), fl(l), L.D[l], color);
            if (l == 0) c->t_smooth.end(s);
          }
          continue;
        }
        if (l == 0) c->t_smooth.begin(s);
        k_rb_sweep<<<tiles(l), 256, 0, s>>>(psi(l), fl(l), L.D[l], 0, nullptr, L.D[l]);
        if (l == 0) c->t_smooth.end(s);
      }
      k_restrict<<<nblk(L.D[l + 1].cells(), 256), 256, 0, s>>>(psi(l), fl(l), L.D[l], psi(l + 1), fl(l + 1), L.D[l + 1]);
    }
    k_bottom<<<1, BOTTOM_THREADS, 0, s>>>(B);
    for (int l = G - 1; l >= 0; l--) {
      if (l < HALF_LEVELS)
        k_prolong<<<nblk(L.D[l].cells(), 256), 256, 0, s>>>(psi(l + 1), L.D[l + 1], psi(l), L.D[l]);
      for (int sw = 0; sw < (l == 0 ? NU0_POST : NU_POST); sw++) {
        if (l < HALF_LEVELS) {
          for (int color = 1; color >= 0; color--) {
            if (l == 0) c->t_smooth.begin(s);
            k_rb_half<<<nblk(L.D[l].cells() / 2, 256), 256, 0, s>>>(psi(l), fl(l), L.D[l], color);
            if (l == 0) c->t_smooth.end(s);
          }
          continue;
        }
        if (l == 0) c->t_smooth.begin(s);
        k_rb_sweep<<<tiles(l), 256, 0, s>>>(psi(l), fl(l), L.D[l], 1, sw == 0 ? psi(l + 1) : nullptr, L.D[l + 1]);
        if (l == 0) c->t_smooth.end(s);
      }
    }
  }
  if (c->stats) {
    const unsigned nb = min(nblk(L.D[0].cells(), 256), 4096u);
    k_resnorm<<<nb, 256, 0, s>>>(psi0, f0, L.D[0], (double*)(c->ws + L.resp));
    k_resnorm_final<<<1, 64, 0, s>>>((const double*)(c->ws + L.resp), (int)nb, (double*)(c->ws + L.resout));
  }
}

// One launch of transforms: 32 lines a workgroup, two wavefronts per SIMD at 128^3
// (16 lines along z: 11.2 and 15.1 us).  A wavefront takes a pair of output tiles
// at a time; where an axis has more pairs than a workgroup wavefronts and the lines
// alone make fewer than AXIS_FILL workgroups, the pairs are dealt to several
// workgroups of a line (six transforms, us, one workgroup a line and as dealt:
// 8 x 8 x 1024 617 and 87, 64 x 64 x 512 183 and 85, 512 x 64 x 64 167 and 95,
// 256 x 32 x 256 100 and 84, 1024 x 8 x 1024 1515 and 912; with a line at 256
// workgroups 64 x 64 x 512 takes 111, at 1024 256 x 256 x 64 164 instead of 140).
// Every output's sum keeps its order.
constexpr unsigned AXIS_FILL = 512;
struct AxisShape {
  unsigned groups, nw, rounds, split;   // workgroups of lines, wavefronts, rounds of a wavefront, workgroups a line
};
template <int C = 2>
AxisShape axis_shape(int n, int lines, int planes) {
  AxisShape G;
  const unsigned pairs = (unsigned)(axis_steps(n) + AXIS_MT - 1) / AXIS_MT;
  G.groups = (unsigned)((lines + 16 * C - 1) / (16 * C)) * (unsigned)planes;
  G.nw = pairs < 4u ? pairs : 4u;
  G.rounds = (pairs + G.nw - 1) / G.nw;
  const unsigned per = (unsigned)std::max<size_t>(1, (size_t)G.rounds * G.groups / AXIS_FILL);   // rounds a workgroup keeps
  G.split = (G.rounds + per - 1) / per;
  return G;
}
template <bool INNER, int KIND, int C = 2>
void launch_axis(const AxisArgs& X, int lines, int planes, hipStream_t s) {
  const AxisShape G = axis_shape<C>(X.n, lines, planes);
  const size_t lds = KIND == AXIS_BOTH ? (size_t)X.n * 16 * C * 4 : 0;
  const dim3 grid((lines + 16 * C - 1) / (16 * C), planes, KIND == AXIS_BOTH ? 1u : G.split);
  k_axis<INNER, KIND, C><<<grid, 64 * G.nw, lds, s>>>(X);
}

// A psi = f exactly by the axis transforms (psi0 receives the solution with
// zero mean; f0 is left unchanged)
void spectral_solve(gas_ctx* c, float* psi0, const float* f0) {
  const GP& P = c->P;
  hipStream_t s = c->stream;
  float* T = (float*)(c->ws + c->L.spec_tmp);
  const float4* Mf[3] = {(const float4*)(c->ws + c->L.dct[0]), (const float4*)(c->ws + c->L.dct[1]),
                         (const float4*)(c->ws + c->L.dct[2])};
  const float4* Mi[3] = {(const float4*)(c->ws + c->L.idct[0]), (const float4*)(c->ws + c->L.idct[1]),
                         (const float4*)(c->ws + c->L.idct[2])};
  const int nx = P.nx, ny = P.ny, nz = P.nz;
  auto args = [&](const float* in, float* out, const float4* M, int n, int A, int B) {
    AxisArgs X = {};
    X.in = in; X.out = out; X.M = M; X.n = n; X.A = A; X.B = B;
    return X;
  };
  // one event pair around the back-to-back transforms (read as six): a pair
  // per launch would add its own overhead to each
  c->t_smooth.begin(s);
  launch_axis<true, AXIS_ONE>(args(f0, T, Mf[2], nz, nx * ny, 1), nx * ny, 1, s);
  launch_axis<false, AXIS_ONE>(args(T, psi0, Mf[1], ny, nx, nz), nz, nx, s);
  // along x in place: every workgroup has read its lines when it writes them
  // (with more than 512 values an axis does not fit the 64 KB of a workgroup's
  // coefficients, and where the output tiles have to be dealt to several workgroups
  // none of them has all coefficients: two launches)
  const bool both = nx <= 512 && axis_shape(nx, ny * nz, 1).split == 1u;
  AxisArgs X = args(psi0, both ? psi0 : T, Mf[0], nx, 1, ny * nz);
  X.M2 = Mi[0];
  X.lx = (const float*)(c->ws + c->L.lam[0]);
  X.ly = (const float*)(c->ws + c->L.lam[1]);
  X.lz = (const float*)(c->ws + c->L.lam[2]);
  X.nz = nz;
  if (both) {
    launch_axis<false, AXIS_BOTH>(X, ny * nz, 1, s);
  } else {
    launch_axis<false, AXIS_ONE>(X, ny * nz, 1, s);
    launch_axis<false, AXIS_ONE>(args(T, psi0, Mi[0], nx, 1, ny * nz), ny * nz, 1, s);
  }
  launch_axis<false, AXIS_ONE>(args(psi0, T, Mi[1], ny, nx, nz), nz, nx, s);
  launch_axis<true, AXIS_ONE>(args(T, psi0, Mi[2], nz, nx * ny, 1), nx * ny, 1, s);
  c->t_smooth.end(s);
}

void pressure_solve(gas_ctx* c, float* psi0, float* f0) {
  if (c->d.pressure_solver != 0) {
    mg_solve(c, psi0, f0);
    return;
  }
  spectral_solve(c, psi0, f0);
  if (c->stats) {
    const Layout& L = c->L;
    const unsigned nb = min(nblk(L.D[0].cells(), 256), 4096u);
    k_resnorm<<<nb, 256, 0, c->stream>>>(psi0, f0, L.D[0], (double*)(c->ws + L.resp));
    k_resnorm_final<<<1, 64, 0, c->stream>>>((const double*)(c->ws + L.resp), (int)nb, (double*)(c->ws + L.resout));
  }
}

// one forward step from `in` to `out` (their scalars distinct), emitter at pose t
void gas_forward_step(gas_ctx* c, const gas_state& in, const gas_state& out, int t) {
  const GP& P = c->P;
  hipStream_t s = c->stream;
  gas_state tmp = packed(c, c->ws + c->L.tmp);
  float* psi0 = (float*)(c->ws + c->L.psi[0]);
  float* f0 = (float*)(c->ws + c->L.f[0]);
  c->t_adv.begin(s);
  const PointGrid Ga = point_grid(P, 4, ADV_U), Gd = point_grid(P, 1, DIV_U), Gf = point_grid(P, 3, FIN_U);
  k_gas_advect<<<Ga.blocks, 256, 0, s>>>(P, VelPtrs{in.u, in.v, in.w}, in.s, tmp.u, tmp.v, tmp.w, out.s,
                                        pose_at(c, t), Ga);
  c->t_adv.end(s);
  k_gas_div<true><<<Gd.blocks, 256, 0, s>>>(P, tmp.u, tmp.v, tmp.w, out.s, f0, c->d.pressure_solver ? psi0 : nullptr, Gd);
  pressure_solve(c, psi0, f0);
  k_gas_final<true><<<Gf.blocks, 256, 0, s>>>(P, tmp.u, tmp.v, tmp.w, out.s, psi0, out.u, out.v, out.w, Gf);
}

// one adjoint step: abar_next (adjoint of s_{t+1}) -> abar (adjoint of s_t);
// st is s_t
void gas_adjoint_step(gas_ctx* c, const gas_state& st, const gas_state& an, const gas_state& ab, int t, double* acc_t) {
  const GP& P = c->P;
  hipStream_t s = c->stream;
  gas_state tmp = packed(c, c->ws + c->L.tmp);
  float* psi0 = (float*)(c->ws + c->L.psi[0]);
  float* f0 = (float*)(c->ws + c->L.f[0]);
  const PointGrid Gd = point_grid(P, 1, DIV_U), Gf = point_grid(P, 3, FIN_U), G1 = column_grid(P, 1), Gu = point_grid(P, 3, UG_U);
  k_gas_div<false><<<Gd.blocks, 256, 0, s>>>(P, an.u, an.v, an.w, nullptr, f0, c->d.pressure_solver ? psi0 : nullptr, Gd);
  pressure_solve(c, psi0, f0);
  k_gas_final<false><<<Gf.blocks, 256, 0, s>>>(P, an.u, an.v, an.w, nullptr, psi0, tmp.u, tmp.v, tmp.w, Gf);
  launch_zero(ab.u, c->L.state_floats * 4, s);
  const bool one = G1.blocks <= ADJ_SHORT_BLOCKS;
  const PointGrid Ga = one ? G1 : column_grid(P, ADJ_J);
  (one ? k_gas_adj_advect<1> : k_gas_adj_advect<ADJ_J>)<<<Ga.blocks, 64 * ADJ_I, 0, s>>>(
      P, VelPtrs{st.u, st.v, st.w}, st.s, tmp.u, tmp.v, tmp.w, an.s, AdjOut{ab.u, ab.v, ab.w, ab.s}, pose_at(c, t),
      (double*)(c->ws + c->L.slots), (float*)(c->ws + c->L.ub), Ga);
  k_gas_adj_ugather<<<Gu.blocks, 256, 0, s>>>(P, (const float*)(c->ws + c->L.ub), AdjOut{ab.u, ab.v, ab.w, ab.s}, Gu);
  k_gas_pose_acc<<<1, 64, 0, s>>>((double*)(c->ws + c->L.slots), acc_t);
}

// Waits for the call's work; reads (and clears) the device error word.
int sync_ok(gas_ctx* c) {
  if (hipMemcpyAsync(c->err_host.p, c->ws + c->L.err, sizeof(int), hipMemcpyDeviceToHost, c->stream) != hipSuccess)
    return MPM_EHIP;
  if (hipStreamSynchronize(c->stream) != hipSuccess) return MPM_EHIP;
  if (hipGetLastError() != hipSuccess) return MPM_EHIP;
  c->t_adv.collect();
  c->t_smooth.collect();
  if (c->stats) {
    double r = 0.0;
    if (hipMemcpy(&r, c->ws + c->L.resout, sizeof(double), hipMemcpyDeviceToHost) != hipSuccess) return MPM_EHIP;
    c->last_res = r;
  }
  if (const int bits = *c->err_host.p) {
    c->last_err_bits = bits;
    if (hipMemsetAsync(c->ws + c->L.err, 0, sizeof(int), c->stream) != hipSuccess) return MPM_EHIP;
    if (hipStreamSynchronize(c->stream) != hipSuccess) return MPM_EHIP;
    return MPM_EDOMAIN;
  }
  return MPM_OK;
}

}  // namespace

extern "C" {

size_t gas_workspace_bytes(const gas_desc* d) {
  if (!desc_ok(d) || !levels_ok(d)) return 0;
  return plan(d).total;
}

int gas_create(const gas_desc* d, void* workspace_dev, size_t ws_bytes, void* stream, gas_ctx** out) {
  if (!out) return MPM_EINVAL;
  *out = nullptr;
  if (!desc_ok(d) || !levels_ok(d) || !workspace_dev || ((uintptr_t)workspace_dev % 256)) return MPM_EINVAL;
  Layout L = plan(d);
  if (ws_bytes < L.total) return MPM_EWORKSPACE;
  gas_ctx* c = new (std::nothrow) gas_ctx();
  if (!c) return MPM_EINVAL;
  c->d = *d;
  c->src.assign(d->src, d->src + d->n_scalars);
  c->d.src = c->src.data();
  c->L = L;
  c->stream = (hipStream_t)stream;
  c->ws = (char*)workspace_dev;
  c->has_state = false;
  c->t = 0;
  c->stats = false;
  c->last_res = 0.0;
  c->last_err_bits = 0;
  c->t_adv.name = "k_gas_advect";
  c->t_smooth.name = d->pressure_solver == 0 ? "k_axis" : "k_rb_half";
  c->act_set.assign(d->horizon, 0);
  GP& P = c->P;
  P.nx = d->nx; P.ny = d->ny; P.nz = d->nz; P.K = d->n_scalars;
  P.h = d->h; P.inv_h = 1.f / d->h; P.dt = d->dt; P.beta = d->buoyancy; P.t_amb = d->t_amb;
  P.s2inv = 1.f / (2.f * d->emit_sigma * d->emit_sigma);
  P.kappa = d->emit_kappa;
  P.speed = d->emit_speed;
  for (int k = 0; k < MAXK; k++) P.src[k] = k < d->n_scalars ? d->src[k] : 0.f;
  P.nu = (size_t)(d->nx + 1) * d->ny * d->nz;
  P.nv = (size_t)d->nx * (d->ny + 1) * d->nz;
  P.nw = (size_t)d->nx * d->ny * (d->nz + 1);
  P.nc = (size_t)d->nx * d->ny * d->nz;
  P.big = P.nu >= (1u << 30) || P.nv >= (1u << 30) || P.nw >= (1u << 30);
  P.mz = (uint32_t)((0x100000000ull + d->nz - 1) / d->nz);
  P.mz1 = (uint32_t)((0x100000000ull + d->nz) / (d->nz + 1));
  P.err = (int*)(c->ws + L.err);
  launch_zero(c->ws + L.slots, SLOTS * POSE_PARTIALS * sizeof(double), c->stream);
  launch_zero(c->ws + L.err, 64, c->stream);
  // spectral tables: per axis the DCT-II matrix C[i][k] = cos(pi k (i + 1/2) / n),
  // its inverse Ci[k][i] = w_k C[i][k] (w_0 = 1/n, w_k = 2/n) and the 1-D
  // Neumann eigenvalues -4 sin^2(pi k / 2n), computed in FP64
  {
    const int nn[3] = {d->nx, d->ny, d->nz};
    for (int a = 0; a < 3; a++) {
      const int n = nn[a];
      // as fragments [output tile][step][lane (lr, lc)][t]: term 16 step + 4 t + lr,
      // output 16 tile + lc (forward: terms i, outputs k; inverse: terms k, outputs
      // i); zero past n.  Every cosine is computed once, for its place in both
      // (computed for each, a room with an axis of 1024 took 20 ms to create, not 11).
      const int st = axis_steps(n);
      auto place = [](int o, int term) { return ((term & 3) * 16 + o) * 4 + (term >> 2); };
      std::vector<float> C((size_t)st * st * 256, 0.f), Ci(C.size(), 0.f), lam(n);
      for (int kt = 0; kt < st; kt++)
        for (int it = 0; it < st; it++) {
          float* f = C.data() + ((size_t)kt * st + it) * 256;
          float* fi = Ci.data() + ((size_t)it * st + kt) * 256;
          for (int dk = 0; dk < 16 && 16 * kt + dk < n; dk++)
            for (int di = 0; di < 16 && 16 * it + di < n; di++) {
              const int k = 16 * kt + dk, i = 16 * it + di;
              const double v = cos(M_PI * k * (i + 0.5) / n);
              f[place(dk, di)] = (float)v;
              fi[place(di, dk)] = (float)(v * (k == 0 ? 1.0 / n : 2.0 / n));
            }
        }
      for (int k = 0; k < n; k++) {
        const double sk = sin(M_PI * k / (2.0 * n));
        lam[k] = (float)(-4.0 * sk * sk);
      }
      if (hipMemcpy(c->ws + L.dct[a], C.data(), C.size() * 4, hipMemcpyHostToDevice) != hipSuccess ||
          hipMemcpy(c->ws + L.idct[a], Ci.data(), Ci.size() * 4, hipMemcpyHostToDevice) != hipSuccess ||
          hipMemcpy(c->ws + L.lam[a], lam.data(), lam.size() * 4, hipMemcpyHostToDevice) != hipSuccess) {
        delete c;
        return MPM_EHIP;
      }
    }
  }
  // the emitter's pose at t = 0: its slot is written here only
  double pose0[POSE_DOUBLES];
  for (int k = 0; k < 3; k++) pose0[k] = c->d.emit_pos0[k];
  for (int k = 0; k < 9; k++) pose0[3 + k] = c->d.emit_rot0[k];
  if (!c->err_host.create() ||
      hipMemcpyAsync(c->ws + c->L.pose, pose0, sizeof(pose0), hipMemcpyHostToDevice, c->stream) != hipSuccess ||
      hipStreamSynchronize(c->stream) != hipSuccess || hipGetLastError() != hipSuccess) {
    c->err_host.destroy();
    delete c;
    return MPM_EHIP;
  }
  *out = c;
  return MPM_OK;
}

int gas_set_state(gas_ctx* c, const gas_state* st) {
  if (!c || !st || !st->u || !st->v || !st->w || !st->s) return MPM_EINVAL;
  c->user = *st;
  c->has_state = true;
  c->t = 0;
  return MPM_OK;
}

int gas_set_actions(gas_ctx* c, int32_t t0, int32_t n, const float* actions_dev) {
  if (!c || !actions_dev || t0 < 0 || n < 1 || t0 + n > c->d.horizon) return MPM_EINVAL;
  if (hipMemcpyAsync(c->ws + c->L.act + (size_t)t0 * 6 * sizeof(float), actions_dev, (size_t)n * 6 * sizeof(float),
                     hipMemcpyDeviceToDevice, c->stream) != hipSuccess)
    return MPM_EHIP;
  for (int t = t0; t < t0 + n; t++) c->act_set[t] = 1;
  return MPM_OK;
}

int gas_step(gas_ctx* c, int32_t n_steps) {
  if (!c || n_steps < 0) return MPM_EINVAL;
  if (!c->has_state) return MPM_ESTATE;
  if (n_steps == 0) return MPM_OK;
  if (c->t + n_steps > c->d.horizon) return MPM_EINVAL;
  for (int t = c->t; t < c->t + n_steps; t++)
    if (!c->act_set[t]) return MPM_ESTATE;
  launch_pose(1, c->t, n_steps, c->d.dt, (const float*)(c->ws + c->L.act), (double*)(c->ws + c->L.pose), c->stream);
  // the step reads the user's velocities and writes them back through the
  // temporaries; the scalars, which advection finishes, alternate between the
  // user array and the temporaries', so that the last step ends in the user's
  // (an odd number of steps starts from a copy); a checkpoint is taken before
  // every k-th step
  gas_state from = c->user, to = c->user;
  float* tmp_s = packed(c, c->ws + c->L.tmp).s;
  if (n_steps & 1) {
    hipMemcpyAsync(tmp_s, from.s, (size_t)c->P.K * c->P.nc * 4, hipMemcpyDeviceToDevice, c->stream);
    from.s = tmp_s;
  } else {
    to.s = tmp_s;
  }
  for (int t = c->t; t < c->t + n_steps; t++) {
    if (c->d.requires_grad && t % c->d.ckpt_every == 0)
      copy_state(c, from, packed(c, c->ws + c->L.ckpt + (size_t)(t / c->d.ckpt_every) * state_stride(c)));
    gas_forward_step(c, from, to, t);
    float* sw = from.s; from.s = to.s; to.s = sw;
  }
  c->t += n_steps;
  if (hipGetLastError() != hipSuccess) return MPM_EHIP;
  return sync_ok(c);
}

int gas_step_backward(gas_ctx* c, const gas_state* grad_T, float* grad_actions_dev, gas_state* grad_0) {
  if (!c || !grad_T || !grad_T->u || !grad_T->v || !grad_T->w || !grad_actions_dev) return MPM_EINVAL;
  if (!c->has_state || !c->d.requires_grad || c->t < 1) return MPM_ESTATE;
  if (grad_0 && (!grad_0->u || !grad_0->v || !grad_0->w || !grad_0->s)) return MPM_EINVAL;
  const GP& P = c->P;
  hipStream_t s = c->stream;
  const int T = c->t, k = c->d.ckpt_every;
  gas_state a_cur = packed(c, c->ws + c->L.adj0), a_nxt = packed(c, c->ws + c->L.adj1);
  launch_zero(a_cur.u, c->L.state_floats * 4, s);
  hipMemcpyAsync(a_cur.u, grad_T->u, P.nu * 4, hipMemcpyDeviceToDevice, s);
  hipMemcpyAsync(a_cur.v, grad_T->v, P.nv * 4, hipMemcpyDeviceToDevice, s);
  hipMemcpyAsync(a_cur.w, grad_T->w, P.nw * 4, hipMemcpyDeviceToDevice, s);
  if (grad_T->s) hipMemcpyAsync(a_cur.s, grad_T->s, (size_t)P.K * P.nc * 4, hipMemcpyDeviceToDevice, s);
  double* acc = (double*)(c->ws + c->L.acc);
  launch_zero(acc, al256((size_t)T * ACC_DOUBLES * sizeof(double)), s);
  const int n_seg = (T + k - 1) / k;
  for (int seg = n_seg - 1; seg >= 0; seg--) {
    const int ts = seg * k, te = ts + k < T ? ts + k : T;
    // recompute s_ts .. s_{te-1} into the segment slots
    copy_state(c, packed(c, c->ws + c->L.ckpt + (size_t)seg * state_stride(c)), packed(c, c->ws + c->L.seg));
    for (int t = ts; t + 1 < te; t++)
      gas_forward_step(c, packed(c, c->ws + c->L.seg + (size_t)(t - ts) * state_stride(c)),
                       packed(c, c->ws + c->L.seg + (size_t)(t - ts + 1) * state_stride(c)), t);
    for (int t = te - 1; t >= ts; t--) {
      gas_adjoint_step(c, packed(c, c->ws + c->L.seg + (size_t)(t - ts) * state_stride(c)), a_cur, a_nxt, t,
                       acc + (size_t)t * ACC_DOUBLES);
      gas_state sw = a_cur; a_cur = a_nxt; a_nxt = sw;
    }
  }
  launch_pose_adj(1, T, c->d.dt, (const float*)(c->ws + c->L.act), (const double*)(c->ws + c->L.pose), acc,
                  grad_actions_dev, s);
  if (grad_0) copy_state(c, a_cur, *grad_0);
  if (hipGetLastError() != hipSuccess) return MPM_EHIP;
  return sync_ok(c);
}

int gas_sensor_loss(gas_ctx* c, int32_t n, const int32_t* cells_dev, const float* targets_dev, float* loss_dev,
                    gas_state* grad_out) {
  if (!c || n < 1 || !cells_dev || !targets_dev || !loss_dev) return MPM_EINVAL;
  if (!c->has_state) return MPM_ESTATE;
  const GP& P = c->P;
  float* gT = nullptr;
  if (grad_out) {
    if (!grad_out->u || !grad_out->v || !grad_out->w || !grad_out->s) return MPM_EINVAL;
    hipMemsetAsync(grad_out->u, 0, P.nu * 4, c->stream);
    hipMemsetAsync(grad_out->v, 0, P.nv * 4, c->stream);
    hipMemsetAsync(grad_out->w, 0, P.nw * 4, c->stream);
    hipMemsetAsync(grad_out->s, 0, (size_t)P.K * P.nc * 4, c->stream);
    gT = grad_out->s;
  }
  k_gas_sensors<<<1, 256, 0, c->stream>>>(c->user.s, P.nc, n, cells_dev, targets_dev, loss_dev, gT);
  if (hipGetLastError() != hipSuccess) return MPM_EHIP;
  return sync_ok(c);
}

int gas_enable_stats(gas_ctx* c, int32_t enable) {
  if (!c) return MPM_EINVAL;
  c->stats = enable != 0;
  return MPM_OK;
}

int gas_solver_residual(gas_ctx* c, double* rel_residual) {
  if (!c || !rel_residual) return MPM_EINVAL;
  *rel_residual = c->last_res;
  return MPM_OK;
}

int gas_timing_enable(gas_ctx* c, int32_t enable) {
  if (!c) return MPM_EINVAL;
  c->t_adv.on = c->t_smooth.on = enable != 0;
  c->t_adv.total_ms = c->t_smooth.total_ms = 0.0;
  c->t_adv.launches = c->t_smooth.launches = 0;
  c->t_adv.used = c->t_smooth.used = 0;
  return MPM_OK;
}

int gas_timing_read(gas_ctx* c, double* advect_ms, int64_t* advect_launches, double* smooth_ms,
                    int64_t* smooth_launches) {
  if (!c || !advect_ms || !advect_launches || !smooth_ms || !smooth_launches) return MPM_EINVAL;
  *advect_ms = c->t_adv.total_ms;
  *advect_launches = c->t_adv.launches;
  *smooth_ms = c->t_smooth.total_ms;
  *smooth_launches = c->t_smooth.launches * (c->d.pressure_solver == 0 ? 6 : 1);
  c->t_adv.total_ms = c->t_smooth.total_ms = 0.0;
  c->t_adv.launches = c->t_smooth.launches = 0;
  return MPM_OK;
}

int gas_last_error_bits(const gas_ctx* c, int32_t* bits_out) {
  if (!c || !bits_out) return MPM_EINVAL;
  *bits_out = c->last_err_bits;
  return MPM_OK;
}

int gas_clock(const gas_ctx* c, int32_t* t_out) {
  if (!c || !t_out) return MPM_EINVAL;
  *t_out = c->t;
  return MPM_OK;
}

int gas_destroy(gas_ctx* c) {
  if (!c) return MPM_EINVAL;
  c->t_adv.destroy();
  c->t_smooth.destroy();
  c->err_host.destroy();
  delete c;
  return MPM_OK;
}

}  // extern "C"
