// Sums over the 27 nodes of a particle's quadratic B-spline stencil, read
// from a tile of nodes staged in LDS (a block's 8^3 velocity tile with the
// padded strides VT_ROW and VT_PLANE, or one particle's own 3^3 stencil; lb =
// the stencil's first node in the tile), shared by the forward and adjoint
// transfer kernels.
//
// Both sums run over z inside y inside x, so that each partial sum is
// weighted once by the outer weights (w = wx wy wz factorises); the loads of
// one x plane are issued together, and a compiler barrier between planes
// keeps the next plane's loads from being hoisted (nine loads in flight
// rather than 27 bounds the register count).
#pragma once
#include <hip/hip_runtime.h>
#include "mpm_blocks.h"
#include "mpm_fast.h"
#include "mpm_phys.h"

namespace mpm {

// multiplier m with r / d = (r m) >> 20 for r d < 2^19 (2^20 / d < m <= 2^20 / d + 2)
__device__ __forceinline__ uint32_t div_mul(int d) {
  return (uint32_t)(1048576.f * __builtin_amdgcn_rcpf((float)d)) + 2u;
}

// A block's 8^3 window of node values (nodes 4 b - 1 .. 4 b + 6 per axis; zero
// outside the grid) from a block-layout array into LDS, by NT threads.  The
// window spans three blocks per axis, whose key parts are wavefront-uniform:
// spreading each node's own block coordinates cost about 45 vector
// instructions a node.
template <int NT>
__device__ __forceinline__ void stage_window(float4* __restrict__ tile, const float4* __restrict__ src,
                                             const FastGeom& g, int sc, int bx, int by, int bz, int tid) {
  const uint32_t base = (uint32_t)sc << (3 * g.kb);
  const uint32_t kx[3] = {spread3(bx - 1) << 2, spread3(bx) << 2, spread3(bx + 1) << 2};
  const uint32_t ky[3] = {spread3(by - 1) << 1, spread3(by) << 1, spread3(by + 1) << 1};
  const uint32_t kz[3] = {spread3(bz - 1), spread3(bz), spread3(bz + 1)};
  constexpr int R = (VT_NODES + NT - 1) / NT;
  float4 val[R];
#pragma unroll
  for (int r = 0; r < R; r++) {
    const int q = tid + r * NT;
    const int qi = q / (VT * VT), qj = (q / VT) % VT, qk = q % VT;
    const int gx = 4 * bx - 1 + qi, gy = 4 * by - 1 + qj, gz = 4 * bz - 1 + qk;
    val[r] = make_float4(0.f, 0.f, 0.f, 0.f);
    if (q < VT_NODES && gx >= 0 && gy >= 0 && gz >= 0 && gx < g.n && gy < g.n && gz < g.n) {
      // window node 0 lies in the block before, 1..4 in the block, 5..7 after
      const uint32_t kk = base | (qi == 0 ? kx[0] : (qi < 5 ? kx[1] : kx[2])) |
                          (qj == 0 ? ky[0] : (qj < 5 ? ky[1] : ky[2])) | (qk == 0 ? kz[0] : (qk < 5 ? kz[1] : kz[2]));
      val[r] = src[(size_t)kk * 64 + ((((qi + 3) & 3) << 4) | (((qj + 3) & 3) << 2) | ((qk + 3) & 3))];
    }
  }
#pragma unroll
  for (int r = 0; r < R; r++) {
    const int q = tid + r * NT;
    if (q < VT_NODES) tile[(q / (VT * VT)) * VT_PLANE + ((q / VT) % VT) * VT_ROW + q % VT] = val[r];
  }
}

// G2P gather: vn = sum_i w_i v_i and Bi = sum_i w_i v_i idx_i^T with idx_i
// in {0,1,2}^3 the node's offset in the stencil (v_i = the tile's xyz).
template <int ROW = VT_ROW, int PLANE = VT_PLANE>
__device__ __forceinline__ void g2p_gather(const float4* __restrict__ s_v, const int* lb, const Stencil& S,
                                           float* vn, float* Bi) {
#pragma unroll
  for (int q = 0; q < 3; q++) vn[q] = 0.f;
#pragma unroll
  for (int q = 0; q < 9; q++) Bi[q] = 0.f;
  const float wz1 = S.w[2][1], wz2 = S.w[2][2], wz2x2 = 2.f * S.w[2][2];
#pragma unroll
  for (int i = 0; i < 3; i++) {
    float p0[3] = {0, 0, 0}, pj[3] = {0, 0, 0}, pk[3] = {0, 0, 0};
#pragma unroll
    for (int jj = 0; jj < 3; jj++) {
      const float4* row = s_v + (lb[0] + i) * PLANE + (lb[1] + jj) * ROW + lb[2];
      const float4 g0 = row[0], g1 = row[1], g2 = row[2];
      // r = sum_k w_k v_k, rk = sum_k k w_k v_k along z
      const float r[3] = {S.w[2][0] * g0.x + wz1 * g1.x + wz2 * g2.x, S.w[2][0] * g0.y + wz1 * g1.y + wz2 * g2.y,
                          S.w[2][0] * g0.z + wz1 * g1.z + wz2 * g2.z};
      const float rk[3] = {wz1 * g1.x + wz2x2 * g2.x, wz1 * g1.y + wz2x2 * g2.y, wz1 * g1.z + wz2x2 * g2.z};
      const float wy = S.w[1][jj];
#pragma unroll
      for (int a = 0; a < 3; a++) {
        p0[a] += wy * r[a];
        if (jj) pj[a] += ((float)jj * wy) * r[a];
        pk[a] += wy * rk[a];
      }
    }
    const float wx = S.w[0][i];
#pragma unroll
    for (int a = 0; a < 3; a++) {
      vn[a] += wx * p0[a];
      if (i) Bi[a * 3 + 0] += ((float)i * wx) * p0[a];
      Bi[a * 3 + 1] += wx * pj[a];
      Bi[a * 3 + 2] += wx * pk[a];
    }
    asm volatile("" ::: "memory");
  }
}

// The weight-gradient sum of the transfers' adjoints:
//   X = sum_i (dw_x wy wz, wx dw_y wz, wx wy dw_z)_i s_i  (dw = dw/df; the
//   caller divides by dx), with s_i = mw g_i.w + g_i.xyz . (c0 + Ad idx_i)
// for the tile's values g_i (the term affine in the node offset is the
// adjoint of the node's momentum, mom = mvp + A (x_i - x_p), or of the G2P
// terms v_i (vbt + Bb (x_i - x_p)), written as c0 + Ad idx).  With WANT_G it
// also returns G0 = sum_i w_i g_i.xyz and Gi = sum_i w_i g_i.xyz idx_i^T.
template <bool WANT_G, int ROW = VT_ROW, int PLANE = VT_PLANE>
__device__ __forceinline__ void weight_grad_sum(const float4* __restrict__ tile, const int* lb, const Stencil& S,
                                                const float* c0, const float* Ad, float mw, float* X, float* G0,
                                                float* Gi) {
#pragma unroll
  for (int a = 0; a < 3; a++) X[a] = 0.f;
  if (WANT_G) {
#pragma unroll
    for (int q = 0; q < 3; q++) G0[q] = 0.f;
#pragma unroll
    for (int q = 0; q < 9; q++) Gi[q] = 0.f;
  }
#pragma unroll
  for (int i = 0; i < 3; i++) {
    float m1[3];
#pragma unroll
    for (int a = 0; a < 3; a++) m1[a] = c0[a] + (float)i * Ad[a * 3];
    float Px = 0.f, Py = 0.f, Pz = 0.f;
    float p0[3] = {0, 0, 0}, pj[3] = {0, 0, 0}, pk[3] = {0, 0, 0};
#pragma unroll
    for (int jj = 0; jj < 3; jj++) {
      const float4* row = tile + (lb[0] + i) * PLANE + (lb[1] + jj) * ROW + lb[2];
      const float4 g[3] = {row[0], row[1], row[2]};
      float m2[3];
#pragma unroll
      for (int a = 0; a < 3; a++) m2[a] = m1[a] + (float)jj * Ad[a * 3 + 1];
      float sk[3];
#pragma unroll
      for (int k = 0; k < 3; k++) {
        const float u0 = m2[0] + (float)k * Ad[2], u1 = m2[1] + (float)k * Ad[5], u2 = m2[2] + (float)k * Ad[8];
        sk[k] = g[k].x * u0 + g[k].y * u1 + g[k].z * u2;
        if (mw != 0.f) sk[k] += mw * g[k].w;
      }
      // z sums: with w_z and with dw_z
      const float R0 = S.w[2][0] * sk[0] + S.w[2][1] * sk[1] + S.w[2][2] * sk[2];
      const float R1 = S.dw[2][0] * sk[0] + S.dw[2][1] * sk[1] + S.dw[2][2] * sk[2];
      const float wy = S.w[1][jj], dwy = S.dw[1][jj];
      Px += wy * R0;
      Py += dwy * R0;
      Pz += wy * R1;
      if (WANT_G) {
        const float r[3] = {S.w[2][0] * g[0].x + S.w[2][1] * g[1].x + S.w[2][2] * g[2].x,
                            S.w[2][0] * g[0].y + S.w[2][1] * g[1].y + S.w[2][2] * g[2].y,
                            S.w[2][0] * g[0].z + S.w[2][1] * g[1].z + S.w[2][2] * g[2].z};
        const float wz22 = 2.f * S.w[2][2];
        const float rk[3] = {S.w[2][1] * g[1].x + wz22 * g[2].x, S.w[2][1] * g[1].y + wz22 * g[2].y,
                             S.w[2][1] * g[1].z + wz22 * g[2].z};
#pragma unroll
        for (int a = 0; a < 3; a++) {
          p0[a] += wy * r[a];
          if (jj) pj[a] += ((float)jj * wy) * r[a];
          pk[a] += wy * rk[a];
        }
      }
    }
    const float wx = S.w[0][i], dwx = S.dw[0][i];
    X[0] += dwx * Px;
    X[1] += wx * Py;
    X[2] += wx * Pz;
    if (WANT_G) {
#pragma unroll
      for (int a = 0; a < 3; a++) {
        G0[a] += wx * p0[a];
        if (i) Gi[a * 3 + 0] += ((float)i * wx) * p0[a];
        Gi[a * 3 + 1] += wx * pj[a];
        Gi[a * 3 + 2] += wx * pk[a];
      }
    }
    asm volatile("" ::: "memory");
  }
}

// Sum of the published tiles over the 64 nodes of block (cx, cy, cz), one node
// per lane of the wavefront: acc += the tiles' float4 words.  Each lane reads
// one or two of the neighbours' boxes and turns it into the block's nodes that
// it covers; the tiles that cover any (about a third of the 27) are then added
// eight loads at a time.  (All 27 neighbours in turn, box by box through LDS
// permutes, cost about 800 vector instructions a block, and each second tile a
// round trip of its own: k_grid 9.8 us at 250k particles on 128^3, now 6.7,
// 35.9 at 1M on 256^3, now 22.0.)
__device__ __forceinline__ void sum_tiles(const FastGeom& g, int sc, int cx, int cy, int cz, int lane,
                                          const int4* __restrict__ tile_box, const float* __restrict__ tiles,
                                          uint32_t stamp, float4& acc) {
  // this lane's neighbour (lanes 0..26: its entries 0, 2, .., lanes 32..58: 1, 3, ..)
  const int dl = lane & 31, half = lane >> 5;
  const int dx = dl / 9 - 1, dy = (dl / 3) % 3 - 1, dz = dl % 3 - 1;
  const int sx = cx + dx, sy = cy + dy, sz = cz + dz;
  const bool nb = dl < 27 && sx >= 0 && sy >= 0 && sz >= 0 && sx < g.nb && sy < g.nb && sz < g.nb;
  const int4* boxes = tile_box + (size_t)(nb ? block_key(g, sc, sx, sy, sz) : 0u) * NSUB;
  // the lane's node as one bit per axis, and its offset in the tile of the block
  const int li = lane >> 4, lj = (lane >> 2) & 3, lk = lane & 3;
  const int node = (1 << li) | (16 << lj) | (256 << lk);
  const int q0 = (li * TILE + lj) * TILE + lk;
  // neighbour tile coordinates of the block's first node
  const int ax = 2 - 4 * dx, ay = 2 - 4 * dy, az = 2 - 4 * dz;
  const int qn = (ax * TILE + ay) * TILE + az;
  auto span = [](int lo, int hi) -> int {   // bits max(lo, 0) .. min(hi, 3)
    lo = max(lo, 0);
    hi = min(hi, 3);
    return hi >= lo ? (2 << hi) - (1 << lo) : 0;
  };
  auto cover = [&](const int4& b, bool on) -> int {
    if (!on || (uint32_t)b.y != stamp) return 0;
    const int m0 = span((b.x & 15) - ax, ((b.x >> 12) & 15) - ax);
    const int m1 = span(((b.x >> 4) & 15) - ay, ((b.x >> 16) & 15) - ay);
    const int m2 = span(((b.x >> 8) & 15) - az, ((b.x >> 20) & 15) - az);
    return (m0 && m1 && m2) ? (m0 | (m1 << 4) | (m2 << 8)) : 0;
  };
  auto add = [&](int cov, int slot) {
    unsigned long long m = __ballot(cov != 0);
    while (m) {
      constexpr int G = 8;
      float4 tv[G];
      bool in[G];
#pragma unroll
      for (int u = 0; u < G; u++) {
        const int src = m ? __ffsll((long long)m) - 1 : 63;   // (lane 63 covers nothing)
        m &= m - 1ull;
        const int c = __builtin_amdgcn_readlane(cov, src);
        const int q = __builtin_amdgcn_readlane(qn, src);
        const uint32_t sl = (uint32_t)__builtin_amdgcn_readlane(slot, src);
        in[u] = (node & ~c) == 0;
        const uint32_t off = in[u] ? (uint32_t)(q0 + q) : 0u;
        tv[u] = reinterpret_cast<const float4*>(tiles + (size_t)sl * 4 * TILE_NODES)[off];
      }
#pragma unroll
      for (int u = 0; u < G; u++) {
        acc.x += in[u] ? tv[u].x : 0.f;
        acc.y += in[u] ? tv[u].y : 0.f;
        acc.z += in[u] ? tv[u].z : 0.f;
        acc.w += in[u] ? tv[u].w : 0.f;
      }
    }
  };
  int4 b = make_int4(0, 0, 0, 0);
  if (nb) b = boxes[half];
  const int c = cover(b, nb);
  const int slot = c ? b.z : 0;
  const int extra = (nb && (uint32_t)b.y == stamp) ? (b.x >> 24) & 7 : 0;
  const int ex = max(extra, __shfl_xor(extra, 32));
  const bool more = __ballot(ex > 1) != 0ull;
  // (the boxes of entries 2 and up are loaded together, ahead of the first sums)
  constexpr int NP = NSUB / 2 - 1;
  int4 b2[NP];
#pragma unroll
  for (int r = 0; r < NP; r++) {
    b2[r] = make_int4(0, 0, 0, 0);
    if (more && nb && ex >= 2 * r + 2 + half) b2[r] = boxes[2 * r + 2 + half];
  }
  add(c, slot);   // (lane order: entry 0 of every neighbour first, then their entries 1)
  if (more) {
#pragma unroll
    for (int r = 0; r < NP; r++) {
      const int c2 = cover(b2[r], nb && ex >= 2 * r + 2 + half);
      add(c2, c2 ? b2[r].z : 0);
    }
  }
}

}  // namespace mpm
