// Tiled adjoint of the MLS-MPM step for gfx950 (FluidLab section 3.3 and
// App. A: the gradient of a loss through the rollout by reverse-mode
// differentiation, with checkpoints recomputed segment by segment).
//
// Every state of a recomputed segment is kept sorted by the 4^3 block key of
// its own positions, so that the particles of one block sit in contiguous
// rows, like the forward path's.  The adjoint of step t (state s_t -> s_{t+1})
// then runs on s_t's blocks:
//   fast_p2g, fast_grid   recompute the grid of step t: node momenta and
//                         masses (block layout) and the updated velocities
//   k_g2p_adj_tiled       one workgroup per occupied block: G2P recomputed
//                         from an LDS copy of the velocities, the adjoint of
//                         the particle update, and the scatter of the
//                         velocity adjoint into a fixed-point LDS tile whose
//                         non-zero box is published (no global float atomics)
//   k_grid_adj_tiled      per node of the blocks claimed in the recompute:
//                         sum of the 27 neighbouring tiles, then the adjoint
//                         of the node update (walls, contact, gravity,
//                         normalisation) and the collider partials, reduced
//                         per wavefront before one FP64 atomic per scene
//   k_p2g_adj_tiled       one workgroup per occupied block: the P2G adjoint
//                         gathered from an LDS copy of the node adjoints,
//                         through the stress adjoint
// Particles whose FP32 plastic-return or stress adjoint is ill-conditioned are
// done by a second pass in FP64 in the same workgroup, which only workgroups
// that hold such a particle run (kernels of their own over a list of those
// particles cost 2 x 5 us a step with empty lists).
// Both particle kernels are bound by latency at the few wavefronts that their
// registers allow, so they are kept free of spills: held to two wavefronts per
// SIMD they take 40.5 and 29.6 us at 250k particles on 128^3 (half of them
// sand), to three 52.3 and 46.7 (the SVD's and the FP64 pass's live values are
// then spilled).  They took 46.7 and 46.1 us, and 10 us for the FP64 lists,
// with 64-bit row addresses, bound sums through LDS shuffles and four
// barriers a chunk, integer divisions in the flush, and v and C adjoint rows
// that the first kernel zeroed and the second added to.
// The adjoint of s_{t+1} is read through the row map that the segment's sort
// recorded, so no separate permutation pass is needed.
#include <hip/hip_runtime.h>
#include <math.h>
#include <type_traits>
#include "mpm_adjoint.h"
#include "mpm_blocks.h"
#include "mpm_math.h"
#include "mpm_phys.h"
#include "mpm_transfer.h"

namespace mpm {


// ---------------------------------------------------------------------------
// Adjoint of G2P and of the particle update; scatter of the grid velocity
// adjoint.  Writes the direct part of the state adjoint of s_t (x, F, J; the
// v and C adjoints of s_t come only through P2G, whose adjoint writes them).
// ---------------------------------------------------------------------------
template <int NT>
__global__ __launch_bounds__(NT, 2) void k_g2p_adj_tiled(AdjArgs A, StepParams P, FastGeom g) {
  constexpr int NW = NT / 64;
  constexpr int NQ = 3;   // velocity adjoint components
  __shared__ float4 s_v[VT_LDS];
  __shared__ float4 s_tile[TILE_NODES];
  __shared__ __align__(16) int s_itile[NQ * TILE_NODES];
  __shared__ float s_red[NW * NQ];
  __shared__ uint32_t s_ired[NW];
  const int N = A.N;
  const uint32_t n_list = A.list_n[0];
  const uint32_t stamp = (A.gen[0] << 16) | A.sid;
  for (uint32_t e = blockIdx.x; e < n_list; e += gridDim.x) {
    // (opaque to the entry loop, and the entry decoded on the scalar unit: see k_particles)
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));
    int4 ent = A.list[e];
    ent.x = __builtin_amdgcn_readfirstlane(ent.x);
    ent.y = __builtin_amdgcn_readfirstlane(ent.y);
    ent.z = __builtin_amdgcn_readfirstlane(ent.z);
    ent.w = __builtin_amdgcn_readfirstlane(ent.w);
    int sc, bx, by, bz;
    key_decode(g, (uint32_t)ent.x, sc, bx, by, bz);
    const int ox = 4 * bx, oy = 4 * by, oz = 4 * bz;
    const int start = ent.y, count = ent.z;
    // position, material and next row are loaded one chunk ahead
    float px[3] = {0, 0, 0};
    int pm = 0;
    uint32_t pn = 0;
    auto load_inputs = [&](int jn) {
      const uint32_t off = 4u * (uint32_t)jn;
#pragma unroll
      for (int a = 0; a < 3; a++) px[a] = row32(A.st.f, a, N, off);
      pm = A.st.mat[(uint32_t)jn];
      pn = at32(A.map, off);
    };
    auto prefetch = [&](int c0n) {
      const int jn = start + c0n + tid;
      if (c0n + tid < count && jn < N) load_inputs(jn);
    };
    prefetch(0);
    stage_window<NT>(s_v, A.vgrid, g, sc, bx, by, bz, tid);
    if (e == blockIdx.x) {
      // the integer tile starts at zero; every flush leaves it so
      for (int r = tid; r < NQ * TILE_NODES / 4; r += NT) reinterpret_cast<int4*>(s_itile)[r] = make_int4(0, 0, 0, 0);
    }
    __syncthreads();
    const EntrySub es = entry_sub((uint32_t)ent.x, ent.w, g.n_keys);
    float4* tile_out = reinterpret_cast<float4*>(A.tiles + (size_t)es.slot * 4 * TILE_NODES);
    int blo[3] = {1 << 20, 1 << 20, 1 << 20}, bhi[3] = {-(1 << 20), -(1 << 20), -(1 << 20)};
    // One pass over a chunk, as in k_particles: the main pass takes the FP32
    // plastic-return adjoint, and lanes where that is ill-conditioned are done
    // by a second pass (RETRY) in FP64.
    auto pass = [&](auto retry, int c0, const bool has, bool& defer, bool last) -> bool {
      constexpr bool RETRY = decltype(retry)::value;
      const int j = start + c0 + tid;
      const uint32_t off = 4u * (uint32_t)j;
      if (RETRY) {
        if (has) load_inputs(j);
      }
      const float x[3] = {px[0], px[1], px[2]};
      const uint32_t jn = has ? pn : 0u;
      const MatDev& M = P.mats[has ? pm : 0];
      bool ok = has;
      Stencil S;
      int lb[3] = {0, 0, 0}, lv[3] = {0, 0, 0};
      if (ok) {
        const bool in_grid = stencil_setup(x, P, S);
        lv[0] = S.base[0] - (ox - 1); lv[1] = S.base[1] - (oy - 1); lv[2] = S.base[2] - (oz - 1);
        // (inside the velocity window, the stencil is inside the tile: lb = lv + 1)
        const bool in_tile = lv[0] >= 0 && lv[1] >= 0 && lv[2] >= 0 && lv[0] <= VT - 3 && lv[1] <= VT - 3 && lv[2] <= VT - 3;
        if (!in_grid) { atomicOr(P.err, ERR_OUTSIDE); ok = false; }
        else if (!in_tile || jn >= (uint32_t)N) { atomicOr(P.err, ERR_TILE); ok = false; }
#pragma unroll
        for (int a = 0; a < 3; a++) lb[a] = lv[a] + 1;
      }
      float vbt[3] = {0, 0, 0}, Bb[9] = {0, 0, 0, 0, 0, 0, 0, 0, 0}, bnd[NQ] = {0, 0, 0};
      if (ok) {
        // G2P recomputed from the staged velocities
        float vn[3], Bi[9], B[9], Fbo[9], Jbo = 0.f;
        g2p_gather(s_v, lv, S, vn, Bi);
#pragma unroll
        for (int a = 0; a < 3; a++)
#pragma unroll
          for (int b = 0; b < 3; b++) B[a * 3 + b] = P.dx * (Bi[a * 3 + b] - vn[a] * S.f[b]);
        // adjoint of s_{t+1}, row jn of the next state's order, and the F or J of s_t
        float xb[3], vb[3], Cb[9], Fb[9], F[9], J = 0.f;
        const float* an = A.abar_next;
        const uint32_t offn = 4u * jn;
#pragma unroll
        for (int a = 0; a < 3; a++) { xb[a] = row32(an, a, N, offn); vb[a] = row32(an, 3 + a, N, offn); }
#pragma unroll
        for (int k = 0; k < 9; k++) { Cb[k] = row32(an, 6 + k, N, offn); Fb[k] = row32(an, 15 + k, N, offn); }
        const float Jb = row32(an, 24, N, offn);
        if (M.kind == KIND_LIQUID) {
          J = row32(A.st.f, 24, N, off);
        } else {
#pragma unroll
          for (int k = 0; k < 9; k++) F[k] = row32(A.st.f, 15 + k, N, off);
        }
        defer = !particle_update_adjoint<RETRY ? ADJ_FP64 : ADJ_FP32>(vn, B, M, P, F, J, xb, vb, Cb, Fb, Jb, vbt, Bb, Fbo, Jbo);
        if (defer) {
          ok = false;   // (the second pass does it)
        } else {
          // position adjoint through the weights and the node offsets:
          // xo = xb + sum_i grad w_i (v_i . (vbt + Bb (x_i - x_p))) - Bb^T vn
          float c0[3], Ad[9], X[3];
#pragma unroll
          for (int a = 0; a < 3; a++) {
#pragma unroll
            for (int b = 0; b < 3; b++) Ad[a * 3 + b] = P.dx * Bb[a * 3 + b];
            c0[a] = vbt[a] - (Ad[a * 3] * S.f[0] + Ad[a * 3 + 1] * S.f[1] + Ad[a * 3 + 2] * S.f[2]);
          }
          weight_grad_sum<false>(s_v, lv, S, c0, Ad, 0.f, X, nullptr, nullptr);
#pragma unroll
          for (int a = 0; a < 3; a++)
            row32(A.abar, a, N, off) = xb[a] + P.inv_dx * X[a] - (Bb[a] * vn[0] + Bb[3 + a] * vn[1] + Bb[6 + a] * vn[2]);
#pragma unroll
          for (int k = 0; k < 9; k++) row32(A.abar, 15 + k, N, off) = Fbo[k];
          row32(A.abar, 24, N, off) = Jbo;
#pragma unroll
          for (int a = 0; a < 3; a++)
            bnd[a] = fabsf(vbt[a]) + 1.5f * P.dx * (fabsf(Bb[a * 3]) + fabsf(Bb[a * 3 + 1]) + fabsf(Bb[a * 3 + 2]));
          if (!isfinite(bnd[0] + bnd[1] + bnd[2])) {
            atomicOr(P.err, ERR_NONFINITE);
            ok = false;
#pragma unroll
            for (int a = 0; a < NQ; a++) bnd[a] = 0.f;
          }
        }
      } else if (has) {
        // a particle outside the grid carries no adjoint (the call reports it)
#pragma unroll
        for (int a = 0; a < 3; a++) row32(A.abar, a, N, off) = 0.f;
#pragma unroll
        for (int k = 15; k < STATE_FLOATS; k++) row32(A.abar, k, N, off) = 0.f;
      }
      // chunk-wide bound sums and box, as in the forward P2G
      const uint32_t obits = ok ? ((1u << lb[0]) | (1u << (8 + lb[1])) | (1u << (16 + lb[2]))) : 0u;
      const uint32_t wbits = wave_or(obits | (defer ? 1u << 31 : 0u));
      float wb[NQ];
#pragma unroll
      for (int q = 0; q < NQ; q++) wb[q] = wave_sum(bnd[q]);
      const int wv = tid >> 6;
      if ((tid & 63) == 0) {
#pragma unroll
        for (int q = 0; q < NQ; q++) s_red[wv * NQ + q] = wb[q];
        s_ired[wv] = wbits;
      }
      __syncthreads();
      float sc[NQ], isc[NQ];
#pragma unroll
      for (int q = 0; q < NQ; q++) {
        float T = 0.f;
#pragma unroll
        for (int w = 0; w < NW; w++) T += s_red[w * NQ + q];
        // 0.421875: the largest weight of one node, (3/4)^3
        int tb = __builtin_amdgcn_readfirstlane(__float_as_int(T * 0.421875f));
        if ((tb & 0x7f800000) == 0x7f800000) {
          if (tid == 0) atomicOr(P.err, ERR_NONFINITE);
          tb = 0x3f800000;
        }
        const int ex = tb == 0 ? 1 : max((tb >> 23) - 126, -90);
        sc[q] = __int_as_float((157 - ex) << 23);
        isc[q] = __int_as_float((ex + 97) << 23);
      }
      int olo[3], ohi[3];   // the box before this chunk
      uint32_t cb = 0;
#pragma unroll
      for (int w = 0; w < NW; w++) cb |= s_ired[w];
      cb = (uint32_t)__builtin_amdgcn_readfirstlane((int)cb);
      const bool any_deferred = !RETRY && (cb >> 31) != 0u;
#pragma unroll
      for (int a = 0; a < 3; a++) {
        const uint32_t ab = (cb >> (8 * a)) & 0xffu;
        olo[a] = blo[a];
        ohi[a] = bhi[a];
        if (ab) { blo[a] = min(blo[a], __ffs(ab) - 1); bhi[a] = max(bhi[a], 31 - __clz(ab)); }
      }
      if (ok) {
        // c_a(node) = w (vbt_a + sum_b Bb_ab (idx_b - f_b) dx), scaled
        float c0[3], Ad[9];
#pragma unroll
        for (int a = 0; a < 3; a++) {
          const float sa = sc[a];
#pragma unroll
          for (int b = 0; b < 3; b++) Ad[a * 3 + b] = sa * P.dx * Bb[a * 3 + b];
          c0[a] = sa * vbt[a] - (Ad[a * 3] * S.f[0] + Ad[a * 3 + 1] * S.f[1] + Ad[a * 3 + 2] * S.f[2]);
        }
        int* T = s_itile + (lb[0] * TILE + lb[1]) * TILE + lb[2];
#pragma unroll
        for (int i = 0; i < 3; i++) {
          float m1[3];
#pragma unroll
          for (int a = 0; a < 3; a++) m1[a] = c0[a] + (float)i * Ad[a * 3];
#pragma unroll
          for (int jj = 0; jj < 3; jj++) {
            const float wxy = S.w[0][i] * S.w[1][jj];
            float m2[3];
#pragma unroll
            for (int a = 0; a < 3; a++) m2[a] = m1[a] + (float)jj * Ad[a * 3 + 1];
#pragma unroll
            for (int k = 0; k < 3; k++) {
              const float w = wxy * S.w[2][k];
              const int q = (i * TILE + jj) * TILE + k;
#pragma unroll
              for (int a = 0; a < 3; a++)
                atomicAdd(&T[a * TILE_NODES + q], __float2int_rn(w * (m2[a] + (float)k * Ad[a * 3 + 2])));
            }
          }
        }
      }
      if (!RETRY && !any_deferred && c0 + NT < count) prefetch(c0 + NT);
      __syncthreads();
      // flush: see k_particles
      const bool pub = last && !any_deferred;
      if (blo[0] <= bhi[0]) {
        const int ey = bhi[1] - blo[1] + 3, ez = bhi[2] - blo[2] + 3, eyz = ey * ez;
        const int cnt = (bhi[0] - blo[0] + 3) * eyz;
        const uint32_t m1 = div_mul(eyz), m2 = div_mul(ez);
        for (int r = tid; r < cnt; r += NT) {
          const int i = (int)(((uint32_t)r * m1) >> 20), rem = r - i * eyz;
          const int jj = (int)(((uint32_t)rem * m2) >> 20), k = rem - jj * ez;
          const int qi = blo[0] + i, qj = blo[1] + jj, qk = blo[2] + k;
          const int q = (qi * TILE + qj) * TILE + qk;
          float4 val = make_float4((float)s_itile[q] * isc[0], (float)s_itile[TILE_NODES + q] * isc[1],
                                   (float)s_itile[2 * TILE_NODES + q] * isc[2], 0.f);
#pragma unroll
          for (int c = 0; c < NQ; c++) s_itile[c * TILE_NODES + q] = 0;
          if (qi >= olo[0] && qi <= ohi[0] + 2 && qj >= olo[1] && qj <= ohi[1] + 2 && qk >= olo[2] && qk <= ohi[2] + 2) {
            const float4 o = s_tile[q];
            val.x += o.x; val.y += o.y; val.z += o.z;
          }
          if (pub) tile_out[q] = val;
          else s_tile[q] = val;
        }
      }
      return any_deferred;
    };
    for (int c0 = 0; c0 < count; c0 += NT) {
      const bool has = c0 + tid < count && start + c0 + tid < N;
      const bool last = c0 + NT >= count;
      bool defer = false;
      if (pass(std::false_type{}, c0, has, defer, last)) {
        bool none = false;
        pass(std::true_type{}, c0, defer, none, last);
        if (c0 + NT < count) prefetch(c0 + NT);
      }
    }
    // the published tile's box (an empty tile still says that the block has further ones)
    if (tid == 0 && (blo[0] <= bhi[0] || es.extra > 0)) {
      const int hi[3] = {bhi[0] + 2, bhi[1] + 2, bhi[2] + 2};
      A.tile_box[(size_t)(uint32_t)ent.x * NSUB + es.s] =
          make_int4(blo[0] <= bhi[0] ? box_word(blo, hi, es.extra) : (BOX_EMPTY | (es.extra << 24)), (int)stamp,
                    (int)es.slot, 0);
    }
  }
}

// ---------------------------------------------------------------------------
// Adjoint of the grid update on the nodes of the blocks claimed in the
// recompute of step t (the same blocks the velocity-adjoint tiles touch).
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_grid_adj_tiled(AdjArgs A, StepParams P, FastGeom g,
                                                        const double* __restrict__ pose_t,
                                                        const float* __restrict__ act_t, double* __restrict__ acc_t) {
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int li = lane >> 4, lj = (lane >> 2) & 3, lk = lane & 3;
  // one claimed block per wavefront (see k_grid)
  const uint32_t n_waves = 4u * gridDim.x;
  uint32_t it = 4u * blockIdx.x + (uint32_t)wv;
  uint32_t key_it = it < (uint32_t)g.n_keys ? A.cl_list[it] : 0u;
  const uint32_t n_cl = A.cl_count[0];
  const uint32_t stamp = (A.gen[0] << 16) | A.sid;
  for (; it < n_cl && it < (uint32_t)g.n_keys; it += n_waves) {
    const uint32_t key = key_it;
    if (it + n_waves < (uint32_t)g.n_keys) key_it = A.cl_list[it + n_waves];
    int sc, cx, cy, cz;
    key_decode(g, key, sc, cx, cy, cz);
    {
      const int gx = 4 * cx + li, gy = 4 * cy + lj, gz = 4 * cz + lk;
      const size_t node = (size_t)key * 64 + lane;
      const float4 gm = A.mmv[node];
      float4 tsum = make_float4(0.f, 0.f, 0.f, 0.f);
      sum_tiles(g, sc, cx, cy, cz, lane, A.tile_box, A.tiles, stamp, tsum);
      const float vb[3] = {tsum.x, tsum.y, tsum.z};
      float loc[ACC_DOUBLES];
#pragma unroll
      for (int q = 0; q < ACC_DOUBLES; q++) loc[q] = 0.f;
      float4 out = make_float4(0.f, 0.f, 0.f, 0.f);
      if (gm.w > 0.f && gx < g.n && gy < g.n && gz < g.n) {
        const int idx[3] = {gx, gy, gz};
        float mb, mvb[3];
        grid_node_adjoint(P, sc, idx, gm, pose_t, act_t, vb, mb, mvb, loc);
        out = make_float4(mvb[0], mvb[1], mvb[2], mb);
      }
      A.mmvb[node] = out;
      // collider partials: one scene per block, reduced over the wavefront
      bool any = false;
#pragma unroll
      for (int q = 0; q < ACC_DOUBLES; q++) any |= (loc[q] != 0.f);
      if (__ballot(any)) {
#pragma unroll
        for (int q = 0; q < ACC_DOUBLES; q++) loc[q] = wave_sum(loc[q]);
        if (lane == 0) {
          double* dst = acc_t + (size_t)sc * ACC_DOUBLES;
#pragma unroll
          for (int q = 0; q < ACC_DOUBLES; q++)
            if (loc[q] != 0.f) atomicAdd(dst + q, (double)loc[q]);
        }
      }
    }
  }
}

// ---------------------------------------------------------------------------
// Adjoint of P2G: gather of the node adjoints, through the stress adjoint.
// Writes the v and C rows of the state adjoint of s_t and adds to its x and F
// or J rows.
// ---------------------------------------------------------------------------
// One particle of row offset off.  FP64 = false: the stress and its adjoint
// from one FP32 SVD; returns false, before writing anything, for a solid whose
// F is ill-conditioned (s2 < s0/4) or whose FP32 sweeps do not converge.
// FP64 = true: the stress and its adjoint from FP64 SVDs, for the particles
// the FP32 pass returned.  lv is the stencil's first node in the tile.
template <bool FP64>
MPM_DI bool p2g_adj_particle(const AdjArgs& A, const StepParams& P, const MatDev& M, const float4* tile, const int* lv,
                             const Stencil& S, uint32_t off, const float* v, const float* C) {
  const int N = A.N;
  const bool liquid = M.kind == KIND_LIQUID;
  float Ff[9], U[9], sv[3], V[9], tau[9], Jv = 0.f;
  if (liquid) {
    Jv = row32(A.st.f, 24, N, off);
    stress_liquid(Jv, C, M, tau);
  } else {
#pragma unroll
    for (int k = 0; k < 9; k++) Ff[k] = row32(A.st.f, 15 + k, N, off);
    if (FP64) {
      stress_solid(Ff, M, tau);
    } else {
      if (!(svd3(Ff, U, sv, V) && sv[2] > 0.25f * sv[0])) return false;
      stress_solid_usv(Ff, U, sv, V, M, tau);
    }
  }
  float Am[9];
  const float scl = -P.dt * M.vol * 4.f * P.inv_dx * P.inv_dx;
#pragma unroll
  for (int k = 0; k < 9; k++) Am[k] = scl * tau[k] + M.mass * C[k];
  const float mvp[3] = {M.mass * v[0], M.mass * v[1], M.mass * v[2]};
  // node adjoints gathered: mom_i = mvp + Am (x_i - x_p) = c0 + Ad idx_i
  float Ab[9];
  {
    float c0[3], Ad[9], X[3], G0[3], Gi[9];
#pragma unroll
    for (int a = 0; a < 3; a++) {
#pragma unroll
      for (int b = 0; b < 3; b++) Ad[a * 3 + b] = P.dx * Am[a * 3 + b];
      c0[a] = mvp[a] - (Ad[a * 3] * S.f[0] + Ad[a * 3 + 1] * S.f[1] + Ad[a * 3 + 2] * S.f[2]);
    }
    weight_grad_sum<true>(tile, lv, S, c0, Ad, M.mass, X, G0, Gi);
#pragma unroll
    for (int a = 0; a < 3; a++) {
      row32(A.abar, 3 + a, N, off) = M.mass * G0[a];
#pragma unroll
      for (int b = 0; b < 3; b++) Ab[a * 3 + b] = P.dx * (Gi[a * 3 + b] - G0[a] * S.f[b]);
      row32(A.abar, a, N, off) += P.inv_dx * X[a] - (Am[a] * G0[0] + Am[3 + a] * G0[1] + Am[6 + a] * G0[2]);
    }
  }
  float taub[9], Cb[9];
#pragma unroll
  for (int k = 0; k < 9; k++) { taub[k] = scl * Ab[k]; Cb[k] = M.mass * Ab[k]; }
  if (liquid) {
    const float Jo = row32(A.abar, 24, N, off);
    float Jb = 0.f;
    stress_liquid_adjoint(Jv, C, M, taub, Jb, Cb);
    row32(A.abar, 24, N, off) = Jo + Jb;
  } else {
    float Fo[9], Fb[9];
#pragma unroll
    for (int k = 0; k < 9; k++) { Fo[k] = row32(A.abar, 15 + k, N, off); Fb[k] = 0.f; }
    if (FP64) stress_solid_adjoint(Ff, M, taub, Fb);
    else stress_solid_adjoint_usv(Ff, U, sv, V, M, taub, Fb);
#pragma unroll
    for (int k = 0; k < 9; k++) row32(A.abar, 15 + k, N, off) = Fo[k] + Fb[k];
  }
#pragma unroll
  for (int k = 0; k < 9; k++) row32(A.abar, 6 + k, N, off) = Cb[k];
  return true;
}

template <int NT>
__global__ __launch_bounds__(NT, 2) void k_p2g_adj_tiled(AdjArgs A, StepParams P, FastGeom g) {
  __shared__ float4 s_g[VT_LDS];
  const int N = A.N;
  const uint32_t n_list = A.list_n[0];
  // (two workgroups an entry, which take its chunks in turn, the second ones after
  // all the first: 32.2 -> 27.1 us at 250k particles, half of them water, half rigid)
  for (uint32_t e2 = blockIdx.x; e2 < 2u * n_list; e2 += gridDim.x) {
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));
    const uint32_t half = e2 >= n_list ? 1u : 0u;
    int4 ent = A.list[e2 - half * n_list];
    ent.x = __builtin_amdgcn_readfirstlane(ent.x);
    ent.y = __builtin_amdgcn_readfirstlane(ent.y);
    ent.z = __builtin_amdgcn_readfirstlane(ent.z);
    if ((int)half * NT >= ent.z) continue;
    int sc, bx, by, bz;
    key_decode(g, (uint32_t)ent.x, sc, bx, by, bz);
    const int ox = 4 * bx, oy = 4 * by, oz = 4 * bz;
    stage_window<NT>(s_g, A.mmvb, g, sc, bx, by, bz, tid);
    __syncthreads();
    const int start = ent.y, count = ent.z;
    for (int c0 = (int)half * NT; c0 < count; c0 += 2 * NT) {
      const int j = start + c0 + tid;
      // FP32 for every lane, then FP64 for those it returned
      auto pass = [&](auto fp64, bool on) -> bool {
        constexpr bool FP64 = decltype(fp64)::value;
        if (!on) return false;
        const uint32_t off = 4u * (uint32_t)j;
        float x[3], v[3], C[9];
#pragma unroll
        for (int a = 0; a < 3; a++) { x[a] = row32(A.st.f, a, N, off); v[a] = row32(A.st.f, 3 + a, N, off); }
#pragma unroll
        for (int k = 0; k < 9; k++) C[k] = row32(A.st.f, 6 + k, N, off);
        const MatDev& M = P.mats[A.st.mat[(uint32_t)j]];
        Stencil S;
        const bool in_grid = stencil_setup(x, P, S);
        const int lv[3] = {S.base[0] - (ox - 1), S.base[1] - (oy - 1), S.base[2] - (oz - 1)};
        if (!in_grid || lv[0] < 0 || lv[1] < 0 || lv[2] < 0 || lv[0] > VT - 3 || lv[1] > VT - 3 || lv[2] > VT - 3) {
          // no adjoint; reported by the G2P adjoint
#pragma unroll
          for (int k = 3; k < 15; k++) row32(A.abar, k, N, off) = 0.f;
          return false;
        }
        return !p2g_adj_particle<FP64>(A, P, M, s_g, lv, S, off, v, C);
      };
      const bool defer = pass(std::false_type{}, (c0 + tid) < count && j < N);
      if (__ballot(defer)) pass(std::true_type{}, defer);
    }
    __syncthreads();
  }
}

// state adjoint rows from sorted order to user order, as a gather:
// k_adj_pos records the sorted row of every user index (one scattered word
// per particle), then every row is read through it and written in order
__global__ __launch_bounds__(256) void k_adj_pos(const uint32_t* __restrict__ id, int N, uint32_t* __restrict__ pos) {
  const int j = blockIdx.x * blockDim.x + threadIdx.x;
  if (j >= N) return;
  const uint32_t p = id[j];
  if (p < (uint32_t)N) pos[p] = (uint32_t)j;
}
__global__ __launch_bounds__(256) void k_adj_gather(const float* __restrict__ in, float* __restrict__ out,
                                                    const uint32_t* __restrict__ pos, int N) {
  const int p = blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= N) return;
  const uint32_t j = pos[p];
  if (j >= (uint32_t)N) return;
#pragma unroll
  for (int k = 0; k < STATE_FLOATS; k++) out[k * (size_t)N + p] = in[k * (size_t)N + j];
}

static inline unsigned nblk(size_t n, unsigned b) { return (unsigned)((n + b - 1) / b); }

void launch_g2p_adj_tiled(const AdjArgs& A, const StepParams& P, const FastGeom& g, int n_wgs, hipStream_t s) {
  k_g2p_adj_tiled<256><<<n_wgs, 256, 0, s>>>(A, P, g);
}
void launch_grid_adj_tiled(const AdjArgs& A, const StepParams& P, const FastGeom& g, int n_wgs, const double* pose_t,
                           const float* act_t, double* acc_t, hipStream_t s) {
  k_grid_adj_tiled<<<n_wgs, 256, 0, s>>>(A, P, g, pose_t, act_t, acc_t);
}
void launch_p2g_adj_tiled(const AdjArgs& A, const StepParams& P, const FastGeom& g, int n_wgs, hipStream_t s) {
  k_p2g_adj_tiled<256><<<n_wgs, 256, 0, s>>>(A, P, g);
}
__global__ __launch_bounds__(256) void k_row_map(const uint32_t* __restrict__ prev_id, const uint32_t* __restrict__ pos,
                                                 int N, uint32_t* __restrict__ map) {
  const int j = blockIdx.x * blockDim.x + threadIdx.x;
  if (j >= N) return;
  const uint32_t p = prev_id[j];
  map[j] = p < (uint32_t)N ? pos[p] : 0xffffffffu;
}

void launch_row_map(const uint32_t* prev_id, const uint32_t* cur_id, int N, uint32_t* pos, uint32_t* map,
                    hipStream_t s) {
  k_adj_pos<<<nblk(N, 256), 256, 0, s>>>(cur_id, N, pos);
  k_row_map<<<nblk(N, 256), 256, 0, s>>>(prev_id, pos, N, map);
}

__global__ __launch_bounds__(256) void k_copy_list(const int4* __restrict__ src, const uint32_t* __restrict__ src_n,
                                                   int4* __restrict__ dst, uint32_t* __restrict__ dst_n) {
  const uint32_t n = src_n[0];
  for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) dst[i] = src[i];
  if (blockIdx.x == 0 && threadIdx.x == 0) dst_n[0] = n;
}

void launch_copy_list(const int4* src, const uint32_t* src_n, int4* dst, uint32_t* dst_n, hipStream_t s) {
  k_copy_list<<<16, 256, 0, s>>>(src, src_n, dst, dst_n);
}

void launch_adj_reorder(const float* in, float* out, const uint32_t* id, int N, uint32_t* pos, hipStream_t s) {
  k_adj_pos<<<nblk(N, 256), 256, 0, s>>>(id, N, pos);
  k_adj_gather<<<nblk(N, 256), 256, 0, s>>>(in, out, pos, N);
}

}  // namespace mpm
