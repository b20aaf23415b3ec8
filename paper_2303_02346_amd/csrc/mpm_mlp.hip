// Training and batch inference of the learned cone-return closure
// (6 -> 64 -> 64 -> 3 MLP, ReLU).  The forward runs on the matrix cores in
// BF16 with FP32 accumulation; the backward (FP32 matrix cores) and Adam run
// in FP32.  Loss: mean squared error of the normalised outputs.
//
// State layout (device, caller-owned, mpm_mlp_state_bytes()):
//   params  FP32 [MLP_NPARAM]   master weights W1 b1 W2 b2 W3 b3 (row-major [out][in])
//   adam_m  FP32 [MLP_NPARAM]
//   adam_v  FP32 [MLP_NPARAM]
//   grad    FP32 [MLP_NPARAM]   sums of the normalisation statistics (initialisation only)
//   misc    FP64 [8]            loss accumulator, step count
//   blob    MlpBlob             inference copy (normalisation, FP32 biases, BF16 weights)
#include <hip/hip_runtime.h>
#include <math.h>
#include <stddef.h>
#include <stdint.h>
#include <string.h>
#include <mutex>
#include <random>
#include <vector>

#include "../../include/mpm.h"
#include "mpm_mlp.h"

namespace mpm {

namespace {
constexpr size_t A256 = 256;
inline size_t al(size_t x) { return (x + A256 - 1) & ~(A256 - 1); }

struct MlpLayout {
  size_t params, m, v, grad, misc, blob, total;
};
MlpLayout mlp_layout() {
  MlpLayout L;
  size_t o = 0;
  L.params = o; o += al(MLP_NPARAM * 4);
  L.m = o; o += al(MLP_NPARAM * 4);
  L.v = o; o += al(MLP_NPARAM * 4);
  L.grad = o; o += al(MLP_NPARAM * 4);
  L.misc = o; o += al(64);
  L.blob = o; o += al(sizeof(MlpBlob));
  L.total = o;
  return L;
}
constexpr int SAMPLE = MLP_IN + MLP_OUT;   // floats per logged sample
}  // namespace

// normalisation statistics (mean, std) of the 9 sample columns, FP64 sums:
// reduced over the workgroup before the atomics, of which there are then 18
// per workgroup (18 per wavefront of 256 workgroups took 113 us for 131072
// samples, all of it the queue at the 18 addresses)
__global__ __launch_bounds__(1024) void k_mlp_stats(const float* __restrict__ samples, long long n,
                                                    double* __restrict__ acc) {
  __shared__ double s_w[16][2 * SAMPLE];
  double s[SAMPLE], q[SAMPLE];
#pragma unroll
  for (int c = 0; c < SAMPLE; c++) { s[c] = 0.0; q[c] = 0.0; }
  for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < n; i += (long long)gridDim.x * blockDim.x) {
#pragma unroll
    for (int c = 0; c < SAMPLE; c++) { double v = samples[i * SAMPLE + c]; s[c] += v; q[c] += v * v; }
  }
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
#pragma unroll
  for (int c = 0; c < SAMPLE; c++) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) { s[c] += __shfl_xor(s[c], off); q[c] += __shfl_xor(q[c], off); }
    if (lane == 0) { s_w[wv][c] = s[c]; s_w[wv][SAMPLE + c] = q[c]; }
  }
  __syncthreads();
  if (threadIdx.x < 2 * SAMPLE) {
    double t = 0.0;
#pragma unroll
    for (int w = 0; w < 16; w++) t += s_w[w][threadIdx.x];
    atomicAdd(acc + threadIdx.x, t);
  }
}

__global__ void k_mlp_stats_final(const double* __restrict__ acc, long long n, MlpBlob* __restrict__ blob) {
  int c = threadIdx.x;
  if (c >= SAMPLE) return;
  double mean = acc[c] / (double)n;
  double var = acc[SAMPLE + c] / (double)n - mean * mean;
  double sd = sqrt(var > 0.0 ? var : 0.0);
  // a column that barely varies in the training set (one material) keeps a
  // deviation floor so that other values stay in a sane range
  double floor_sd = 1e-4 + 1e-3 * fabs(mean);
  if (sd < floor_sd) sd = floor_sd;
  if (c < MLP_IN) { blob->in_mean[c] = (float)mean; blob->in_std[c] = (float)sd; }
  else { blob->out_mean[c - MLP_IN] = (float)mean; blob->out_std[c - MLP_IN] = (float)sd; }
}

// FP32 master parameters -> inference blob (BF16 weights, padded; FP32 biases)
__global__ void k_mlp_publish(const float* __restrict__ p, MlpBlob* __restrict__ blob) {
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < MLP_H * MLP_K1 + MLP_H * MLP_H + MLP_N3 * MLP_H + 2 * MLP_H + MLP_N3;
       i += gridDim.x * blockDim.x) {
    if (i < MLP_H * MLP_K1) {
      int n = i / MLP_K1, k = i % MLP_K1;
      blob->W1[i] = f2bf(k < MLP_IN ? p[OFF_W1 + n * MLP_IN + k] : 0.f);
      continue;
    }
    int j = i - MLP_H * MLP_K1;
    if (j < MLP_H * MLP_H) { blob->W2[j] = f2bf(p[OFF_W2 + j]); continue; }
    j -= MLP_H * MLP_H;
    if (j < MLP_N3 * MLP_H) {
      int n = j / MLP_H, k = j % MLP_H;
      blob->W3[j] = f2bf(n < MLP_OUT ? p[OFF_W3 + n * MLP_H + k] : 0.f);
      continue;
    }
    j -= MLP_N3 * MLP_H;
    if (j < MLP_H) { blob->b1[j] = p[OFF_B1 + j]; continue; }
    j -= MLP_H;
    if (j < MLP_H) { blob->b2[j] = p[OFF_B2 + j]; continue; }
    j -= MLP_H;
    blob->b3[j] = j < MLP_OUT ? p[OFF_B3 + j] : 0.f;
  }
}

// ---------------------------------------------------------------------------
// The network on 16 samples per wavefront (the row block of one 16x16 MFMA
// tile; lane (lr, lg) = (lane % 16, lane / 16)), every weight fragment in
// registers: 24 fragments of 4 BF16 values, loaded once per wavefront with
// 8-byte loads and used for every row block it works through.  (Staging the
// 13 KB of weights in LDS for each workgroup instead costs the staging and
// 16-way bank conflicts: the rows are 128 bytes.)
// ---------------------------------------------------------------------------
struct MlpFrag {
  bf16x4_t w1[4], w2[4][4], w3[4];   // [16-output tile]([16-input tile])
  float b1[4], b2[4], b3;
};

__device__ __forceinline__ bf16x4_t load_frag(const uint16_t* p) {
  const uint2 v = *reinterpret_cast<const uint2*>(p);
  union { uint2 u; bf16x4_t b; } c;
  c.u = v;
  return c.b;
}

__device__ __forceinline__ void load_frags(const MlpBlob* __restrict__ W, int lr, int lg, MlpFrag& F) {
  static_assert(offsetof(MlpBlob, W1) % 8 == 0 && offsetof(MlpBlob, W2) % 8 == 0 && offsetof(MlpBlob, W3) % 8 == 0,
                "8-byte fragment loads");
#pragma unroll
  for (int nt = 0; nt < 4; nt++) {
    F.w1[nt] = load_frag(W->W1 + (16 * nt + lr) * MLP_K1 + 4 * lg);
    F.w3[nt] = load_frag(W->W3 + lr * MLP_H + 16 * nt + 4 * lg);
    F.b1[nt] = W->b1[16 * nt + lr];
    F.b2[nt] = W->b2[16 * nt + lr];
#pragma unroll
    for (int kt = 0; kt < 4; kt++) F.w2[nt][kt] = load_frag(W->W2 + (16 * nt + lr) * MLP_H + 16 * kt + 4 * lg);
  }
  F.b3 = W->b3[lr];
}

// LDS row stride of a sample's 64 activations: rows stay 16-byte aligned and
// begin 4 banks apart
constexpr int HS = 68;

// One layer's input fragments from the wavefront's 16 LDS rows (the values are
// already rounded to BF16, so the upper half is exact).
__device__ __forceinline__ void frags_from_rows(const float* H, int lr, int lg, bf16x4_t* a) {
#pragma unroll
  for (int kt = 0; kt < 4; kt++) {
    const float4 v = *reinterpret_cast<const float4*>(H + lr * HS + 16 * kt + 4 * lg);
    a[kt][0] = (short)(__float_as_uint(v.x) >> 16);
    a[kt][1] = (short)(__float_as_uint(v.y) >> 16);
    a[kt][2] = (short)(__float_as_uint(v.z) >> 16);
    a[kt][3] = (short)(__float_as_uint(v.w) >> 16);
  }
}

// Forward of the wavefront's 16 samples: x = the 6 inputs of sample lr (every
// lane of a sample's group holds them).  H1, H2: the wavefront's LDS rows,
// left with the BF16-rounded activations; h1, h2: the same in the lane's
// accumulator places (sample 4 lg + q, unit 16 nt + lr); Y: 16 rows of 4 floats,
// left with the normalised outputs.
__device__ __forceinline__ void mlp_rows16(const MlpBlob* __restrict__ W, const MlpFrag& F, const float* xn, int lr,
                                           int lg, float* H1, float* H2, float* Y, f32x4_t* h1, f32x4_t* h2) {
  bf16x4_t a1;
#pragma unroll
  for (int q = 0; q < 4; q++) {
    float v = lg == 0 ? xn[q] : (lg == 1 && q < 2 ? xn[(4 + q) % MLP_IN] : 0.f);
    a1[q] = (short)f2bf(v);
  }
#pragma unroll
  for (int nt = 0; nt < 4; nt++) {
    f32x4_t c = {0.f, 0.f, 0.f, 0.f};
    c = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a1, F.w1[nt], c, 0, 0, 0);
#pragma unroll
    for (int q = 0; q < 4; q++) {
      h1[nt][q] = bf2f(f2bf(fmaxf(c[q] + F.b1[nt], 0.f)));
      H1[(4 * lg + q) * HS + 16 * nt + lr] = h1[nt][q];
    }
  }
  wave_lds_sync();
  bf16x4_t a[4];
  frags_from_rows(H1, lr, lg, a);
#pragma unroll
  for (int nt = 0; nt < 4; nt++) {
    f32x4_t c = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int kt = 0; kt < 4; kt++) c = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a[kt], F.w2[nt][kt], c, 0, 0, 0);
#pragma unroll
    for (int q = 0; q < 4; q++) {
      h2[nt][q] = bf2f(f2bf(fmaxf(c[q] + F.b2[nt], 0.f)));
      H2[(4 * lg + q) * HS + 16 * nt + lr] = h2[nt][q];
    }
  }
  wave_lds_sync();
  frags_from_rows(H2, lr, lg, a);
  f32x4_t c3 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int kt = 0; kt < 4; kt++) c3 = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a[kt], F.w3[kt], c3, 0, 0, 0);
  if (lr < MLP_OUT) {
#pragma unroll
    for (int q = 0; q < 4; q++) Y[(4 * lg + q) * 4 + lr] = c3[q] + F.b3;
  }
  wave_lds_sync();
}

// Denormalised outputs of one sample, shifted equally onto the inputs' trace.
__device__ __forceinline__ void mlp_outputs(const MlpBlob* __restrict__ W, const float* x, const float* Yrow, float* y) {
#pragma unroll
  for (int o = 0; o < MLP_OUT; o++) y[o] = Yrow[o] * W->out_std[o] + W->out_mean[o];
  const float dtr = ((x[0] + x[1] + x[2]) - (y[0] + y[1] + y[2])) * (1.f / 3.f);
#pragma unroll
  for (int o = 0; o < MLP_OUT; o++) y[o] += dtr;
}

// Batch inference, one wavefront per 16 records at a time.
__global__ __launch_bounds__(256) void k_mlp_predict(const MlpBlob* __restrict__ W, const float* __restrict__ samples,
                                                     long long n, float* __restrict__ y_out) {
  __shared__ __align__(16) float sH[4][2][16 * HS];
  __shared__ __align__(16) float sY[4][16 * 4];
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, lr = lane & 15, lg = lane >> 4;
  MlpFrag F;
  load_frags(W, lr, lg, F);
  for (long long r0 = ((long long)blockIdx.x * 4 + wv) * 16; r0 < n; r0 += (long long)gridDim.x * 64) {
    const bool has = r0 + lr < n;
    const float* rec = samples + (has ? r0 + lr : r0) * SAMPLE;
    float x[MLP_IN], xn[MLP_IN];
#pragma unroll
    for (int c = 0; c < MLP_IN; c++) x[c] = rec[c];
#pragma unroll
    for (int c = 0; c < MLP_IN; c++) xn[c] = (x[c] - W->in_mean[c]) / W->in_std[c];
    f32x4_t h1[4], h2[4];
    mlp_rows16(W, F, xn, lr, lg, sH[wv][0], sH[wv][1], sY[wv], h1, h2);
    if (lg == 0 && has) {
      float y[MLP_OUT];
      mlp_outputs(W, x, sY[wv] + 4 * lr, y);
#pragma unroll
      for (int c = 0; c < MLP_OUT; c++) y_out[(r0 + lr) * MLP_OUT + c] = y[c];
    }
    wave_lds_sync();
  }
}

// A batch's gradient takes two launches: k_mlp_batch (forward and input
// gradients per sample) and k_mlp_update (weight gradients, and in training
// the Adam step and the published copy).  Both run their FP32 products on the
// matrix cores: v_mfma_f32_16x16x4f32 adds its four products to the
// accumulator as a chain of FMAs in the order of the contraction index, so a
// weight's gradient is the sequential FP32 sum over the samples of each of 16
// slices of the batch, the slices added in FP64 and rounded once.  At a batch of
// 4096 the work is 140 MFLOP (1 us at the FP32 rate); the time is the latency
// of the two launches' chains.  One thread per sample with scalar products,
// then one thread per weight and slice reading every sample's stored
// activations with float atomics, took 66 + 96 us per batch (and 10 us for Adam
// and the copy in launches of their own); these take 10 + 14 us.
//
// Per-sample scratch of a batch of nb, structure of arrays.  Units are grouped
// by 16 (a matrix tile's edge), so that a wavefront of k_mlp_update reads four
// samples' 16 values of a group as 256 contiguous bytes.
struct BatchScratch {
  float* d1;        // [4][nb][16] adjoints of the first hidden layer's sums
  float* d2;        // [4][nb][16] of the second's
  float* x;         // [nb][12] normalised inputs (6), 1, 0, adjoint of the output (3), 0
  uint16_t* h1;     // [4][nb][16] BF16 activations
  uint16_t* h2;
  double* loss;     // [ceil(nb / 16)] per wavefront
};
constexpr int XS = 12;
constexpr size_t SCR_BYTES = 2 * MLP_H * 4 + XS * 4 + 2 * MLP_H * 2;   // per sample, without the loss
static_assert(SCR_BYTES % 16 == 0, "alignment of the arrays");
__host__ __device__ constexpr size_t scratch_bytes(size_t nb) { return nb * SCR_BYTES + (nb + 15) / 16 * 8; }
__host__ __device__ inline BatchScratch scratch_of(void* base, size_t nb) {
  char* p = (char*)base;
  BatchScratch S;
  S.d1 = (float*)p; p += nb * MLP_H * 4;
  S.d2 = (float*)p; p += nb * MLP_H * 4;
  S.x = (float*)p; p += nb * XS * 4;
  S.h1 = (uint16_t*)p; p += nb * MLP_H * 2;
  S.h2 = (uint16_t*)p; p += nb * MLP_H * 2;
  S.loss = (double*)p;
  return S;
}

// Forward and input gradients of the batch (samples i0 .. i0 + nb - 1,
// wrapping at n), 16 samples per wavefront, one row block each, so that a batch
// of 4096 has 256 wavefronts (two per workgroup).
constexpr int BATCH_NT = 128;
__global__ __launch_bounds__(BATCH_NT) void k_mlp_batch(const MlpBlob* __restrict__ W, const float* __restrict__ samples,
                                                        long long n, long long i0, int nb, void* scr) {
  constexpr int NW = BATCH_NT / 64;
  __shared__ __align__(16) float sH1[NW][16 * HS], sH2[NW][16 * HS];
  __shared__ __align__(16) float sY[NW][16 * 4], sD[NW][16 * 4];
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, lr = lane & 15, lg = lane >> 4;
  const int base = (blockIdx.x * NW + wv) * 16;
  if (base >= nb) return;
  const BatchScratch S = scratch_of(scr, (size_t)nb);
  const int b = base + lr;                       // the sample of the lane's group
  const bool has = b < nb;
  long long si = i0 + (has ? b : base);
  if (si >= n) si -= n;                          // (i0 < n and nb <= n)
  float x[MLP_IN], xn[MLP_IN], t[MLP_OUT];
#pragma unroll
  for (int c = 0; c < MLP_IN; c++) x[c] = samples[si * SAMPLE + c];
#pragma unroll
  for (int c = 0; c < MLP_OUT; c++) t[c] = samples[si * SAMPLE + MLP_IN + c];
  MlpFrag F;
  load_frags(W, lr, lg, F);
  // W2 for dh1 = dh2 W2: rows 4 k + lg, tile nt's column lr standing for input
  // 4 lr + nt, so that a row's four tiles are one 8-byte load
  bf16x4_t wb[16];
#pragma unroll
  for (int k = 0; k < 16; k++) wb[k] = load_frag(W->W2 + (4 * k + lg) * MLP_H + 4 * lr);
  float w3[4][MLP_OUT];
#pragma unroll
  for (int nt = 0; nt < 4; nt++)
#pragma unroll
    for (int c = 0; c < MLP_OUT; c++) w3[nt][c] = bf2f(W->W3[c * MLP_H + 16 * nt + lr]);
#pragma unroll
  for (int c = 0; c < MLP_IN; c++) xn[c] = (x[c] - W->in_mean[c]) / W->in_std[c];
  float* H1 = sH1[wv];
  float* H2 = sH2[wv];
  f32x4_t h1[4], h2[4];
  mlp_rows16(W, F, xn, lr, lg, H1, H2, sY[wv], h1, h2);
  double loss = 0.0;
  {
    // normalised error of the trace-projected output y; the adjoint of the
    // network's normalised output yn goes back through the projection
    // y = P(yn * std + mean), P(u) = u + (tr x - sum u) / 3
    float y[MLP_OUT], g[MLP_OUT], dy[MLP_OUT], gs = 0.f;
    mlp_outputs(W, x, sY[wv] + 4 * lr, y);
#pragma unroll
    for (int c = 0; c < MLP_OUT; c++) {
      const float yn = (y[c] - W->out_mean[c]) / W->out_std[c];
      const float tn = (t[c] - W->out_mean[c]) / W->out_std[c];
      const float e = yn - tn;
      loss += (double)e * e;
      g[c] = 2.f * e / (float)(MLP_OUT * nb) / W->out_std[c];   // dL/dy
      gs += g[c];
    }
#pragma unroll
    for (int c = 0; c < MLP_OUT; c++) dy[c] = (g[c] - gs * (1.f / 3.f)) * W->out_std[c];
    if (!has || lg != 0) loss = 0.0;
    if (lg == 0) *reinterpret_cast<float4*>(sD[wv] + 4 * lr) = make_float4(dy[0], dy[1], dy[2], 0.f);
    if (has && lg < 3)
      *reinterpret_cast<float4*>(S.x + (size_t)b * XS + 4 * lg) =
          lg == 0 ? make_float4(xn[0], xn[1], xn[2], xn[3])
                  : (lg == 1 ? make_float4(xn[4], xn[5], 1.f, 0.f) : make_float4(dy[0], dy[1], dy[2], 0.f));
  }
  wave_lds_sync();
  // dh2 = W3^T dy masked by ReLU (BF16 weights), over the H2 rows in LDS (the
  // third layer has read them)
#pragma unroll
  for (int q = 0; q < 4; q++) {
    const float4 d = *reinterpret_cast<const float4*>(sD[wv] + 4 * (4 * lg + q));
    const int bq = base + 4 * lg + q;
#pragma unroll
    for (int nt = 0; nt < 4; nt++) {
      float v = 0.f;
      v += w3[nt][0] * d.x;
      v += w3[nt][1] * d.y;
      v += w3[nt][2] * d.z;
      v = h2[nt][q] > 0.f ? v : 0.f;
      H2[(4 * lg + q) * HS + 16 * nt + lr] = v;
      if (bq < nb) {
        const size_t o = ((size_t)nt * nb + bq) * 16 + lr;
        S.d2[o] = v;
        S.h1[o] = (uint16_t)(__float_as_uint(h1[nt][q]) >> 16);
        S.h2[o] = (uint16_t)(__float_as_uint(h2[nt][q]) >> 16);
      }
    }
  }
  wave_lds_sync();
  f32x4_t d1[4];
#pragma unroll
  for (int nt = 0; nt < 4; nt++) d1[nt] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int k = 0; k < 16; k++) {
    const float a = H2[lr * HS + 4 * k + lg];
#pragma unroll
    for (int nt = 0; nt < 4; nt++)
      d1[nt] = __builtin_amdgcn_mfma_f32_16x16x4f32(a, bf2f((uint16_t)wb[k][nt]), d1[nt], 0, 0, 0);
  }
#pragma unroll
  for (int q = 0; q < 4; q++) {
    const int bq = base + 4 * lg + q;
    const float4 h = *reinterpret_cast<const float4*>(H1 + (4 * lg + q) * HS + 4 * lr);
    if (bq < nb)
      *reinterpret_cast<float4*>(S.d1 + ((size_t)(lr >> 2) * nb + bq) * 16 + 4 * (lr & 3)) =
          make_float4(h.x > 0.f ? d1[0][q] : 0.f, h.y > 0.f ? d1[1][q] : 0.f, h.z > 0.f ? d1[2][q] : 0.f,
                      h.w > 0.f ? d1[3][q] : 0.f);
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) loss += __shfl_xor(loss, off);
  if (lane == 0) S.loss[base / 16] = loss / (double)(MLP_OUT * nb);
}

// One 16 x 16 tile of weight gradients over the samples b0 .. b1 - 1, as a
// sequential chain: acc += A^T B with A the tile's 16 adjoint values of a
// sample and B its 16 input values.
//   AD: A = d[b][lr] of one unit group (row stride 16), else the output adjoint (x row, 8 ..)
//   BH: B = h[b][lr] of one unit group (BF16), else the inputs and the 1 (x row, 0 ..)
template <bool AD, bool BH>
__device__ __forceinline__ f32x4_t wgrad_chain(const float* __restrict__ d, const uint16_t* __restrict__ h,
                                               const float* __restrict__ x, int b0, int b1, int lr, int lg) {
  f32x4_t acc = {0.f, 0.f, 0.f, 0.f};
  auto av = [&](int b) { return AD ? d[(size_t)b * 16 + lr] : (lr < MLP_OUT ? x[(size_t)b * XS + 8 + lr] : 0.f); };
  auto bv = [&](int b) { return BH ? bf2f(h[(size_t)b * 16 + lr]) : (lr <= MLP_IN ? x[(size_t)b * XS + lr] : 0.f); };
  // operands loaded 16 products ahead: one group is in flight while the other
  // is multiplied
  int b = b0;
  constexpr int U = 16;
  float a[2][U], c[2][U];
  auto load = [&](int s, int at) {
#pragma unroll
    for (int u = 0; u < U; u++) { a[s][u] = av(at + 4 * u + lg); c[s][u] = bv(at + 4 * u + lg); }
  };
  auto mul = [&](int s) {
#pragma unroll
    for (int u = 0; u < U; u++) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a[s][u], c[s][u], acc, 0, 0, 0);
  };
  if (b + 4 * U <= b1) {
    load(0, b);
    for (; b + 12 * U <= b1; b += 8 * U) {
      load(1, b + 4 * U);
      mul(0);
      load(0, b + 8 * U);
      mul(1);
    }
    if (b + 8 * U <= b1) {
      load(1, b + 4 * U);
      mul(0);
      mul(1);
      b += 8 * U;
    } else {
      mul(0);
      b += 4 * U;
    }
  }
  for (; b < b1; b += 4) {
    const bool ok = b + lg < b1;
    const float at = ok ? av(b + lg) : 0.f, ct = ok ? bv(b + lg) : 0.f;
    acc = __builtin_amdgcn_mfma_f32_16x16x4f32(at, ct, acc, 0, 0, 0);
  }
  return acc;
}

// Place of parameter i in the inference blob.
__device__ __forceinline__ void publish_param(MlpBlob* __restrict__ blob, int i, float v) {
  if (i < OFF_B1) blob->W1[(i / MLP_IN) * MLP_K1 + i % MLP_IN] = f2bf(v);
  else if (i < OFF_W2) blob->b1[i - OFF_B1] = v;
  else if (i < OFF_B2) blob->W2[i - OFF_W2] = f2bf(v);
  else if (i < OFF_W3) blob->b2[i - OFF_B2] = v;
  else if (i < OFF_B3) blob->W3[i - OFF_W3] = f2bf(v);
  else blob->b3[i - OFF_B3] = v;
}

// Weight gradients of the batch, one 16 x 16 tile per workgroup and one of 16
// slices of the samples per wavefront; the slices meet in LDS.  Tiles 0..15: dW2; 16..19: dW1 with db1 as the column of ones; 20..23: db2;
// 24..27: dW3; 28: db3, which also sums the loss into misc[0] (first: stores it).
// With ADAM the step (Kingma and Ba 2015) on the FP32 master weights and their
// copy in the blob follow in the same launch; else the gradient goes to grad.
constexpr int SLICES = 16, UPDATE_TILES = 29;
template <bool ADAM>
__global__ __launch_bounds__(64 * SLICES) void k_mlp_update(void* scr, int nb, float* __restrict__ grad,
                                                            double* __restrict__ misc, int first, float* __restrict__ p,
                                                            float* __restrict__ m, float* __restrict__ v,
                                                            MlpBlob* __restrict__ blob, float lr, float b1, float b2,
                                                            float eps, float c1, float c2) {
  __shared__ float sG[SLICES][256];
  const BatchScratch S = scratch_of(scr, (size_t)nb);
  const int lane = threadIdx.x & 63, sl = threadIdx.x >> 6, lc = lane & 15, lg = lane >> 4;
  const int tile = blockIdx.x;
  const int s0 = (int)((long long)nb * sl / SLICES), s1 = (int)((long long)nb * (sl + 1) / SLICES);
  const size_t grp = (size_t)nb * 16;      // one group of 16 units
  f32x4_t acc;
  if (tile < 16) acc = wgrad_chain<true, true>(S.d2 + (tile >> 2) * grp, S.h1 + (tile & 3) * grp, nullptr, s0, s1, lc, lg);
  else if (tile < 20) acc = wgrad_chain<true, false>(S.d1 + (tile - 16) * grp, nullptr, S.x, s0, s1, lc, lg);
  else if (tile < 24) acc = wgrad_chain<true, false>(S.d2 + (tile - 20) * grp, nullptr, S.x, s0, s1, lc, lg);
  else if (tile < 28) acc = wgrad_chain<false, true>(nullptr, S.h2 + (tile - 24) * grp, S.x, s0, s1, lc, lg);
  else acc = wgrad_chain<false, false>(nullptr, nullptr, S.x, s0, s1, lc, lg);
#pragma unroll
  for (int q = 0; q < 4; q++) sG[sl][(4 * lg + q) * 16 + lc] = acc[q];
  if (tile == 28 && sl == SLICES - 1) {
    double l = 0.0;
    for (int r = lane; r < (nb + 15) / 16; r += 64) l += S.loss[r];
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) l += __shfl_xor(l, off);
    if (lane == 0) {
      misc[0] = first ? l : misc[0] + l;
      if (!ADAM) misc[1] = 0.0;   // (a gradient call ends a training run: its Adam step count starts anew)
    }
  }
  __syncthreads();
  const int tid = threadIdx.x;
  if (tid >= 256) return;
  const int r = tid >> 4, c = tid & 15;    // row (adjoint unit) and column (input unit) of the tile
  int i = -1;
  if (tile < 16) i = OFF_W2 + (16 * (tile >> 2) + r) * MLP_H + 16 * (tile & 3) + c;
  else if (tile < 20) { if (c < MLP_IN) i = OFF_W1 + (16 * (tile - 16) + r) * MLP_IN + c; else if (c == MLP_IN) i = OFF_B1 + 16 * (tile - 16) + r; }
  else if (tile < 24) { if (c == MLP_IN) i = OFF_B2 + 16 * (tile - 20) + r; }
  else if (tile < 28) { if (r < MLP_OUT) i = OFF_W3 + r * MLP_H + 16 * (tile - 24) + c; }
  else if (r < MLP_OUT && c == MLP_IN) i = OFF_B3 + r;
  if (i < 0) return;
  double gs = 0.0;
#pragma unroll
  for (int q = 0; q < SLICES; q++) gs += (double)sG[q][tid];
  const float gi = (float)gs;
  if (!ADAM) {
    grad[i] = gi;
    return;
  }
  float mi = b1 * m[i] + (1.f - b1) * gi;
  float vi = b2 * v[i] + (1.f - b2) * gi * gi;
  m[i] = mi;
  v[i] = vi;
  const float w = p[i] - lr * (mi / c1) / (sqrtf(vi / c2) + eps);
  p[i] = w;
  publish_param(blob, i, w);
}

// Per-sample scratch of mpm_mlp_grad_noalloc for at most
// MPM_MLP_NOALLOC_MAX_BATCH samples (1.7 MB), one copy per device for the
// life of the process.  Host code never passes this name to a kernel: it uses
// the address hipGetSymbolAddress returns for the device.
static __device__ __align__(256) char scratch[scratch_bytes(MPM_MLP_NOALLOC_MAX_BATCH)];

}  // namespace mpm

using namespace mpm;

static int hipok(hipError_t e) { return e == hipSuccess ? MPM_OK : MPM_EHIP; }

// Device address of `scratch` on device dev, looked up once per device (with
// that device current: the caller's) and kept.
static void* noalloc_scratch(int dev) {
  constexpr int kMaxDevices = 64;
  static std::mutex mu;
  static void* ptr[kMaxDevices] = {};
  if (dev < 0 || dev >= kMaxDevices) return nullptr;
  std::lock_guard<std::mutex> lock(mu);
  if (!ptr[dev]) {
    void* p = nullptr;
    if (hipGetSymbolAddress(&p, HIP_SYMBOL(mpm::scratch)) != hipSuccess || !p) return nullptr;
    ptr[dev] = p;
  }
  return ptr[dev];
}

extern "C" {

// The arrays are read and written in 16-byte words, but a caller's scratch may
// start anywhere.  (Aligned here and not in the kernels: a pointer made from an
// integer there is no longer known to be global, and its loads become flat ones.)
constexpr size_t SCR_ALIGN = 16;
static void* aligned_scratch(void* p) { return (void*)(((uintptr_t)p + SCR_ALIGN - 1) & ~(uintptr_t)(SCR_ALIGN - 1)); }

size_t mpm_mlp_state_bytes(void) { return mlp_layout().total; }

size_t mpm_mlp_scratch_bytes(int32_t batch) {
  if (batch < 1) return 0;
  return al(scratch_bytes((size_t)batch) + SCR_ALIGN);
}

int mpm_mlp_init(void* state_dev, const float* samples_dev, int64_t n, const float* init_params, uint64_t seed,
                 void* stream) {
  if (!state_dev || !samples_dev || n < 2) return MPM_EINVAL;
  hipStream_t s = (hipStream_t)stream;
  MlpLayout L = mlp_layout();
  char* st = (char*)state_dev;
  std::vector<float> p(MLP_NPARAM, 0.f);
  if (init_params) {
    memcpy(p.data(), init_params, sizeof(float) * MLP_NPARAM);
  } else {
    // He-uniform initialisation, zero biases
    std::mt19937_64 rng(seed);
    auto fill = [&](int off, int fan_in, int count) {
      float lim = sqrtf(6.f / fan_in);
      std::uniform_real_distribution<float> u(-lim, lim);
      for (int q = 0; q < count; q++) p[off + q] = u(rng);
    };
    fill(OFF_W1, MLP_IN, MLP_H * MLP_IN);
    fill(OFF_W2, MLP_H, MLP_H * MLP_H);
    fill(OFF_W3, MLP_H, MLP_OUT * MLP_H);
  }
  int rc = MPM_OK;
  if (hipMemcpyAsync(st + L.params, p.data(), sizeof(float) * MLP_NPARAM, hipMemcpyHostToDevice, s) != hipSuccess ||
      hipMemsetAsync(st + L.m, 0, L.misc - L.m, s) != hipSuccess || hipMemsetAsync(st + L.misc, 0, 64, s) != hipSuccess ||
      hipMemsetAsync(st + L.blob, 0, sizeof(MlpBlob), s) != hipSuccess)
    rc = MPM_EHIP;
  if (rc == MPM_OK) {
    // the statistics need 18 doubles: accumulate in the (still zero) gradient block
    double* acc = (double*)(st + L.grad);
    k_mlp_stats<<<(unsigned)(n < 64 * 1024 ? (n + 1023) / 1024 : 64), 1024, 0, s>>>((const float*)samples_dev, n, acc);
    k_mlp_stats_final<<<1, 64, 0, s>>>(acc, n, (MlpBlob*)(st + L.blob));
    if (hipMemsetAsync(st + L.grad, 0, al(MLP_NPARAM * 4), s) != hipSuccess) rc = MPM_EHIP;
    k_mlp_publish<<<32, 256, 0, s>>>((const float*)(st + L.params), (MlpBlob*)(st + L.blob));
  }
  if (rc == MPM_OK) rc = hipok(hipStreamSynchronize(s));
  return rc;
}

// Forward and input gradients of the batch (samples i0 .. i0 + nb - 1) into scr.
static void batch_forward(const char* st, const float* samples, long long n, long long i0, int nb, void* scr,
                          hipStream_t s) {
  constexpr int per = BATCH_NT / 4;   // samples of a workgroup
  k_mlp_batch<<<(nb + per - 1) / per, BATCH_NT, 0, s>>>((const MlpBlob*)(st + mlp_layout().blob), samples, n, i0, nb, scr);
}

// Loss and gradient of the first nb records with the per-sample scratch scr
// (shared by mpm_mlp_grad and mpm_mlp_grad_noalloc).
static int grad_impl(void* state_dev, const float* samples_dev, int64_t n, int nb, void* scr, float* grad_out_dev,
                     double* loss_out_host, hipStream_t s) {
  MlpLayout L = mlp_layout();
  char* st = (char*)state_dev;
  batch_forward(st, samples_dev, n, 0, nb, scr, s);
  k_mlp_update<false><<<UPDATE_TILES, 64 * SLICES, 0, s>>>(scr, nb, grad_out_dev, (double*)(st + L.misc), 1, nullptr,
                                                          nullptr, nullptr, nullptr, 0.f, 0.f, 0.f, 0.f, 1.f, 1.f);
  double loss = 0.0;
  if (hipMemcpyAsync(&loss, st + L.misc, sizeof(double), hipMemcpyDeviceToHost, s) != hipSuccess) return MPM_EHIP;
  if (hipStreamSynchronize(s) != hipSuccess) return MPM_EHIP;
  if (loss_out_host) *loss_out_host = loss;
  return hipok(hipGetLastError());
}

int mpm_mlp_grad(void* state_dev, const float* samples_dev, int64_t n, int32_t batch, void* scratch_dev,
                 float* grad_out_dev, double* loss_out_host, void* stream) {
  if (!state_dev || !samples_dev || n < 1 || batch < 1 || !scratch_dev || !grad_out_dev) return MPM_EINVAL;
  const int nb = (int)(n < batch ? n : batch);
  return grad_impl(state_dev, samples_dev, n, nb, aligned_scratch(scratch_dev), grad_out_dev, loss_out_host,
                   (hipStream_t)stream);
}

int mpm_mlp_grad_noalloc(void* state_dev, const float* samples_dev, int64_t n, int32_t batch, float* grad_out_dev,
                         double* loss_out_host, void* stream) {
  if (!state_dev || !samples_dev || n < 1 || batch < 1 || !grad_out_dev) return MPM_EINVAL;
  const int64_t nb = n < batch ? n : batch;
  if (nb > MPM_MLP_NOALLOC_MAX_BATCH) return MPM_EWORKSPACE;
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess) return MPM_EHIP;
  void* scr = noalloc_scratch(dev);
  if (!scr) return MPM_EHIP;
  return grad_impl(state_dev, samples_dev, n, (int)nb, scr, grad_out_dev, loss_out_host, (hipStream_t)stream);
}

int mpm_mlp_train(void* state_dev, const float* samples_dev, int64_t n, int32_t batch, int32_t epochs, float lr,
                  uint64_t seed, void* scratch_dev, double* loss_hist_host, void* stream) {
  if (!state_dev || !samples_dev || n < 1 || batch < 1 || epochs < 1 || !scratch_dev || !(lr > 0.f)) return MPM_EINVAL;
  hipStream_t s = (hipStream_t)stream;
  scratch_dev = aligned_scratch(scratch_dev);
  MlpLayout L = mlp_layout();
  char* st = (char*)state_dev;
  const float b1 = 0.9f, b2 = 0.999f, eps = 1e-8f;
  double t_adam = 0.0;
  {
    double misc[8];
    if (hipMemcpyAsync(misc, st + L.misc, sizeof(misc), hipMemcpyDeviceToHost, s) != hipSuccess) return MPM_EHIP;
    if (hipStreamSynchronize(s) != hipSuccess) return MPM_EHIP;
    t_adam = misc[1];
  }
  std::mt19937_64 rng(seed);
  const int nb = (int)(n < batch ? n : batch);
  const long long steps_per_epoch = (n + nb - 1) / nb;
  for (int ep = 0; ep < epochs; ep++) {
    const long long offset = (long long)(rng() % (unsigned long long)n);
    for (long long k = 0; k < steps_per_epoch; k++) {
      batch_forward(st, samples_dev, n, (offset + k * nb) % n, nb, scratch_dev, s);
      t_adam += 1.0;
      float c1 = (float)(1.0 - pow((double)b1, t_adam)), c2 = (float)(1.0 - pow((double)b2, t_adam));
      k_mlp_update<true><<<UPDATE_TILES, 64 * SLICES, 0, s>>>(
          scratch_dev, nb, nullptr, (double*)(st + L.misc), k == 0 ? 1 : 0, (float*)(st + L.params), (float*)(st + L.m),
          (float*)(st + L.v), (MlpBlob*)(st + L.blob), lr, b1, b2, eps, c1, c2);
    }
    double loss = 0.0;
    if (hipMemcpyAsync(&loss, st + L.misc, sizeof(double), hipMemcpyDeviceToHost, s) != hipSuccess) return MPM_EHIP;
    if (hipStreamSynchronize(s) != hipSuccess) return MPM_EHIP;
    if (loss_hist_host) loss_hist_host[ep] = loss / (double)steps_per_epoch;
  }
  double t_store[2] = {0.0, t_adam};
  if (hipMemcpyAsync(st + L.misc, t_store, sizeof(t_store), hipMemcpyHostToDevice, s) != hipSuccess) return MPM_EHIP;
  return hipok(hipStreamSynchronize(s));
}

int mpm_mlp_predict(const void* state_dev, const float* x_dev, int64_t n, float* y_dev, void* stream) {
  if (!state_dev || !x_dev || !y_dev || n < 1) return MPM_EINVAL;
  hipStream_t s = (hipStream_t)stream;
  MlpLayout L = mlp_layout();
  const char* st = (const char*)state_dev;
  // (the records are those of the training set, 9 floats each; the targets are
  // not read)
  const long long blocks = (n + 63) / 64;
  k_mlp_predict<<<(unsigned)(blocks < 2048 ? blocks : 2048), 256, 0, s>>>((const MlpBlob*)(st + L.blob), x_dev, n, y_dev);
  return hipok(hipStreamSynchronize(s));
}

int mpm_mlp_params(const void* state_dev, float* params_host, void* blob_host, void* stream) {
  if (!state_dev) return MPM_EINVAL;
  hipStream_t s = (hipStream_t)stream;
  MlpLayout L = mlp_layout();
  const char* st = (const char*)state_dev;
  if (params_host && hipMemcpyAsync(params_host, st + L.params, sizeof(float) * MLP_NPARAM, hipMemcpyDeviceToHost, s) != hipSuccess)
    return MPM_EHIP;
  if (blob_host && hipMemcpyAsync(blob_host, st + L.blob, sizeof(MlpBlob), hipMemcpyDeviceToHost, s) != hipSuccess)
    return MPM_EHIP;
  return hipok(hipStreamSynchronize(s));
}

size_t mpm_mlp_blob_offset(void) { return mlp_layout().blob; }

}  // extern "C"
