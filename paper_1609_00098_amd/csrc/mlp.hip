// Pressure-guess network: features, inference, training (forward, backward,
// Adam), all FP32, all in HIP kernels.
//
// Training: one launch forms a batch's gradient, one row of sums per
// workgroup, a second adds the rows in a fixed order (bit-reproducible, no
// atomics) and, in training, updates the weights (Adam).
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>
#include <cstring>
#include <new>
#include <vector>

#include "../../include/dgmi.h"
#include "kernels.hpp"
#include "mlp.hpp"
#include "physics.hpp"

namespace dgmi {

__device__ __forceinline__ float sigm(float a) { return 1.0f / (1.0f + expf(-a)); }

template <int SYS>
__global__ void __launch_bounds__(256) features_kernel(const double *U, const double *prim, int64_t n, double g,
                                                       float *x, float *t) {
  constexpr int NV = SysTraits<SYS>::nv;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; q < n; q += stride) {
    double u[NV];
#pragma unroll
    for (int v = 0; v < NV; ++v) u[v] = U[v * n + q];
    float f[kIn];
    mlp_features<SYS>(u, g, f);
#pragma unroll
    for (int i = 0; i < kIn; ++i) x[i * n + q] = f[i];
    if (t) t[q] = (float)log(prim[4 * n + q] / u[0]);  // target ln(p/D)
  }
}

// Network output for raw features x[5][B]: y = de-normalised ln(p/D).  One
// wave per 32 samples at a time (mlp_net32); 1,024 workgroups of four waves
// fill the chip at the registers this takes, each loading the weights once.
// (A thread per sample with the weights from LDS: 165 us for 10^6 samples; now
// 72 us, 62 of them with the activations' quotients by the reciprocal alone.)
constexpr int kForwardBlocks = 1024;
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4))) forward_kernel(const float *params, const float *x, int64_t ld, int64_t B,
                                                      float *y) {
  __shared__ MlpNet net;
  mlp_net_load(params, &net);
  __syncthreads();
  const int l = threadIdx.x & 63, r = l & 31, h = l >> 5;
  const int64_t stride = (int64_t)gridDim.x * 128;
  for (int64_t s0 = (int64_t)blockIdx.x * 128 + (threadIdx.x >> 6) * 32; s0 < B; s0 += stride) {
    const int64_t q = s0 + r < B ? s0 + r : B - 1;
    float xb[3];
#pragma unroll
    for (int ks = 0; ks < 3; ++ks) {
      const int k = 2 * ks + h;
      xb[ks] = k < kIn ? (x[k * ld + q] - net.mu[k]) / net.sd[k] : 1.0f;
    }
    const float yn = mlp_net32<true>(&net, xb[0], xb[1], xb[2]);
    if (h == 0 && s0 + r < B) y[q] = yn * net.ysd + net.ymu;
  }
}

// Loss = mean over the batch of (y_n - t_n)^2 in normalised units, and its
// gradient.  A workgroup of four waves walks tiles of kTile = 32 samples and
// keeps its sums over them in registers; at the end it writes one row of
// kPartialLd floats: the gradient sums, then its squared-error sum.
//
// The four 64-wide products of a tile run on v_mfma_f32_16x16x4_f32 (FP32
// operands and accumulation).  Wave w owns the hidden units 16 w .. 16 w + 15
// of both layers: in the 16 x 16 result layout lane l holds unit
// u = 16 w + l % 16 of the samples s = 16 t + 4 (l / 16) + a (t = 0, 1;
// a = 0 .. 3), the same eight values for A1, H1, A2, dA2 and dA1, so that all
// activations and their derivatives are lane-local.  W2 stays in registers
// as the operand fragments of both products that use it; dA2 is its own A
// operand in dW2 = dA2^T H1.  Only H1 and dA2 pass through LDS, between the
// waves (rows of 68 floats: no bank conflicts in either read direction).
// Contraction indices are taken in the order that gives every lane four
// consecutive floats of a row for four products (kk below).
//
// A tile is a chain of about 100 matrix instructions and four barriers; a
// batch of 8,192 is 256 tiles, one per CU.  Bound by that chain's latency.
// Scalar FP32 code on tiles of 64 samples with every operand read from LDS
// took 33.2 us for 8,192 samples, this 8 to 10 us.
constexpr int kTile = 32;            // samples per tile
constexpr int kTrainThreads = 256;
constexpr int kTrainBlocks = 512;    // two workgroups per CU; larger batches loop
constexpr int kPartialLd = 4672;     // floats per workgroup row: 73 x 64 >= kNumWeights + 1
constexpr int kLossCol = kNumWeights;
constexpr int kRowH = 68;

typedef float floatx4_t __attribute__((ext_vector_type(4)));

__global__ void __launch_bounds__(kTrainThreads) grad_tile_kernel(const float *params, const float *x, int64_t ld,
                                                                   const float *t, int64_t B, float *partial) {
  __shared__ __align__(16) float sX[kTile * 8];      // normalised features, 1 (the bias), 0, 0
  __shared__ __align__(16) float sH[kTile * kRowH];  // H1
  __shared__ __align__(16) float sG[kTile * kRowH];  // dA2
  __shared__ float sT[kTile], sY[4][kTile];
  const int tid = threadIdx.x, w = tid >> 6, l = tid & 63, u16 = l & 15, g = l >> 4;
  const int u = 16 * w + u16;
  // operand fragments: W1 with b1 as its sixth column, W2 by rows (layer 2)
  // and by columns (dH1)
  float w1f[2];
#pragma unroll
  for (int ks = 0; ks < 2; ++ks) {
    const int k = 4 * ks + g;
    w1f[ks] = k < kIn ? params[kOffW1 + u * kIn + k] : (k == kIn ? params[kOffB1 + u] : 0.0f);
  }
  floatx4_t w2r[4], w2c[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    w2r[q] = *reinterpret_cast<const floatx4_t *>(params + kOffW2 + u * kH + 16 * q + 4 * g);
#pragma unroll
    for (int r = 0; r < 4; ++r) w2c[q][r] = params[kOffW2 + (16 * q + 4 * g + r) * kH + u];
  }
  const float b2 = params[kOffB2 + u], w3 = params[kOffW3 + u], b3 = params[kOffB3];
  const float ymu = params[kOffYmu], ysd = params[kOffYsd];
  const float inv_b = 1.0f / (float)B;
  floatx4_t dw2[4];  // dW2[16 w + 4 g + a][16 n + u16]
  float dw1[kIn + 1], dw3 = 0.0f, db2 = 0.0f, db3 = 0.0f, se = 0.0f;
#pragma unroll
  for (int n = 0; n < 4; ++n) dw2[n] = floatx4_t{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
  for (int k = 0; k <= kIn; ++k) dw1[k] = 0.0f;
  const int64_t ntiles = (B + kTile - 1) / kTile;
  for (int64_t tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
    const int64_t s0 = tile * kTile;
    {
      const int s = tid & (kTile - 1), i = tid >> 5;  // feature i of sample s
      const bool in = s0 + s < B;
      if (i < kIn)
        sX[s * 8 + i] = in ? (x[i * ld + s0 + s] - params[kOffMu + i]) / params[kOffSd + i] : 0.0f;
      else
        sX[s * 8 + i] = i == kIn ? 1.0f : 0.0f;
      if (i == kIn) sT[s] = in ? (t[s0 + s] - ymu) / ysd : 0.0f;
    }
    __syncthreads();
    // layer 1 and its activation
    float a1[2][4], h1[2][4];
#pragma unroll
    for (int tt = 0; tt < 2; ++tt) {
      floatx4_t c = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
      for (int ks = 0; ks < 2; ++ks)
        c = __builtin_amdgcn_mfma_f32_16x16x4f32(sX[(16 * tt + u16) * 8 + 4 * ks + g], w1f[ks], c, 0, 0, 0);
#pragma unroll
      for (int a = 0; a < 4; ++a) {
        a1[tt][a] = c[a];
        h1[tt][a] = c[a] * sigm(c[a]);
        sH[(16 * tt + 4 * g + a) * kRowH + u] = h1[tt][a];
      }
    }
    __syncthreads();
    // layer 2: A2[s][u] = b2 + sum_k H1[s][k] W2[u][k]
    floatx4_t a2[2];
#pragma unroll
    for (int tt = 0; tt < 2; ++tt) a2[tt] = floatx4_t{b2, b2, b2, b2};
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      floatx4_t hr[2];
#pragma unroll
      for (int tt = 0; tt < 2; ++tt)
        hr[tt] = *reinterpret_cast<const floatx4_t *>(sH + (16 * tt + u16) * kRowH + 16 * q + 4 * g);
#pragma unroll
      for (int kk = 0; kk < 4; ++kk)
#pragma unroll
        for (int tt = 0; tt < 2; ++tt)
          a2[tt] = __builtin_amdgcn_mfma_f32_16x16x4f32(hr[tt][kk], w2r[q][kk], a2[tt], 0, 0, 0);
    }
    // output: this wave's part of sum_u W3[u] silu(A2[s][u])
    float sg[2][4];
#pragma unroll
    for (int tt = 0; tt < 2; ++tt)
#pragma unroll
      for (int a = 0; a < 4; ++a) {
        sg[tt][a] = sigm(a2[tt][a]);
        float y = w3 * (a2[tt][a] * sg[tt][a]);
#pragma unroll
        for (int off = 1; off < 16; off <<= 1) y += __shfl_xor(y, off);
        if (u16 == 0) sY[w][16 * tt + 4 * g + a] = y;
      }
    __syncthreads();
    // dL/dy, then dA2 = dy W3 silu'(A2)
    float g2[2][4];
#pragma unroll
    for (int tt = 0; tt < 2; ++tt)
#pragma unroll
      for (int a = 0; a < 4; ++a) {
        const int s = 16 * tt + 4 * g + a;
        float r = ((b3 + sY[0][s]) + (sY[1][s] + sY[2][s])) + sY[3][s] - sT[s];
        r = s0 + s < B ? r : 0.0f;
        se += r * r;
        const float dy = 2.0f * r * inv_b, v = a2[tt][a], sv = sg[tt][a];
        db3 += dy;
        dw3 += dy * (v * sv);
        g2[tt][a] = dy * w3 * sv * (1.0f + v * (1.0f - sv));
        db2 += g2[tt][a];
        sG[s * kRowH + u] = g2[tt][a];
      }
    __syncthreads();
    // dW2[j][i] += sum_s dA2[s][j] H1[s][i]: rows j of this wave, every i
#pragma unroll
    for (int tt = 0; tt < 2; ++tt)
#pragma unroll
      for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int n = 0; n < 4; ++n)
          dw2[n] = __builtin_amdgcn_mfma_f32_16x16x4f32(g2[tt][a], sH[(16 * tt + 4 * g + a) * kRowH + 16 * n + u16],
                                                        dw2[n], 0, 0, 0);
    // dH1[s][u] = sum_j dA2[s][j] W2[j][u], then dA1 = dH1 silu'(A1)
    floatx4_t dh[2];
#pragma unroll
    for (int tt = 0; tt < 2; ++tt) dh[tt] = floatx4_t{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      floatx4_t gr[2];
#pragma unroll
      for (int tt = 0; tt < 2; ++tt)
        gr[tt] = *reinterpret_cast<const floatx4_t *>(sG + (16 * tt + u16) * kRowH + 16 * q + 4 * g);
#pragma unroll
      for (int kk = 0; kk < 4; ++kk)
#pragma unroll
        for (int tt = 0; tt < 2; ++tt)
          dh[tt] = __builtin_amdgcn_mfma_f32_16x16x4f32(gr[tt][kk], w2c[q][kk], dh[tt], 0, 0, 0);
    }
#pragma unroll
    for (int tt = 0; tt < 2; ++tt)
#pragma unroll
      for (int a = 0; a < 4; ++a) {
        const float v = a1[tt][a], sv = sigm(v);
        const float d1 = dh[tt][a] * sv * (1.0f + v * (1.0f - sv));
        const float *xs = sX + (16 * tt + 4 * g + a) * 8;
#pragma unroll
        for (int k = 0; k <= kIn; ++k) dw1[k] += d1 * xs[k];  // the sixth column is db1
      }
    __syncthreads();
  }
  // sums over the four sample groups of a unit, then this workgroup's row
#pragma unroll
  for (int off = 16; off < 64; off <<= 1) {
#pragma unroll
    for (int k = 0; k <= kIn; ++k) dw1[k] += __shfl_xor(dw1[k], off);
    dw3 += __shfl_xor(dw3, off);
    db2 += __shfl_xor(db2, off);
    db3 += __shfl_xor(db3, off);
    se += __shfl_xor(se, off);
  }
  float *part = partial + (int64_t)blockIdx.x * kPartialLd;
#pragma unroll
  for (int n = 0; n < 4; ++n)
#pragma unroll
    for (int a = 0; a < 4; ++a) part[kOffW2 + (16 * w + 4 * g + a) * kH + 16 * n + u16] = dw2[n][a];
  if (g == 0) {
#pragma unroll
    for (int k = 0; k < kIn; ++k) part[kOffW1 + u * kIn + k] = dw1[k];
    part[kOffB1 + u] = dw1[kIn];
    part[kOffB2 + u] = db2;
    part[kOffW3 + u] = dw3;
  }
  if (tid == 0) {
    part[kOffB3] = db3;
    part[kLossCol] = se;
  }
}

// grad[k] = sum over workgroups of partial[b][k], in a fixed order: sixteen
// waves take every sixteenth row each, 64 columns per workgroup; the loss is
// column kLossCol over the batch.  ADAM: the weights are updated in the same
// launch.  (One thread per column over all rows took 37.8 us for 128 rows of
// 4,609 columns, this 2 to 4 us for 256.)
struct AdamArgs {
  float *params, *m, *v;
  float lr, bc1, bc2;
};

template <bool ADAM>
__global__ void __launch_bounds__(1024) reduce_partials_kernel(const float *partial, int nblk, float *grad, float inv_b,
                                                               float *loss, AdamArgs A) {
  __shared__ float red[16][64];
  const int w = threadIdx.x >> 6, l = threadIdx.x & 63;
  const int k = blockIdx.x * 64 + l;
  float s = 0.0f;
#pragma unroll 8
  for (int b = w; b < nblk; b += 16) s += partial[(int64_t)b * kPartialLd + k];
  red[w][l] = s;
  __syncthreads();
  if (w != 0 || k > kLossCol) return;
#pragma unroll
  for (int i = 0; i < 8; ++i) red[i][l] += red[i + 8][l];
#pragma unroll
  for (int i = 0; i < 4; ++i) red[i][l] += red[i + 4][l];
  const float gk = (red[0][l] + red[2][l]) + (red[1][l] + red[3][l]);
  if (k == kLossCol) {
    if (loss) *loss = gk * inv_b;
    return;
  }
  grad[k] = gk;
  if (ADAM) {
    const float mk = 0.9f * A.m[k] + 0.1f * gk;
    const float vk = 0.999f * A.v[k] + 0.001f * gk * gk;
    A.m[k] = mk;
    A.v[k] = vk;
    A.params[k] -= A.lr * (mk / A.bc1) / (sqrtf(vk / A.bc2) + 1e-8f);
  }
}

// Mean and standard deviation of the raw features and targets, accumulated in
// FP64: every workgroup sums x and x^2 of the six columns over a grid-stride
// range into fit[block][12], and one more workgroup adds those in a fixed
// order.  Bound by HBM (24 B per sample); one workgroup for the whole set had
// kept 255 of the 256 CUs idle: 5.34 ms for 10^6
// samples, now 8.4 us for the sums (2.9 TB/s) and 3.9 us for the rest.
constexpr int kFitBlocks = 512;  // two workgroups per CU
constexpr int kFitSums = 2 * (kIn + 1);

__global__ void __launch_bounds__(256) fit_sums_kernel(const float *x, int64_t ld, const float *t, int64_t n,
                                                       double *fit) {
  __shared__ double red[4][kFitSums];
  double s[kFitSums];
#pragma unroll
  for (int c = 0; c < kFitSums; ++c) s[c] = 0.0;
  const int64_t stride = (int64_t)gridDim.x * 256;
#pragma unroll 2
  for (int64_t q = (int64_t)blockIdx.x * 256 + threadIdx.x; q < n; q += stride) {
#pragma unroll
    for (int c = 0; c <= kIn; ++c) {
      const double v = c < kIn ? x[c * ld + q] : t[q];
      s[2 * c] += v;
      s[2 * c + 1] += v * v;
    }
  }
#pragma unroll
  for (int c = 0; c < kFitSums; ++c)
    for (int off = 32; off > 0; off >>= 1) s[c] += __shfl_xor(s[c], off);
  if ((threadIdx.x & 63) == 0) {
#pragma unroll
    for (int c = 0; c < kFitSums; ++c) red[threadIdx.x >> 6][c] = s[c];
  }
  __syncthreads();
  if (threadIdx.x < kFitSums) {
    const int c = threadIdx.x;
    fit[blockIdx.x * kFitSums + c] = (red[0][c] + red[1][c]) + (red[2][c] + red[3][c]);
  }
}

// One wave per sum.
__global__ void __launch_bounds__(64 * kFitSums) fit_finish_kernel(const double *fit, int nblk, int64_t n,
                                                                  float *params) {
  __shared__ double sum[kFitSums];
  const int c = threadIdx.x >> 6, l = threadIdx.x & 63;
  double s = 0.0;
  for (int b = l; b < nblk; b += 64) s += fit[b * kFitSums + c];
  for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off);
  if (l == 0) sum[c] = s;
  __syncthreads();
  if (threadIdx.x <= kIn) {
    const int k = threadIdx.x;
    const double mean = sum[2 * k] / (double)n;
    const double var = sum[2 * k + 1] / (double)n - mean * mean;
    params[k < kIn ? kOffMu + k : kOffYmu] = (float)mean;
    params[k < kIn ? kOffSd + k : kOffYsd] = (float)(var > 1e-24 ? sqrt(var) : 1.0);
  }
}

}  // namespace dgmi

namespace {
dgmi_status merr(dgmi_status st, const char *msg) { return (dgmi_status)dgmi::set_error(st, msg); }
uint64_t splitmix64(uint64_t &s) {
  uint64_t z = (s += 0x9E3779B97F4A7C15ull);
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  return z ^ (z >> 31);
}
void free_all(dgmi_mlp *m) {
  (void)hipFree(m->params);
  (void)hipFree(m->grad);
  (void)hipFree(m->adam_m);
  (void)hipFree(m->adam_v);
  (void)hipFree(m->partial);
  (void)hipFree(m->fit);
  delete m;
}
// Rows of partial gradients, allocated on first use: kTrainBlocks rows serve
// every batch size.
dgmi_status ensure_partials(dgmi_mlp *m) {
  if (m->partial) return DGMI_OK;
  if (hipMalloc(&m->partial, sizeof(float) * dgmi::kPartialLd * dgmi::kTrainBlocks) != hipSuccess) {
    (void)hipGetLastError();
    m->partial = nullptr;
    return merr(DGMI_ENOMEM, "mlp: partial buffer allocation failed");
  }
  return DGMI_OK;
}
}  // namespace

extern "C" {

dgmi_status mlp_create(dgmi_mlp **out, uint64_t seed, void *stream) {
  using namespace dgmi;
  if (!out) return merr(DGMI_EINVAL, "mlp_create: null argument");
  dgmi_mlp *m = new (std::nothrow) dgmi_mlp();
  if (!m) return merr(DGMI_ENOMEM, "mlp_create: out of host memory");
  (void)hipGetDevice(&m->device);
  std::vector<float> h(kNumParams, 0.0f);
  uint64_t s = seed * 0x2545F4914F6CDD1Dull + 1;
  auto uni = [&](float bound) {
    const double u = (double)(splitmix64(s) >> 11) * (1.0 / 9007199254740992.0);
    return (float)((2.0 * u - 1.0) * bound);
  };
  const float b1 = 1.0f / std::sqrt((float)kIn), b2 = 1.0f / std::sqrt((float)kH);
  for (int k = 0; k < kH * kIn; ++k) h[kOffW1 + k] = uni(b1);
  for (int k = 0; k < kH; ++k) h[kOffB1 + k] = uni(b1);
  for (int k = 0; k < kH * kH; ++k) h[kOffW2 + k] = uni(b2);
  for (int k = 0; k < kH; ++k) h[kOffB2 + k] = uni(b2);
  for (int k = 0; k < kH; ++k) h[kOffW3 + k] = uni(b2);
  h[kOffB3] = 0.0f;
  for (int i = 0; i < kIn; ++i) { h[kOffMu + i] = 0.0f; h[kOffSd + i] = 1.0f; }
  h[kOffYmu] = 0.0f;
  h[kOffYsd] = 1.0f;
  if (hipMalloc(&m->params, sizeof(float) * kNumParams) != hipSuccess ||
      hipMalloc(&m->grad, sizeof(float) * kNumWeights) != hipSuccess ||
      hipMalloc(&m->adam_m, sizeof(float) * kNumWeights) != hipSuccess ||
      hipMalloc(&m->adam_v, sizeof(float) * kNumWeights) != hipSuccess ||
      hipMalloc(&m->fit, sizeof(double) * kFitBlocks * kFitSums) != hipSuccess) {
    (void)hipGetLastError();
    free_all(m);
    return merr(DGMI_ENOMEM, "mlp_create: device allocation failed");
  }
  const hipStream_t cs = (hipStream_t)stream;
  if (hipMemcpyAsync(m->params, h.data(), sizeof(float) * kNumParams, hipMemcpyHostToDevice, cs) != hipSuccess ||
      hipMemsetAsync(m->adam_m, 0, sizeof(float) * kNumWeights, cs) != hipSuccess ||
      hipMemsetAsync(m->adam_v, 0, sizeof(float) * kNumWeights, cs) != hipSuccess ||
      hipStreamSynchronize(cs) != hipSuccess) {
    (void)hipGetLastError();
    (void)hipStreamSynchronize(cs);
    free_all(m);
    return merr(DGMI_EHIP, "mlp_create: upload failed");
  }
  *out = m;
  return DGMI_OK;
}

dgmi_status mlp_destroy(dgmi_mlp *m) {
  if (!m) return DGMI_OK;
  (void)hipDeviceSynchronize();
  free_all(m);
  return DGMI_OK;
}

dgmi_status mlp_get(const dgmi_mlp *m, float *params_out, void *stream) {
  if (!m || !params_out) return merr(DGMI_EINVAL, "mlp_get: null argument");
  if (hipMemcpyAsync(params_out, m->params, sizeof(float) * dgmi::kNumParams, hipMemcpyDeviceToDevice,
                     (hipStream_t)stream) != hipSuccess)
    return merr(DGMI_EHIP, "mlp_get: copy failed");
  return DGMI_OK;
}

dgmi_status mlp_set(dgmi_mlp *m, const float *params_in, void *stream) {
  if (!m || !params_in) return merr(DGMI_EINVAL, "mlp_set: null argument");
  if (hipMemcpyAsync(m->params, params_in, sizeof(float) * dgmi::kNumParams, hipMemcpyDeviceToDevice,
                     (hipStream_t)stream) != hipSuccess)
    return merr(DGMI_EHIP, "mlp_set: copy failed");
  m->step = 0;
  if (hipMemsetAsync(m->adam_m, 0, sizeof(float) * dgmi::kNumWeights, (hipStream_t)stream) != hipSuccess ||
      hipMemsetAsync(m->adam_v, 0, sizeof(float) * dgmi::kNumWeights, (hipStream_t)stream) != hipSuccess)
    return merr(DGMI_EHIP, "mlp_set: reset failed");
  return DGMI_OK;
}

dgmi_status mlp_features(int32_t system, double gamma, const double *U, const double *prim, int64_t n, float *x_out,
                         float *t_out, void *stream) {
  using namespace dgmi;
  if (system != 1 && system != 2) return merr(DGMI_EINVAL, "mlp_features: relativistic systems only");
  if (!U || !x_out || n < 0 || (t_out && !prim) || !(gamma > 1.0 && gamma <= 2.0))
    return merr(DGMI_EINVAL, "mlp_features: bad argument");
  if (n == 0) return DGMI_OK;
  const int64_t b = (n + 255) / 256;
  const int grid = (int)(b < 65536 ? b : 65536);
  if (system == 1)
    hipLaunchKernelGGL(features_kernel<kSR>, dim3(grid), dim3(256), 0, (hipStream_t)stream, U, prim, n, gamma, x_out,
                       t_out);
  else
    hipLaunchKernelGGL(features_kernel<kMHD>, dim3(grid), dim3(256), 0, (hipStream_t)stream, U, prim, n, gamma, x_out,
                       t_out);
  return hipGetLastError() == hipSuccess ? DGMI_OK : merr(DGMI_EHIP, "mlp_features: launch failed");
}

dgmi_status mlp_fit_normalization(dgmi_mlp *m, const float *x, int64_t ldx, const float *t, int64_t n, void *stream) {
  if (!m || !x || !t || n < 2 || ldx < n) return merr(DGMI_EINVAL, "mlp_fit_normalization: bad argument");
  // (four samples per thread before another workgroup pays)
  const int64_t want = (n + 1023) / 1024;
  const int nblk = (int)(want < dgmi::kFitBlocks ? want : dgmi::kFitBlocks);
  hipLaunchKernelGGL(dgmi::fit_sums_kernel, dim3(nblk), dim3(256), 0, (hipStream_t)stream, x, ldx, t, n, m->fit);
  hipLaunchKernelGGL(dgmi::fit_finish_kernel, dim3(1), dim3(64 * dgmi::kFitSums), 0, (hipStream_t)stream, m->fit, nblk,
                     n, m->params);
  return hipGetLastError() == hipSuccess ? DGMI_OK : merr(DGMI_EHIP, "mlp_fit_normalization: launch failed");
}

dgmi_status mlp_forward(const dgmi_mlp *m, const float *x, int64_t ldx, int64_t batch, float *y_out, void *stream) {
  if (!m || !x || !y_out || batch < 0 || ldx < batch) return merr(DGMI_EINVAL, "mlp_forward: bad argument");
  if (batch == 0) return DGMI_OK;
  const int64_t b = (batch + 127) / 128;
  const int grid = (int)(b < dgmi::kForwardBlocks ? b : dgmi::kForwardBlocks);
  hipLaunchKernelGGL(dgmi::forward_kernel, dim3(grid), dim3(256), 0, (hipStream_t)stream, m->params, x, ldx, batch,
                     y_out);
  return hipGetLastError() == hipSuccess ? DGMI_OK : merr(DGMI_EHIP, "mlp_forward: launch failed");
}

// The gradient of one batch into grads, and the loss; adam: also the update
// of the weights.
static dgmi_status grad_impl(dgmi_mlp *m, const float *x, int64_t ldx, const float *t, int64_t batch, float *grads,
                             float *loss, const dgmi::AdamArgs *adam, hipStream_t s) {
  using namespace dgmi;
  const dgmi_status st = ensure_partials(m);
  if (st != DGMI_OK) return st;
  const int64_t ntiles = (batch + kTile - 1) / kTile;
  const int nblk = (int)(ntiles < kTrainBlocks ? ntiles : kTrainBlocks);
  hipLaunchKernelGGL(grad_tile_kernel, dim3(nblk), dim3(kTrainThreads), 0, s, m->params, x, ldx, t, batch, m->partial);
  const dim3 grid(kPartialLd / 64), block(1024);
  const float inv_b = 1.0f / (float)batch;
  if (adam)
    hipLaunchKernelGGL(reduce_partials_kernel<true>, grid, block, 0, s, m->partial, nblk, grads, inv_b, loss, *adam);
  else
    hipLaunchKernelGGL(reduce_partials_kernel<false>, grid, block, 0, s, m->partial, nblk, grads, inv_b, loss,
                       AdamArgs{});
  return hipGetLastError() == hipSuccess ? DGMI_OK : merr(DGMI_EHIP, "mlp: gradient launch failed");
}

static bool batch_ok(int64_t batch, int64_t ldx) { return batch >= 1 && batch <= ((int64_t)1 << 24) && ldx >= batch; }

dgmi_status mlp_grad(dgmi_mlp *m, const float *x, int64_t ldx, const float *t, int64_t batch, float *grads_out,
                     float *loss_out, void *stream) {
  if (!m || !x || !t || !grads_out || !batch_ok(batch, ldx)) return merr(DGMI_EINVAL, "mlp_grad: bad argument");
  return grad_impl(m, x, ldx, t, batch, grads_out, loss_out, nullptr, (hipStream_t)stream);
}

static dgmi_status train_impl(dgmi_mlp *m, const float *x, int64_t ldx, const float *t, int64_t batch, float lr,
                              float *loss, hipStream_t s) {
  const double step = (double)(m->step + 1);
  const dgmi::AdamArgs a{m->params, m->adam_m, m->adam_v, lr, (float)(1.0 - std::pow(0.9, step)),
                         (float)(1.0 - std::pow(0.999, step))};
  const dgmi_status st = grad_impl(m, x, ldx, t, batch, m->grad, loss, &a, s);
  if (st == DGMI_OK) m->step += 1;
  return st;
}

dgmi_status mlp_train_step(dgmi_mlp *m, const float *x, int64_t ldx, const float *t, int64_t batch, float lr,
                           float *loss_out, void *stream) {
  if (!m || !x || !t || !batch_ok(batch, ldx) || !(lr > 0.0f)) return merr(DGMI_EINVAL, "mlp_train_step: bad argument");
  return train_impl(m, x, ldx, t, batch, lr, loss_out, (hipStream_t)stream);
}

dgmi_status mlp_train(dgmi_mlp *m, const float *x, const float *t, int64_t n, int64_t batch, int32_t epochs,
                      float lr0, float lr1, float *loss_hist, void *stream) {
  if (!m || !x || !t || batch < 1 || batch > ((int64_t)1 << 24) || n < batch || epochs < 1 || !(lr0 > 0.0f) ||
      !(lr1 > 0.0f))
    return merr(DGMI_EINVAL, "mlp_train: bad argument");
  hipStream_t s = (hipStream_t)stream;
  const int64_t per_epoch = n / batch;
  const int64_t total = per_epoch * epochs;
  int64_t k = 0;
  for (int32_t ep = 0; ep < epochs; ++ep) {
    for (int64_t b = 0; b < per_epoch; ++b, ++k) {
      const double c = 0.5 * (1.0 + std::cos(M_PI * (double)k / (double)(total > 1 ? total - 1 : 1)));
      const float lr = (float)(lr1 + (lr0 - lr1) * c);
      const dgmi_status st =
          train_impl(m, x + b * batch, n, t + b * batch, batch, lr, loss_hist ? loss_hist + k : nullptr, s);
      if (st != DGMI_OK) return st;
    }
  }
  return DGMI_OK;
}

}  // extern "C"
