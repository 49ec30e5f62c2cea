// Pressure-guess network for the primitive recovery: a 5 -> 64 -> 64 -> 1
// multilayer perceptron with SiLU activations, FP32.
//
// Inputs are five invariants of the conserved state, normalised with stored
// means and deviations:
//   x = [ln(tau/D), ln(1 + |S|/D), ln(1 + B^2/D), S.B / (|S||B| + tiny), ln(f(0)/D)]
// with f the recovery's pressure function.
// and the output, de-normalised, is y = ln(p/D); the seed is p0 = D e^y.
// The network only proposes the Newton seed; the FP64 bracketed Newton
// iteration decides the result.
//
// Parameter vector (floats): W1[64][5] b1[64] W2[64][64] b2[64] W3[64] b3
// (4609 weights) followed by mu[5] sd[5] ymu ysd (12 normalisation values).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "physics.hpp"

namespace dgmi {

constexpr int kH = 64;
constexpr int kIn = 5;
constexpr int kOffW1 = 0;
constexpr int kOffB1 = kOffW1 + kH * kIn;  // 320
constexpr int kOffW2 = kOffB1 + kH;        // 384
constexpr int kOffB2 = kOffW2 + kH * kH;   // 4480
constexpr int kOffW3 = kOffB2 + kH;        // 4544
constexpr int kOffB3 = kOffW3 + kH;        // 4608
constexpr int kNumWeights = kOffB3 + 1;    // 4609
constexpr int kOffMu = kNumWeights;        // 4609
constexpr int kOffSd = kOffMu + kIn;       // 4614
constexpr int kOffYmu = kOffSd + kIn;      // 4619
constexpr int kOffYsd = kOffYmu + 1;       // 4620
constexpr int kNumParams = kOffYsd + 1;    // 4621

// Raw (un-normalised) features of a conserved state; B = 0 for hydro.  The
// last one is the pressure function at zero pressure, (g-1) rho eps(0): the
// thermal energy left once the kinetic and magnetic parts are accounted for
// (floored at 1e-300 D where it is not positive or undefined).
template <int SYS>
__host__ __device__ __forceinline__ void mlp_features(const double *u, double g, float *x) {
  const double D = u[0], tau = u[4];
  const double S2 = u[1] * u[1] + u[2] * u[2] + u[3] * u[3];
  double BB = 0.0, SB = 0.0;
  if (SYS == 2) {
    BB = u[5] * u[5] + u[6] * u[6] + u[7] * u[7];
    SB = u[1] * u[5] + u[2] * u[6] + u[3] * u[7];
  }
  double f0 = 0.0;
  if (!pressure_function<SYS>(u, g, 0.0, &f0) || !(f0 > 0.0)) f0 = 1e-300 * D;
  const float Df = (float)D;
  x[0] = logf((float)tau / Df);
  x[1] = log1pf(sqrtf((float)S2) / Df);
  x[2] = log1pf((float)BB / Df);
  x[3] = (float)SB / (sqrtf((float)S2) * sqrtf((float)BB) + 1e-30f);
  x[4] = (float)log(f0 / D);
}

// ---------------------------------------------------------------------
// Inference on the matrix cores.  A wave evaluates 32 samples at a time with
// both layers transposed, [units x inputs] x [inputs x samples] in 32 x 32
// tiles: the result of a product then holds, in lane l, the units
// 8 q + 4 (l / 32) + c (q, c = 0 .. 3; + 32 per row tile) of sample l % 32, and
// after the activation those entries are the very B operand (their units as
// rows, column l % 32) of the next layer's product, if its A operand takes
// the columns of W2 in the same order.  So activations never leave their
// lane, the biases ride along (b1 as the weight of a sixth input 1, b2 as the
// accumulators' start), and the output is a dot product in the lane and one
// exchange of the two half-waves.
//
// Layer 1 (K = 6) runs on v_mfma_f32_32x32x2_f32.  Layer 2, 90% of the
// arithmetic, runs on v_mfma_f32_32x32x16_bf16 with both operands split into
// three bfloat16 parts each, x = hi + mid + lo to 2^-27 x, and the six products
// of parts above 2^-25 accumulated in FP32, so that no accuracy is given up:
// against FP64 the outputs are off by 2.2e-8 (2-norm, training distribution),
// by 2.4e-8 with scalar FP32 sums.
// In FP32 the products alone occupy a SIMD for 4,480 cycles per 32 samples and
// do not run beside the vector unit's 2,800 cycles of activations (half of
// them exp and reciprocal): 90 us for 10^6 samples.  Split, they take 1,920
// cycles on cores the activations leave free: 62 us (before the rounded quotients
// of silu).
typedef float floatx16_t __attribute__((ext_vector_type(16)));
typedef float float4_t __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));

typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef float float2_t __attribute__((ext_vector_type(2)));

// x = f[0] + f[1] + f[2] + e with |e| <= 2^-27 |x|, for two values at once (the
// conversion packs two), into the entries j and j + 1 of f
__device__ __forceinline__ void split3(float2_t x, bf16x8_t *f, int j) {
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    const bf16x2_t h = __builtin_convertvector(x, bf16x2_t);
    f[i][j] = h[0];
    f[i][j + 1] = h[1];
    x[0] -= (float)h[0];
    x[1] -= (float)h[1];
  }
}

struct MlpNet {  // per block: the weights as the products read them
  // W2 by A operand: [row tile m][column step k][lane][part], the eight columns
  // of step k = 2 t + p in lane l being 32 t + 8 (2 p + j / 4) + 4 (l / 32) + j % 4
  bf16x8_t w2[2][4][64][3];
  alignas(16) float b2[kH], w3[kH];
  float w1[kH][kIn + 1];  // W1, and b1 as the sixth column
  float b3, mu[kIn], sd[kIn], isd[kIn], isl[kIn], ymu, ysd;  // 1 / sd = isd + isl
};

__device__ __forceinline__ void mlp_net_load(const float *p, MlpNet *s) {
  for (int t = threadIdx.x; t < 2 * 4 * 64; t += blockDim.x) {
    const int l = t & 63, k = (t >> 6) & 3, m = t >> 8;
    const float *row = p + kOffW2 + (32 * m + (l & 31)) * kH + 32 * (k >> 1) + 16 * (k & 1) + 4 * (l >> 5);
    bf16x8_t f[3];
#pragma unroll
    for (int j = 0; j < 8; j += 2) {
      const int c = 8 * (j >> 2) + (j & 3);
      split3(float2_t{row[c], row[c + 1]}, f, j);
    }
#pragma unroll
    for (int i = 0; i < 3; ++i) s->w2[m][k][l][i] = f[i];
  }
  for (int t = threadIdx.x; t < kH * kIn; t += blockDim.x) s->w1[t / kIn][t % kIn] = p[kOffW1 + t];
  for (int t = threadIdx.x; t < kH; t += blockDim.x) {
    s->w1[t][kIn] = p[kOffB1 + t];
    s->b2[t] = p[kOffB2 + t];
    s->w3[t] = p[kOffW3 + t];
  }
  if (threadIdx.x < kIn) {
    s->mu[threadIdx.x] = p[kOffMu + threadIdx.x];
    s->sd[threadIdx.x] = p[kOffSd + threadIdx.x];
    const double isd = 1.0 / (double)p[kOffSd + threadIdx.x];
    s->isd[threadIdx.x] = (float)isd;
    s->isl[threadIdx.x] = (float)(isd - (double)(float)isd);
  }
  if (threadIdx.x == 0) {
    s->b3 = p[kOffB3];
    s->ymu = p[kOffYmu];
    s->ysd = p[kOffYsd];
  }
}

// x sigmoid(x).  ROUNDED: the correctly rounded quotient x / (1 + e^-x), for
// mlp_forward, whose outputs are results: the hardware's reciprocal, one
// correction, the special cases put right; both sides by a quarter, so that the
// reciprocal is a normal number to the end of the exponential's range.  Else the
// reciprocal alone (within one ulp, 0 below -87), for the recovery's seed.
template <bool ROUNDED>
__device__ __forceinline__ float silu(float x) {
  const float e = __expf(-x);
  if (!ROUNDED) return x * __builtin_amdgcn_rcpf(1.0f + e);
  const float n = 0.25f * x, d = fmaf(0.25f, e, 0.25f);
  const float r = __builtin_amdgcn_rcpf(d), q = n * r;
  return __builtin_amdgcn_div_fixupf(fmaf(fmaf(-q, d, n), r, q), d, n);
}

// Normalised output for 32 samples, all 64 lanes of the wave together: lane l
// passes inputs l / 32, 2 + l / 32 and 4 + l / 32 (the sixth being 1) of sample
// l % 32 and receives that sample's output.
template <bool ROUNDED>
__device__ __forceinline__ float mlp_net32(const MlpNet *s, float x0, float x1, float x2) {
  const int r = threadIdx.x & 31, h = (threadIdx.x >> 5) & 1;
  const float xb[3] = {x0, x1, x2};
  floatx16_t H[2], E[2];
  // the weights are read from LDS where they are used (hoisted out of the
  // caller's loop, as the compiler would, they take 130 registers)
#define MLP_KEEP_LOADS() asm volatile("" ::: "memory")
  MLP_KEEP_LOADS();
#pragma unroll
  for (int m = 0; m < 2; ++m)
#pragma unroll
    for (int a = 0; a < 16; ++a) H[m][a] = 0.0f;
#pragma unroll
  for (int ks = 0; ks < 3; ++ks)
#pragma unroll
    for (int m = 0; m < 2; ++m)
      H[m] = __builtin_amdgcn_mfma_f32_32x32x2f32(s->w1[32 * m + r][2 * ks + h], xb[ks], H[m], 0, 0, 0);
#pragma unroll
  for (int m = 0; m < 2; ++m)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const float4_t b = *reinterpret_cast<const float4_t *>(&s->b2[32 * m + 8 * q + 4 * h]);
#pragma unroll
      for (int c = 0; c < 4; ++c) E[m][4 * q + c] = b[c];
    }
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    MLP_KEEP_LOADS();
    const int l = threadIdx.x & 63;
    bf16x8_t w[2][3], f[3];
#pragma unroll
    for (int m = 0; m < 2; ++m)
#pragma unroll
      for (int i = 0; i < 3; ++i) w[m][i] = s->w2[m][k][l][i];
#pragma unroll
    for (int j = 0; j < 8; j += 2) {
      const int a = 8 * (k & 1) + j;
      split3(float2_t{silu<ROUNDED>(H[k >> 1][a]), silu<ROUNDED>(H[k >> 1][a + 1])}, f, j);
    }
    // the smallest products first
#pragma unroll
    for (int o = 2; o >= 0; --o)
#pragma unroll
      for (int i = 0; i <= o; ++i)
#pragma unroll
        for (int m = 0; m < 2; ++m)
          E[m] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(w[m][i], f[o - i], E[m], 0, 0, 0);
  }
  MLP_KEEP_LOADS();
#undef MLP_KEEP_LOADS
  float y[2] = {0.0f, 0.0f};
#pragma unroll
  for (int m = 0; m < 2; ++m)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const float4_t w = *reinterpret_cast<const float4_t *>(&s->w3[32 * m + 8 * q + 4 * h]);
#pragma unroll
      for (int c = 0; c < 4; ++c) y[m] += w[c] * silu<ROUNDED>(E[m][4 * q + c]);
    }
  const float yl = y[0] + y[1];
  return yl + __shfl_xor(yl, 32) + s->b3;
}

// Recovery seed D exp(y) of this lane's point, all 64 lanes of a wave together
// (every lane must take part): its points as two passes of 32.  The features are
// the training's own (with hardware FP32 logarithms, roots and reciprocals in
// their place 4x10^6 SRMHD points took 349 us instead of 410, but the seeds
// were undefined where D has no FP32 reciprocal).
template <int SYS>
__device__ __forceinline__ double mlp_seed_wave(const MlpNet *s, const double *u, double g) {
  const bool lo = (threadIdx.x & 63) < 32;
  float x[kIn];
  mlp_features<SYS>(u, g, x);
#pragma unroll
  for (int i = 0; i < kIn; ++i) {
    const float c = x[i] - s->mu[i];
    x[i] = fmaf(c, s->isl[i], c * s->isd[i]);
  }
  // an input pair (k, k + 1): each half-wave needs its own row of the pair
  // for both passes, the other half holds it for one of them
  const float o0 = __shfl_xor(lo ? x[1] : x[0], 32), o1 = __shfl_xor(lo ? x[3] : x[2], 32), o2 = __shfl_xor(x[4], 32);
  float y = 0.0f;
#pragma unroll 1
  for (int p = 0; p < 2; ++p) {  // (rolled: one pass's registers at a time)
    const bool own = lo == (p == 0);
    const float x0 = own ? (lo ? x[0] : x[1]) : o0, x1 = own ? (lo ? x[2] : x[3]) : o1;
    const float yp = mlp_net32<false>(s, x0, x1, lo ? (p == 0 ? x[4] : o2) : 1.0f);
    if (own) y = yp;
  }
  y = y * s->ysd + s->ymu;
  // the seed needs no more than FP32 (the FP64 iteration decides the result):
  // exp y = 2^t (1 + r ln 2), r the rounding of t = y log2 e
  const float t = y * 1.44269504f;
  const float r = fmaf(y, 1.44269504f, -t) + y * 1.92596299e-8f;
  const float e = __builtin_amdgcn_exp2f(t);
  return u[0] * (double)fmaf(e, r * 0.693147181f, e);
}

}  // namespace dgmi
