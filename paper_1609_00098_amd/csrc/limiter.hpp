// Device pieces of the minmod-family slope limiter shared by the limiter
// kernels and the limited RK stage kernel (high-resolution shock-capturing
// section: eqs. MinModB, MinMod, and the element moments they need).
#pragma once
#include "kernels.hpp"

namespace dgmi {

__device__ __forceinline__ double mm_sign(double a) { return a > 0.0 ? 1.0 : (a < 0.0 ? -1.0 : 0.0); }

// m(a1, a2, a3): the common sign times the smallest magnitude, or 0.
__device__ __forceinline__ double minmod3(double a1, double a2, double a3) {
  const double s = mm_sign(a1);
  if (s == 0.0 || mm_sign(a2) != s || mm_sign(a3) != s) return 0.0;
  return s * fmin(fabs(a1), fmin(fabs(a2), fabs(a3)));
}

// m_B(a1, a2, a3; M): a1 itself while |a1| <= M dx^2.
__device__ __forceinline__ double minmodB(double a1, double a2, double a3, double M, double dx) {
  return fabs(a1) <= M * dx * dx ? a1 : minmod3(a1, a2, a3);
}

// Ten moments per conserved component of the EPB elements e0 .. e0+EPB-1
// whose nodal values sit in LDS as su[EPB][NV][(N+1)^3]: the mean, the
// Legendre slope coefficients c_x, c_y, c_z (3/2 of the first moment along
// the direction, weighted means across it) and the face means -x, +x, -y,
// +y, -z, +z, written to mom[e][10][NV].  Three levels of sums over at most
// N + 1 terms each, so that no thread walks a whole face: every x-line is
// reduced to its weighted sum A, its first moment B (mirror nodes paired:
// the first-moment weights are odd about the element centre, so a line on
// which U is constant gives exactly zero) and its two end values; those over
// y to plane sums; those over z.  sh = w/2 and smu = 3/2 int(ell xi) per node
// index (LDS); lines: LDS scratch of 4 EPB NV (N+1)^2 doubles; su is
// overwritten.  The block holds slots e0 .. e0+EPB-1 of nelem; slot k is
// element eids[k] (mixed-degree lists) or k itself (eids null).  Every thread
// of the block must call it.
template <int N, int NV, int EPB, int BT>
__device__ __forceinline__ void element_moments(double *su, double *lines, const double *sh, const double *smu,
                                                double *mom, int64_t e0, int64_t nelem, const int32_t *eids = nullptr) {
  constexpr int NP = N + 1, NF = NP * NP, NPE = NP * NF;
  const int tid = threadIdx.x;
  // rows of plane sums: A, B, the end values and, where su has room, the y-pair
  // sums of A (at degree 1 the last level forms those, one pair per plane)
  constexpr int ROWS = N >= 2 ? 5 : 4;
  for (int t = tid; t < EPB * NV * NF; t += BT) {
    const int le = t / (NV * NF), r = t - le * NV * NF, v = r / NF, jk = r - v * NF;
    if (e0 + le >= nelem) continue;
    const double *line = su + (le * NV + v) * NPE + jk * NP;
    double a = 0.0, b = 0.0;
#pragma unroll
    for (int i = 0; i < NP; ++i) a += sh[i] * line[i];
#pragma unroll
    for (int i = 0; i < N - i; ++i) b += smu[N - i] * (line[N - i] - line[i]);
    double *L = lines + (le * NV + v) * 4 * NF;
    L[jk] = a;
    L[NF + jk] = b;
    L[2 * NF + jk] = line[0];
    L[3 * NF + jk] = line[N];
  }
  __syncthreads();
  // planes of constant z: weighted sums over y of A, B and the end values, and
  // the y-pair sums of A, into su as [element, component][ROWS][NP]
  for (int t = tid; t < EPB * NV * ROWS * NP; t += BT) {
    const int c = t / (ROWS * NP), r = t - c * ROWS * NP, x = r / NP, k = r - x * NP;
    if (e0 + c / NV >= nelem) continue;
    const double *X = lines + c * 4 * NF + (x < 4 ? x * NF : 0) + NP * k;
    double s = 0.0;
    if (x < 4) {
#pragma unroll
      for (int j = 0; j < NP; ++j) s += sh[j] * X[j];
    } else {
#pragma unroll
      for (int j = 0; j < N - j; ++j) s += smu[N - j] * (X[N - j] - X[j]);
    }
    su[c * NPE + x * NP + k] = s;
  }
  __syncthreads();
  for (int t = tid; t < EPB * NV * 10; t += BT) {
    const int le = t / (NV * 10), r = t - le * NV * 10, kind = r / NV, v = r - kind * NV;
    if (e0 + le >= nelem) continue;
    const int c = le * NV + v;
    const double *R = su + c * NPE, *A = lines + c * 4 * NF;
    double s = 0.0;
    if (kind == 3) {  // c_z: mirror planes paired
#pragma unroll
      for (int k = 0; k < N - k; ++k) s += smu[N - k] * (R[N - k] - R[k]);
    } else if (kind >= 8) {  // the z faces are planes
      s = R[kind == 8 ? 0 : N];
    } else if (N == 1 && kind == 2) {
#pragma unroll
      for (int k = 0; k < NP; ++k) s += sh[k] * (smu[N] * (A[N + NP * k] - A[NP * k]));
    } else {
      // mean, c_x, c_y, x faces: plane sums; y faces: the x-line sums at j = 0, N
      const double *X = kind >= 6 ? A + (kind == 6 ? 0 : N) : R + NP * (kind == 2 ? 4 : (kind < 2 ? kind : kind - 2));
      const int st = kind >= 6 ? NP : 1;
#pragma unroll
      for (int k = 0; k < NP; ++k) s += sh[k] * X[k * st];
    }
    const int64_t eid = eids ? (int64_t)eids[e0 + le] : e0 + le;
    mom[(eid * 10 + kind) * NV + v] = s;
  }
}

}  // namespace dgmi
