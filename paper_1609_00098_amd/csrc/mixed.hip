// Mortars between elements of unequal polynomial degree (the paper leaves
// p-nonconforming faces to future work).  A face between degrees Na and Nb
// carries the GLL nodes of degree Nm = max(Na, Nb):
//   - the higher-degree side's face nodes are the mortar nodes;
//   - the lower-degree side is interpolated there in (rho, W v, p [, B, Phi])
//     (the spatial four-velocity W v cannot be interpolated past the light
//     speed) and mapped to conserved variables;
//   - one numerical flux F*.n per mortar node (LLF, or HLL);
//   - the higher side's lift term is F*.n - F.n at its nodes, as on a
//     conforming face; the lower side's is P (F*.n - I F_h.n): the difference
//     between F* and the interpolant of its own nodal fluxes, integrated
//     against its face basis with the mortar's GLL rule over its lumped face
//     mass, P(i,m) = w_m l_i(x_m) / w_i (tensorised).
// The mortar kernel runs one wave per face and writes both sides' lift terms
// to a face buffer; the element kernels (the uniform kernels in their
// mixed-degree mode) read them in place of their own face computation.  Both
// terms come from the same F*, so the scheme conserves exactly.
#include "kernels.hpp"
#include "physics.hpp"

namespace dgmi {

namespace {

__device__ __forceinline__ int sel3i(int d, int a, int b, int c) { return d == 0 ? a : (d == 1 ? b : c); }

// Local node of face-tangential coordinates (ta, tb) on the face normal to d
// at normal index nrm, for an element with np nodes per direction.
__device__ __forceinline__ int face_idx(int np, int d, int nrm, int ta, int tb) {
  return sel3i(d, nrm + np * (ta + np * tb), ta + np * (nrm + np * tb), ta + np * (tb + np * nrm));
}


template <int SYS>
struct Interp {
  // (rho, u^x, u^y, u^z, p) and, for MHD, (B^x, B^y, B^z, Phi)
  static constexpr int ns = (SYS == kMHD) ? 9 : 5;
};

// Interpolation state -> conserved variables and primitives.
template <int SYS>
__device__ __forceinline__ void interp_to_state(const double *s, double g, double *u, Prim &P) {
  double iW = 1.0;
  if (SYS != kNE) iW = fast_rcp(fast_sqrt(1.0 + s[1] * s[1] + s[2] * s[2] + s[3] * s[3]));
  P.rho = s[0];
  P.v[0] = s[1] * iW;
  P.v[1] = s[2] * iW;
  P.v[2] = s[3] * iW;
  P.p = s[4];
  if (SYS == kMHD) {
    const double mag[4] = {s[5], s[6], s[7], s[8]};
    prim_to_cons<SYS>(P, mag, g, u);
  } else {
    prim_to_cons<SYS>(P, nullptr, g, u);
  }
}

// A node's conserved state and primitives (SRMHD reads all five primitive
// rows; SR only the pressure and NE none, the rest follows from U and p).
template <int SYS>
__device__ __forceinline__ void load_node(const double *U, const double *Pr, int64_t nn, int64_t q, double g,
                                          double *u, Prim &P) {
#pragma unroll
  for (int v = 0; v < SysTraits<SYS>::nv; ++v) u[v] = U[v * nn + q];
  if (SYS == kMHD) {
    P.rho = Pr[q];
    P.v[0] = Pr[nn + q];
    P.v[1] = Pr[2 * nn + q];
    P.v[2] = Pr[3 * nn + q];
    P.p = Pr[4 * nn + q];
  } else {
    P = prims_at_pressure<SYS>(u, g, SYS == kSR ? Pr[4 * nn + q] : 0.0);
  }
}

typedef __attribute__((address_space(4))) const double scalar_f64;

// Doubles between the channels of a face's buffer: a lane per line reads and
// writes with at most two lanes to a bank.
constexpr int kChan = 72;

// One direction of a tensor-product map on NCH channels of a face, a lane per
// line: out[c][o + so r] = sum_i M[o][i] in[c][i + si r] in buf (channel stride
// kChan), for r < nr lines per channel; input index i at stride sti, output o
// at stride sto (and the line number at the other one).  M (row stride 8) is the
// same for every lane and comes through the scalar cache, so that a line is
// read once, NI values for NI NO multiply-adds.  The lines of all passes are
// read before any is written.
template <int NCH, int NI, int NO, int NR, bool FIRST>
__device__ __forceinline__ void map_lines(double *buf, scalar_f64 *M) {
  // FIRST: lines run along the first tangential direction (line r at NI r in,
  // NO r out), else along the second (line r starts at r, stride NR)
  constexpr int LINES = NCH * NR, PASSES = (LINES + 63) / 64;
  double x[PASSES][NI];
#pragma unroll
  for (int p = 0; p < PASSES; ++p) {
    const int t = (int)threadIdx.x + 64 * p, c = t / NR, r = t - NR * c;
    if (t < LINES) {
#pragma unroll
      for (int i = 0; i < NI; ++i) x[p][i] = buf[c * kChan + (FIRST ? i + NI * r : r + NR * i)];
    }
  }
  __syncthreads();
#pragma unroll
  for (int o = 0; o < NO; ++o) {
#pragma unroll
    for (int p = 0; p < PASSES; ++p) {
      const int t = (int)threadIdx.x + 64 * p, c = t / NR, r = t - NR * c;
      if (t < LINES) {
        double s = 0.0;
#pragma unroll
        for (int i = 0; i < NI; ++i) s += M[o * 8 + i] * x[p][i];
        buf[c * kChan + (FIRST ? o + NO * r : r + NR * o)] = s;
      }
    }
  }
  __syncthreads();
}

// The same map with a lane per output node, o and r from its index as the output
// lies in buf; the matrix from LDS.  Results stay in the lane's registers.
template <int NCH, int NI, int NO, int NR, bool FIRST>
__device__ __forceinline__ void map_nodes(const double *buf, const double *sM, double (&out)[NCH]) {
#pragma unroll
  for (int c = 0; c < NCH; ++c) out[c] = 0.0;
  const int l = threadIdx.x;
  if (l < NO * NR) {
    const int o = FIRST ? l % NO : l / NR, r = FIRST ? l / NO : l % NR;
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      const double w = sM[o * 8 + i];
#pragma unroll
      for (int c = 0; c < NCH; ++c) out[c] += w * buf[c * kChan + (FIRST ? i + NI * r : r + NR * i)];
    }
  }
}

// A lane's channels to its place in buf, every lane's reads done before.
template <int NCH>
__device__ __forceinline__ void put_channels(double *buf, const double (&v)[NCH], int n) {
  __syncthreads();
  if ((int)threadIdx.x < n) {
#pragma unroll
    for (int c = 0; c < NCH; ++c) buf[c * kChan + threadIdx.x] = v[c];
  }
  __syncthreads();
}

}  // namespace


// The work of one face (wave) between degrees NLO < NMX, every loop bound a
// compile-time constant.
template <int SYS, int FLUX, bool LINES, int NLO, int NMX>
__device__ __forceinline__ void mortar_face(const MortarArgs &A, int64_t qhi, int64_t qlo, int64_t ohi, int64_t olo,
                                            int d, int side_hi, double *buf, double *sI, double *sP) {
  constexpr int NV = SysTraits<SYS>::nv, NS = Interp<SYS>::ns;
  // channels interpolated to the mortar: the state, then the lower side's
  // nodal normal fluxes
  constexpr int NC = NS + NV;
  constexpr int nm = NMX + 1, nl = NLO + 1;
  // one buffer [channel][kChan] serves every phase
  const int l = threadIdx.x;
  const int side_lo = 1 - side_hi;
  const double sgn_hi = side_hi ? 1.0 : -1.0, sgn_lo = -sgn_hi;
  const int64_t nn = A.nnodes;
  constexpr int tab = (NLO * 8 + NMX) * 64;
  scalar_f64 *I = (scalar_f64 *)(A.Itab + tab), *Pm = (scalar_f64 *)(A.Ptab + tab);  // I[ma][ia], P[a][ma]
  if constexpr (!LINES) {
    sI[l] = A.Itab[tab + l];
    sP[l] = A.Ptab[tab + l];
  }

  // the higher side's node of this lane's mortar position, loaded up front so
  // that its latency overlaps the lower side's loads
  double uh[NV], Fh[NV], ah = 0.0, lmh = 0.0, lph = 0.0;
#pragma unroll
  for (int v = 0; v < NV; ++v) {
    uh[v] = 0.0;
    Fh[v] = 0.0;
  }
  if (l < nm * nm) {
    Prim Ph;
    load_node<SYS>(A.U, A.P, nn, qhi + face_idx(nm, d, side_hi ? NMX : 0, l % nm, l / nm), A.gamma, uh, Ph);
    flux_normal<SYS>(d, uh, Ph, Fh);
    if constexpr (FLUX == kHLL) wave_bounds<SYS>(d, uh, Ph, A.gamma, A.gratio, lmh, lph);
    else ah = max_speed<SYS>(d, uh, Ph, A.gamma, A.gratio);
  }

  // L: lower side's face nodes
  if (l < nl * nl) {
    const int ka = l % nl, kb = l / nl;
    const int64_t q = qlo + face_idx(nl, d, side_lo ? NLO : 0, ka, kb);
    double u[NV];
    Prim P;
    load_node<SYS>(A.U, A.P, nn, q, A.gamma, u, P);
    double W = 1.0;
    if (SYS != kNE) W = fast_rcp(fast_sqrt(1.0 - (P.v[0] * P.v[0] + P.v[1] * P.v[1] + P.v[2] * P.v[2])));
    buf[l] = P.rho;
    buf[kChan + l] = P.v[0] * W;
    buf[2 * kChan + l] = P.v[1] * W;
    buf[3 * kChan + l] = P.v[2] * W;
    buf[4 * kChan + l] = P.p;
    if (SYS == kMHD) {
#pragma unroll
      for (int c = 0; c < 4; ++c) buf[(5 + c) * kChan + l] = u[5 + c];
    }
    double F[NV];
    flux_normal<SYS>(d, u, P, F);
#pragma unroll
    for (int v = 0; v < NV; ++v) buf[(NS + v) * kChan + l] = F[v];
  }
  __syncthreads();

  // I1, I2: the channels at the mortar nodes, one tangential direction at a time
  double s[NC];
  if constexpr (LINES) {
    map_lines<NC, nl, nm, nl, true>(buf, I);
    map_lines<NC, nl, nm, nm, false>(buf, I);
#pragma unroll
    for (int c = 0; c < NC; ++c) s[c] = buf[c * kChan + l];
  } else {
    map_nodes<NC, nl, nm, nl, true>(buf, sI, s);
    put_channels<NC>(buf, s, nm * nl);
    map_nodes<NC, nl, nm, nm, false>(buf, sI, s);
  }

  // flux at the mortar node
  double jr[NV];
  if (l < nm * nm) {
    double ul[NV], Fl[NV];
    Prim Pl;
    interp_to_state<SYS>(s, A.gamma, ul, Pl);
    flux_normal<SYS>(d, ul, Pl, Fl);
    const double hs = 0.5 * sgn_hi;
    double *out_hi = A.facebuf + ohi + l;
    if constexpr (FLUX == kHLL) {
      // the higher side as the interior: F*.n - F_h.n = c [sg (F_l - F_h) -
      // s+ (U_l - U_h)], c = -s- / (s+ - s-), with the largest and smallest
      // speeds along its outward normal of either side, clipped by zero
      double lml, lpl;
      wave_bounds<SYS>(d, ul, Pl, A.gamma, A.gratio, lml, lpl);
      const double sp = fmax(0.0, side_hi ? fmax(lph, lpl) : -fmin(lmh, lml));
      const double sm = fmin(0.0, side_hi ? fmin(lmh, lml) : -fmax(lph, lpl));
      const double cf = -sm * fast_rcp(sp - sm);
#pragma unroll
      for (int v = 0; v < NV; ++v) {
        double oh;
        if (SYS == kMHD && (v == 8 || v == 5 + d))  // bounds -1, +1: the LLF form with alpha = 1
          oh = hs * (Fl[v] - Fh[v]) - 0.5 * (ul[v] - uh[v]);
        else
          oh = cf * (sgn_hi * (Fl[v] - Fh[v]) - sp * (ul[v] - uh[v]));
        out_hi[v * nm * nm] = oh;
        // F*.n_lo = -(F*.n_hi), less the interpolant of the lower side's own
        // normal fluxes (s[NS + v] is along +e_d)
        jr[v] = -(oh + sgn_hi * Fh[v]) - sgn_lo * s[NS + v];
      }
    } else {
      const double alpha = fmax(ah, max_speed<SYS>(d, ul, Pl, A.gamma, A.gratio));
#pragma unroll
      for (int v = 0; v < NV; ++v) {
        double al = alpha;
        if (SYS == kMHD && (v == 8 || v == 5 + d)) al = 1.0;
        // F*.n_hi with the higher side interior
        const double diss = 0.5 * al * (ul[v] - uh[v]);
        out_hi[v * nm * nm] = hs * (Fl[v] - Fh[v]) - diss;
        // F*.n_lo = -F*.n_hi, less the interpolant of the lower side's own
        // normal fluxes (s[NS + v] is along +e_d)
        jr[v] = diss - hs * (Fh[v] + Fl[v]) - sgn_lo * s[NS + v];
      }
    }
  }
  put_channels<NV>(buf, jr, nm * nm);

  // P1, P2: lower side's lift term P (F*.n_lo - I F_h.n_lo) at its nodes
  double g[NV];
  if constexpr (LINES) {
    map_lines<NV, nm, nl, nm, true>(buf, Pm);
    map_lines<NV, nm, nl, nl, false>(buf, Pm);
#pragma unroll
    for (int v = 0; v < NV; ++v) g[v] = buf[v * kChan + l];
  } else {
    map_nodes<NV, nm, nl, nm, true>(buf, sP, g);
    put_channels<NV>(buf, g, nl * nm);
    map_nodes<NV, nm, nl, nl, false>(buf, sP, g);
  }
  if (l < nl * nl) {
    double *out_lo = A.facebuf + olo + l;
#pragma unroll
    for (int v = 0; v < NV; ++v) out_lo[v * nl * nl] = g[v];
  }
}

// One wave per non-conforming face, in separable passes (tensor-product
// interpolation and projection one direction at a time):
//   L  lanes k < (Nlo+1)^2 load the lower side's face nodes: interpolation
//      state and normal fluxes F_h;
//   I1, I2 interpolate the state and F_h along each tangential direction; each
//      mortar lane (which loaded its higher-side node at the start) forms
//      F*.n, writes the higher side's lift term F*.n - F.n and keeps
//      F*.n_lo - I F_h.n_lo;
//   P1, P2 project that difference onto the lower side's nodes along each
//      direction.
// LINES: the maps run a lane per line with the matrix on the scalar side
// (map_lines), about 80 LDS reads a face and 71 VGPRs.  Else a lane per output
// node reads every input value once per output: 230 LDS reads and 140 VGPRs, which
// bound a pass over many faces, but a shorter chain, which is what counts where
// every face runs at once (few_faces below).
// Workgroups are mapped XCD-major (hardware block b runs on XCD b % 8 and
// walks its own contiguous range of the face list), so that faces of nearby
// elements, which share cache lines of the node blocks, share an L2.  The
// degree pair selects a body compiled for it (every face of a wave has the
// same pair, so the branch is uniform).
template <int SYS, int FLUX, bool LINES>
__global__ void __launch_bounds__(64) mortar_kernel(const MortarArgs A) {
  constexpr int NC = Interp<SYS>::ns + SysTraits<SYS>::nv;
  __shared__ double buf[NC * kChan];
  __shared__ double sI[LINES ? 1 : 64], sP[LINES ? 1 : 64];
  const int64_t per = (A.nfaces + 7) >> 3;
  const int64_t t = (int64_t)(blockIdx.x & 7) * per + (int64_t)(blockIdx.x >> 3);
  if (t >= A.nfaces) return;
  const int64_t *fd = A.fdesc + 5 * t;
  const int64_t qhi = fd[0], qlo = fd[1], ohi = fd[2], olo = fd[3];
  const int info = (int)fd[4];
  const int d = info & 3, side_hi = (info >> 2) & 1, Nm = (info >> 3) & 7, Nlo = (info >> 6) & 7;
#define DGMI_MORTAR_CASE(LO, HI) \
  case LO * 8 + HI: mortar_face<SYS, FLUX, LINES, LO, HI>(A, qhi, qlo, ohi, olo, d, side_hi, buf, sI, sP); break;
  switch (Nlo * 8 + Nm) {
    DGMI_MORTAR_CASE(1, 2) DGMI_MORTAR_CASE(1, 3) DGMI_MORTAR_CASE(1, 4) DGMI_MORTAR_CASE(1, 5)
    DGMI_MORTAR_CASE(1, 6) DGMI_MORTAR_CASE(1, 7) DGMI_MORTAR_CASE(2, 3) DGMI_MORTAR_CASE(2, 4)
    DGMI_MORTAR_CASE(2, 5) DGMI_MORTAR_CASE(2, 6) DGMI_MORTAR_CASE(2, 7) DGMI_MORTAR_CASE(3, 4)
    DGMI_MORTAR_CASE(3, 5) DGMI_MORTAR_CASE(3, 6) DGMI_MORTAR_CASE(3, 7) DGMI_MORTAR_CASE(4, 5)
    DGMI_MORTAR_CASE(4, 6) DGMI_MORTAR_CASE(4, 7) DGMI_MORTAR_CASE(5, 6) DGMI_MORTAR_CASE(5, 7)
    DGMI_MORTAR_CASE(6, 7)
    default: break;  // the face list holds only pairs 1 <= Nlo < Nm <= 7
  }
#undef DGMI_MORTAR_CASE
}

// Node coordinates of a mixed-degree mesh: one workgroup per element.
__global__ void __launch_bounds__(256) mixed_coords_kernel(const int32_t *deg, const int64_t *off, const double *xtab,
                                                           int nx, int ny, int64_t nelem, double lo0, double lo1,
                                                           double lo2, double dx0, double dx1, double dx2,
                                                           double *xyz, int64_t nn) {
  const int64_t e = blockIdx.x;
  if (e >= nelem) return;
  const int N = deg[e], np = N + 1, npe = np * np * np;
  const int64_t c0 = e % nx, c1 = (e / nx) % ny, c2 = e / ((int64_t)nx * ny);
  const double *x = xtab + 8 * N;
  for (int a = threadIdx.x; a < npe; a += blockDim.x) {
    const int i = a % np, j = (a / np) % np, k = a / (np * np);
    const int64_t qn = off[e] + a;
    xyz[qn] = lo0 + c0 * dx0 + 0.5 * (1.0 + x[i]) * dx0;
    xyz[nn + qn] = lo1 + c1 * dx1 + 0.5 * (1.0 + x[j]) * dx1;
    xyz[2 * nn + qn] = lo2 + c2 * dx2 + 0.5 * (1.0 + x[k]) * dx2;
  }
}

__global__ void set_scalar_kernel(double *p, double v) {
  if (threadIdx.x == 0 && blockIdx.x == 0) *p = v;
}

__global__ void __launch_bounds__(256) fill_kernel(double *p, int64_t n, double v) {
  for (int64_t i = blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) p[i] = v;
}

// ------------------------------------------------------------ launchers
// Whether every face runs at once with a lane per node: twelve waves per CU for
// NE and SR (140 VGPRs), eight for SRMHD (174).  Then the chain of one face counts,
// which is shorter than by line, else the work.  Us a pass, by node / by line, of
// degrees 2 to 7: NE 168 faces 4.6 / 6.3, 1,304 7.0 / 8.2, 3,336 13.2 / 13.3,
// 10,272 23.3 / 20.4; SR 5.0 / 6.3, 7.6 / 9.2, 14.1 / 14.0, 25.4 / 23.5; SRMHD 5.7 /
// 9.2, 11.8 / 13.4, 1,808 faces 13.4 / 15.0, 2,504 17.3 / 16.3, 10,272 42.2 / 38.7.
static bool few_faces(int sys, int64_t n) { return n <= 256 * (sys == kMHD ? 8 : 12); }

template <int SYS>
static void mortar_sys(bool hll, const MortarArgs &a, hipStream_t s) {
  const dim3 grid((unsigned)(((a.nfaces + 7) >> 3) << 3)), block(64);
  if (few_faces(SYS, a.nfaces)) {
    if (hll) hipLaunchKernelGGL((mortar_kernel<SYS, kHLL, false>), grid, block, 0, s, a);
    else hipLaunchKernelGGL((mortar_kernel<SYS, kLLF, false>), grid, block, 0, s, a);
  } else {
    if (hll) hipLaunchKernelGGL((mortar_kernel<SYS, kHLL, true>), grid, block, 0, s, a);
    else hipLaunchKernelGGL((mortar_kernel<SYS, kLLF, true>), grid, block, 0, s, a);
  }
}

hipError_t launch_mortar(int sys, int flux, const MortarArgs &a, hipStream_t s) {
  if (a.nfaces <= 0) return hipSuccess;
  if (a.nfaces > ((int64_t)1 << 31) - 1) return hipErrorInvalidValue;
  if (flux != kLLF && flux != kHLL) return hipErrorInvalidValue;
  switch (sys) {
    case kNE: mortar_sys<kNE>(flux == kHLL, a, s); break;
    case kSR: mortar_sys<kSR>(flux == kHLL, a, s); break;
    case kMHD: mortar_sys<kMHD>(flux == kHLL, a, s); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_mixed_coords(const int32_t *deg, const int64_t *off, const double *xtab, int nx, int ny,
                               int64_t nelem, const double *lo, const double *dx, double *xyz, int64_t nn,
                               hipStream_t s) {
  if (nelem <= 0) return hipSuccess;
  hipLaunchKernelGGL(mixed_coords_kernel, dim3((unsigned)nelem), dim3(256), 0, s, deg, off, xtab, nx, ny, nelem,
                     lo[0], lo[1], lo[2], dx[0], dx[1], dx[2], xyz, nn);
  return hipGetLastError();
}

hipError_t launch_fill(double *p, int64_t n, double v, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  const int64_t blocks = (n + 255) / 256;
  hipLaunchKernelGGL(fill_kernel, dim3((unsigned)(blocks < 8192 ? blocks : 8192)), dim3(256), 0, s, p, n, v);
  return hipGetLastError();
}

hipError_t launch_set_scalar(double *p, double v, hipStream_t s) {
  hipLaunchKernelGGL(set_scalar_kernel, dim3(1), dim3(64), 0, s, p, v);
  return hipGetLastError();
}

}  // namespace dgmi
