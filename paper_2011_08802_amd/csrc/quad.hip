// Quadrature and assembly kernels (Sec. 3.3-3.4): residual R = dPi/dU and
// tangent K = d^2 Pi / dU^2 of the discrete potential on Q1 hexahedra with
// 2x2x2 Gauss points, assembled without atomics:
//   1. residual_element, residual_nodes: the elements' residual parts and their
//      node sums;
//   2. qp_kernel: one thread per (Gauss point, element) evaluates the local
//      Hessian of the density and stores it (SoA, coalesced); qp_mf_kernel: the
//      same into the matrix-free layout;
//   3. element_matrix: element blocks for the 36 node pairs a <= b, with the
//      Gauss-point Hessians shared through LDS;
//   4. jacobian_gather: a workgroup per (64 node rows, stored stencil block) sums
//      the <= 8 element blocks of the elements containing both nodes and
//      writes the 9x9 block into the tiled half-stencil layout.
// Summation order is fixed, so results are bitwise reproducible.
#include "pair.h"

namespace mvpf {

// Gauss abscissae on [0,1]: (1 -+ 1/sqrt(3)) / 2
constexpr double GQ0 = 0.21132486540518711775;
constexpr double GQ1 = 0.78867513459481288225;

struct Shape {
  double N;
  double dN[3];  // reference-cube derivatives (divide by h for physical)
};

__device__ __forceinline__ Shape shape(int g, int a) {
  const double x[3] = {(g & 1) ? GQ1 : GQ0, (g & 2) ? GQ1 : GQ0, (g & 4) ? GQ1 : GQ0};
  double f[3], df[3];
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    const bool bit = (a >> d) & 1;
    f[d] = bit ? x[d] : 1.0 - x[d];
    df[d] = bit ? 1.0 : -1.0;
  }
  Shape s;
  s.N = f[0] * f[1] * f[2];
  s.dN[0] = df[0] * f[1] * f[2];
  s.dN[1] = f[0] * df[1] * f[2];
  s.dN[2] = f[0] * f[1] * df[2];
  return s;
}

// reference Laplacian 1/8 sum_g dN_a(g) . dN_b(g)  (element matrix = h * this)
__device__ __forceinline__ double lap_ref(int a, int b) {
  double s = 0.0;
#pragma unroll
  for (int g = 0; g < 8; ++g) {
    const Shape sa = shape(g, a), sb = shape(g, b);
    s += sa.dN[0] * sb.dN[0] + sa.dN[1] * sb.dN[1] + sa.dN[2] * sb.dN[2];
  }
  return 0.125 * s;
}

// Packed Hessians of a slab's Gauss points, one thread per (point, element).
template <int PD, int MIX>
__device__ __forceinline__ void qp_body(const Grid& g, const Chunk& ck, const double* __restrict__ state,
                                        const DevCard* __restrict__ cd, double* __restrict__ qp, int bid) {
  const int64_t tid = (int64_t)bid * 128 + threadIdx.x;
  const int gp = (int)(tid / ck.NEcpad);
  const int el = (int)(tid - (int64_t)gp * ck.NEcpad);
  if (gp >= 8 || el >= ck.NEc) return;
  const int64_t e = ck.e0 + el;
  const int ex = (int)(e % g.nx), ey = (int)((e / g.nx) % g.ny), ez = (int)(e / ((int64_t)g.nx * g.ny));
  const double ih = 1.0 / g.h;
  double F[9] = {1, 0, 0, 0, 1, 0, 0, 0, 1};
  double eh[NV];
#pragma unroll
  for (int k = 0; k < NV; ++k) eh[k] = 0.0;
#pragma unroll
  for (int a = 0; a < 8; ++a) {
    const int node = (ex + (a & 1)) + g.nnx * ((ey + ((a >> 1) & 1)) + g.nny * (ez + ((a >> 2) & 1)));
    const Shape s = shape(gp, a);
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      const double u = state[(int64_t)i * g.Npad + node];
#pragma unroll
      for (int j = 0; j < 3; ++j) F[3 * i + j] += u * s.dN[j] * ih;
    }
#pragma unroll
    for (int k = 0; k < NV; ++k) eh[k] += s.N * state[(int64_t)(3 + k) * g.Npad + node];
  }
  const uint32_t off = (uint32_t)gp * (uint32_t)ck.NEcpad + (uint32_t)el;  // < 8 NEcpad
  local_hessian<PD, MIX>(F, eh, *cd, PackedOut{F, qp, (int64_t)8 * ck.NEcpad, off});
}
template <int PD, int MIX>
__global__ void __launch_bounds__(128) qp_kernel(Grid g, Chunk ck, const double* __restrict__ state,
                                                 const DevCard* __restrict__ cd, double* __restrict__ qp) {
  qp_body<PD, MIX>(g, ck, state, cd, qp, blockIdx.x);
}

// Kernel K::run<order, mixing>(args...) of a card: pade 11, 22 or 33, mixing
// MVPF_MIX_LINEAR or MVPF_MIX_LOG (validated at creation).
template <class K, class... A>
void run_card(int pade, int mixing, A... a) {
  if (mixing == MVPF_MIX_LOG) {
    switch (pade) {
      case 11: K::template run<11, 1>(a...); break;
      case 33: K::template run<33, 1>(a...); break;
      default: K::template run<22, 1>(a...); break;
    }
    return;
  }
  switch (pade) {
    case 11: K::template run<11, 0>(a...); break;
    case 33: K::template run<33, 0>(a...); break;
    default: K::template run<22, 0>(a...); break;
  }
}
struct QpRun {
  template <int PD, int MIX>
  static void run(const Grid& g, const Chunk& ck, const double* state, const DevCard* cd, double* qp, hipStream_t s) {
    qp_kernel<PD, MIX><<<(int)(((int64_t)8 * ck.NEcpad + 127) / 128), 128, 0, s>>>(g, ck, state, cd, qp);
  }
};
void launch_qp(const Grid& g, const Chunk& ck, const double* state, const DevCard* cd, int pade, int mixing,
               double* qp, hipStream_t s) {
  run_card<QpRun>(pade, mixing, g, ck, state, cd, qp, s);
}

// ---- residual ---------------------------------------------------------------
// One pass over the elements: a wavefront holds 8 elements x 8 points (lane = 8 *
// element + point); lane j loads the state of corner j, the point's F, eta,
// grad eta and eta_n come from three pair interpolations, and the density's
// gradient (and the gradient energy's) goes back to the corners through the
// transposed stages.  The corner values are merged along x in the workgroup and
// a node sum of at most 4 merged rows follows.  Bound: vector issue (2500
// instructions per point, 1500 of them FP64) at two wavefronts per SIMD; 64^3:
// 0.19 ms and 0.03 ms for the node sums, against 0.30 ms for gradients stored
// per point and 0.35 ms for a node gather that read each of them eight times.
template <int PD, int MIX>
__device__ __forceinline__ void residual_element_body(const Grid& g, const Chunk& ck, const double* __restrict__ state,
                                                      const DevCard* __restrict__ cd, double* __restrict__ E, int wg,
                                                      int nb) {
  __shared__ double eo[8 * NDOF * (SLAB_EPW + 1)];
  const int xcd = wg & 7;  // one contiguous range of elements per XCD
  const int bid = xcd * (nb >> 3) + min(xcd, nb & 7) + (wg >> 3);
  const int gp = threadIdx.x & 7, jw = threadIdx.x >> 3;
  const int el = bid * SLAB_EPW + jw;
  const bool b0 = gp & 1, b1 = (gp >> 1) & 1, b2 = (gp >> 2) & 1;
  constexpr int NS = 3 + 2 * NV;
  double F[9], eh[NV], ehn[NV], ge[3 * NV];
  {
    double x[NS];
#pragma unroll
    for (int c = 0; c < NS; ++c) x[c] = 0.0;
    if (el < ck.NEc) {
      const int64_t e = ck.e0 + el;
      const int ex = (int)(e % g.nx), ey = (int)((e / g.nx) % g.ny), ez = (int)(e / ((int64_t)g.nx * g.ny));
      const int node = (ex + b0) + g.nnx * ((ey + b1) + g.nny * (ez + b2));
#pragma unroll
      for (int c = 0; c < NS; ++c) x[c] = state[(int64_t)c * g.Npad + node];
    }
    double s1[NS], d1[NDOF], i2[NS + NDOF], s2[NS + NDOF], d2[NDOF], i3[NS + 2 * NDOF], s3[NS + 2 * NDOF], d3[NDOF];
    interp_pair<1>(x, MGQ0, b0 ? -1.0 : 1.0, s1, d1);
#pragma unroll
    for (int c = 0; c < NS; ++c) i2[c] = s1[c];
#pragma unroll
    for (int c = 0; c < NDOF; ++c) i2[NS + c] = d1[c];
    interp_pair<2>(i2, MGQ0, b1 ? -1.0 : 1.0, s2, d2);
#pragma unroll
    for (int c = 0; c < NS + NDOF; ++c) i3[c] = s2[c];
#pragma unroll
    for (int c = 0; c < NDOF; ++c) i3[NS + NDOF + c] = d2[c];
    interp_pair<4>(i3, MGQ0, b2 ? -1.0 : 1.0, s3, d3);
    const double ih = 1.0 / g.h;
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      F[3 * i] = s3[NS + i] * ih + (i == 0 ? 1.0 : 0.0);
      F[3 * i + 1] = s3[NS + NDOF + i] * ih + (i == 1 ? 1.0 : 0.0);
      F[3 * i + 2] = d3[i] * ih + (i == 2 ? 1.0 : 0.0);
    }
#pragma unroll
    for (int k = 0; k < NV; ++k) {
      eh[k] = s3[3 + k], ehn[k] = s3[3 + NV + k];
      ge[3 * k] = s3[NS + 3 + k], ge[3 * k + 1] = s3[NS + NDOF + 3 + k], ge[3 * k + 2] = d3[3 + k];
    }
  }
  double gr[NQ];
  local_gradient<PD, MIX>(F, eh, ehn, *cd, gr);
  // coefficients of the values and of the x, y, z reference derivatives, each
  // derivative's with the transposed stage's sign of its direction
  const double h = g.h, cu = 0.125 * h * h, cg = 0.125 * h;
  const double sx = b0 ? 1.0 : -1.0, sy = b1 ? 1.0 : -1.0, sz = b2 ? 1.0 : -1.0;
  double a3[3 * NDOF], bz[3 * NDOF], r3[3 * NDOF];
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    a3[i] = 0.0, a3[NDOF + i] = sx * cu * gr[3 * i], a3[2 * NDOF + i] = sy * cu * gr[3 * i + 1];
    bz[i] = sz * cu * gr[3 * i + 2];
  }
#pragma unroll
  for (int m = 0; m < NV; ++m) {
    double z[3] = {0.0, 0.0, 0.0};
#pragma unroll
    for (int m2 = 0; m2 < NV; ++m2)
#pragma unroll
      for (int j = 0; j < 3; ++j) z[j] += cd->Mg[m][m2] * ge[3 * m2 + j];
    a3[3 + m] = h * cu * gr[9 + m], a3[NDOF + 3 + m] = sx * cg * z[0], a3[2 * NDOF + 3 + m] = sy * cg * z[1];
    bz[3 + m] = sz * cg * z[2];
  }
#pragma unroll
  for (int c = NDOF; c < 3 * NDOF; ++c) bz[c] = 0.0;
  interp_pair_t<4>(a3, bz, MGQ1, MGQ0, r3);
  double a2[2 * NDOF], by[2 * NDOF], r2[2 * NDOF], a1[NDOF], bx[NDOF], out[NDOF];
#pragma unroll
  for (int c = 0; c < 2 * NDOF; ++c) a2[c] = r3[c], by[c] = c < NDOF ? r3[2 * NDOF + c] : 0.0;
  interp_pair_t<2>(a2, by, MGQ1, MGQ0, r2);
#pragma unroll
  for (int c = 0; c < NDOF; ++c) a1[c] = r2[c], bx[c] = r2[NDOF + c];
  interp_pair_t<1>(a1, bx, MGQ1, MGQ0, out);
  store_corners<double, NDOF>(eo, out, gp, jw, SLAB_EPW, bid, g.nx, ck.NEc, E, ck.NEcpad, slab_nw(ck), ck.NEc / g.nx);
}
__device__ __forceinline__ void residual_nodes_body(const Grid& g, const Chunk& ck, const double* __restrict__ E,
                                                    double* __restrict__ R, int bid) {
  // one value per thread (8^3: 19 -> 4.6 us against a node per thread)
  const int c = bid % NDOF, n = ck.n0 + bid / NDOF * 256 + threadIdx.x;
  if (n >= ck.n1) return;
  const int i = n % g.nnx, j = (n / g.nnx) % g.nny, k = n / (g.nnx * g.nny) - (int)(ck.e0 / ((int64_t)g.nx * g.ny));
  R[(int64_t)c * g.Npad + n] = n < g.N ? slab_node_sum(g, ck, E, NDOF, c, i, j, k) : 0.0;
}
template <int PD, int MIX>
__global__ void __launch_bounds__(256) residual_element_kernel(Grid g, Chunk ck, const double* __restrict__ state,
                                                               const DevCard* __restrict__ cd, double* __restrict__ E) {
  residual_element_body<PD, MIX>(g, ck, state, cd, E, blockIdx.x, gridDim.x);
}
__global__ void __launch_bounds__(256) residual_nodes_kernel(Grid g, Chunk ck, const double* __restrict__ E,
                                                             double* __restrict__ R) {
  residual_nodes_body(g, ck, E, R, blockIdx.x);
}
struct ResidualRun {
  template <int PD, int MIX>
  static void run(const Grid& g, const Chunk& ck, const double* state, const DevCard* cd, double* E, hipStream_t s) {
    residual_element_kernel<PD, MIX><<<ck.NEcpad / SLAB_EPW, 256, 0, s>>>(g, ck, state, cd, E);
  }
};
void launch_residual(const Grid& g, const Chunk& ck, const double* state, const DevCard* cd, int pade, int mixing,
                     double* E, double* R, hipStream_t s) {
  run_card<ResidualRun>(pade, mixing, g, ck, state, cd, E, s);
  residual_nodes_kernel<<<(ck.n1 - ck.n0 + 255) / 256 * NDOF, 256, 0, s>>>(g, ck, E, R);
}

// Gauss-point tangents of a matrix-free level, straight into the matrix-free
// layout (no pass over a scratch form).  A wavefront holds 8 elements x 8 points
// (lane = 8 * element + point): lane j loads the 9 unknowns of corner j of its
// element, and the point's F and eta come from three pair interpolations,
// instead of 72 loads per point.  Bound: vector issue at one wavefront per SIMD
// (7800 instructions per point, 5600 of them FP64, 1200 moves from and to the
// accumulation registers); 64^3: 0.69 ms, 1.15 KB written per point (3.5 TB/s),
// against 2.43 ms for the Hessian in (F, eta) and 1.10 ms for the pass that
// repacked it.
struct MfOut {
  const double* F;
  double2* D64;   // the wavefront's group of 8 elements
  float4* D32;    // or null
  uint32_t slot;  // 8 * point + element
  double pend[4];
  double col[6];
  __device__ __forceinline__ void vec2(int k, double a, double b) const {
    (D64 + (int64_t)(k / 2) * 64)[slot] = make_double2(a, b);
  }
  __device__ __forceinline__ void vec4(int k, double a, double b, double c, double d) const {
    vec2(k, a, b);
    vec2(k + 2, c, d);
    if (D32) (D32 + (int64_t)(k / 4) * 64)[slot] = make_float4((float)a, (float)b, (float)c, (float)d);
  }
  __device__ __forceinline__ void strain(const double S[6], const double Dee[21]) const {
    auto at = [&](int k) {
      return k < MF_S ? F[k] - (k % 4 == 0 ? 1.0 : 0.0) : k < MF_EE ? S[k - MF_S] : Dee[k - MF_EE];
    };
#pragma unroll
    for (int k = 0; k < MF_EK; k += 4) vec4(k, at(k), at(k + 1), at(k + 2), at(k + 3));
  }
  __device__ __forceinline__ void eps_eta(int k, const double d[6]) {
    const int at = MF_EK + 6 * k;
    if (k % 2 == 0) {
#pragma unroll
      for (int i = 0; i < 6; ++i) col[i] = d[i];
    } else {
      vec4(at - 6, col[0], col[1], col[2], col[3]);
      vec4(at - 2, col[4], col[5], d[0], d[1]);
      vec4(at + 2, d[2], d[3], d[4], d[5]);
    }
  }
  __device__ __forceinline__ void eta_eta(int k, int l, double v) {
    const int i = k * (k + 1) / 2 + l;
    pend[i % 4] = v;
    if (k == NV - 1 && l == NV - 1) {
#pragma unroll
      for (int j = 0; j < 4; ++j)
        if (j > i % 4) pend[j] = 0.0;
    }
    if (i % 4 == 3 || (k == NV - 1 && l == NV - 1))
      vec4(MF_KK + i / 4 * 4, pend[0], pend[1], pend[2], pend[3]);
  }
};
template <int PD, int MIX>
__device__ __forceinline__ void qp_mf_body(const Grid& g, const Chunk& ck, const double* __restrict__ state,
                                           const DevCard* __restrict__ cd, double* __restrict__ D64,
                                           float* __restrict__ D32, int bid) {
  static_assert(NV == 6 || !MF_AVAILABLE, "entry counts of the matrix-free layout");
  const int lane = threadIdx.x & 63, gp = lane & 7;
  // group of 8 elements, uniform over the wavefront
  const int64_t eg = ck.e0 / 8 + __builtin_amdgcn_readfirstlane(bid * 2 + (threadIdx.x >> 6));
  const int64_t e = eg * 8 + (lane >> 3), el = e - ck.e0;
  const bool active = el >= 0 && el < ck.NEc;
  const bool b0 = gp & 1, b1 = (gp >> 1) & 1, b2 = (gp >> 2) & 1;
  double F[9], eh[NV];
  {
    double x[NDOF];
#pragma unroll
    for (int c = 0; c < NDOF; ++c) x[c] = 0.0;
    if (active) {
      const int ex = (int)(e % g.nx), ey = (int)((e / g.nx) % g.ny), ez = (int)(e / ((int64_t)g.nx * g.ny));
      const int node = (ex + b0) + g.nnx * ((ey + b1) + g.nny * (ez + b2));
#pragma unroll
      for (int c = 0; c < NDOF; ++c) x[c] = state[(int64_t)c * g.Npad + node];
    }
    const double ih = 1.0 / g.h;
    constexpr int n = NDOF;
    double s1[n], d1[3], i2[n + 3], s2[n + 3], d2[3], i3[n + 6], s3[n + 6], d3[3];
    interp_pair<1>(x, MGQ0, b0 ? -ih : ih, s1, d1);
#pragma unroll
    for (int c = 0; c < n; ++c) i2[c] = s1[c];
#pragma unroll
    for (int c = 0; c < 3; ++c) i2[n + c] = d1[c];
    interp_pair<2>(i2, MGQ0, b1 ? -ih : ih, s2, d2);
#pragma unroll
    for (int c = 0; c < n + 3; ++c) i3[c] = s2[c];
#pragma unroll
    for (int c = 0; c < 3; ++c) i3[n + 3 + c] = d2[c];
    interp_pair<4>(i3, MGQ0, b2 ? -ih : ih, s3, d3);
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      F[3 * i] = s3[n + i] + (i == 0 ? 1.0 : 0.0);
      F[3 * i + 1] = s3[n + 3 + i] + (i == 1 ? 1.0 : 0.0);
      F[3 * i + 2] = d3[i] + (i == 2 ? 1.0 : 0.0);
    }
#pragma unroll
    for (int k = 0; k < NV; ++k) eh[k] = s3[3 + k];
  }
  if (!active) return;  // no lane exchanges from here on
  MfOut out{F,
            reinterpret_cast<double2*>(D64) + eg * (MF_NK / 2) * 64,
            D32 ? reinterpret_cast<float4*>(D32) + eg * (MF_NK / 4) * 64 : nullptr,
            (uint32_t)(8 * gp + (lane >> 3)),
            {0.0, 0.0, 0.0, 0.0},
            {0.0, 0.0, 0.0, 0.0, 0.0, 0.0}};
  local_hessian<PD, MIX>(F, eh, *cd, out);
}
template <int PD, int MIX>
__global__ void __launch_bounds__(128) qp_mf_kernel(Grid g, Chunk ck, const double* __restrict__ state,
                                                    const DevCard* __restrict__ cd, double* __restrict__ D64,
                                                    float* __restrict__ D32) {
  qp_mf_body<PD, MIX>(g, ck, state, cd, D64, D32, blockIdx.x);
}
// groups of 8 elements touching the slab, two wavefronts per workgroup
int qp_mf_blocks(const Chunk& ck) { return (int)(((ck.e0 + ck.NEc + 7) / 8 - ck.e0 / 8 + 1) / 2); }
struct QpMfRun {
  template <int PD, int MIX>
  static void run(const Grid& g, const Chunk& ck, const double* state, const DevCard* cd, double* D64, float* D32,
                  hipStream_t s) {
    qp_mf_kernel<PD, MIX><<<qp_mf_blocks(ck), 128, 0, s>>>(g, ck, state, cd, D64, D32);
  }
};
void launch_qp_mf(const Grid& g, const Chunk& ck, const double* state, const DevCard* cd, int pade, int mixing,
                  double* D64, float* D32, hipStream_t s) {
  if constexpr (MF_AVAILABLE) run_card<QpMfRun>(pade, mixing, g, ck, state, cd, D64, D32, s);
}

// Element matrices K_e = sum_g w_g B_g^T D_g B_g + h Lap (x) Mg for the 36
// node pairs a <= b.  A workgroup of EM_WAVES wavefronts covers 64
// consecutive elements and EM_WAVES pairs; the Gauss-point Hessians of those
// elements are staged once per Gauss point in LDS and shared by the
// wavefronts (wave = pair, lane = element), so each Hessian is read from L2
// 36 / EM_WAVES times in total.  Four waves leave room for the NDOF^2 FP64
// accumulators in registers (81 for N = 6: no spills).
constexpr int EM_WAVES = 4;
// workgroups per CU the registers are budgeted for (the staged Hessians of
// 15 unknowns per node take 116 KB of LDS: one workgroup per CU)
constexpr int EM_MINB = NHP_PAD * 64 * 8 <= 80 * 1024 ? 2 : 1;

__device__ __forceinline__ void element_matrix_body(const Grid& g, const Chunk& ck, const double* __restrict__ qp,
                                                    const DevCard* __restrict__ cd, double* __restrict__ E,
                                                    int bid, int nblk) {
  __shared__ double Ds[NHP_PAD * 64];
  // the NPAIR / EM_WAVES pair chunks of one element group are consecutive
  // logical blocks on one XCD, so the group's Hessians are read from HBM once
  // and then hit that XCD's L2
  const int groups = ck.NEcpad / 64;
  constexpr int chunks = NPAIR / EM_WAVES;
  const int Lb = xcd_logical(bid, nblk);
  if (Lb >= groups * chunks) return;  // uniform; before any barrier
  const int eg = Lb / chunks;
  const int pc = Lb % chunks;  // pair chunk
  const int w = threadIdx.x >> 6, l = threadIdx.x & 63;
  const int p = pc * EM_WAVES + w;  // pair 0..35
  int a = 0, rem = p;
  while (rem >= 8 - a) { rem -= 8 - a; ++a; }
  const int b = a + rem;
  const int e = eg * 64 + l;
  const double cuu = g.h * 0.125, cue = g.h * g.h * 0.125, cee = g.h * g.h * g.h * 0.125;
  const int64_t stride = (int64_t)8 * ck.NEcpad;
  double K[NBLK];
#pragma unroll
  for (int q = 0; q < NBLK; ++q) K[q] = 0.0;
  for (int gp = 0; gp < 8; ++gp) {
    __syncthreads();
    {
      // direct global -> LDS loads (no registers involved): each wavefront
      // instruction moves two Hessian components of the group's 64 elements,
      // lanes 0-31 component c and lanes 32-63 component c + 1, 16 B (two
      // elements) per lane, landing at LDS base + 16 * lane
      const double* src = qp + (int64_t)(2 * w + (l >> 5)) * stride + (int64_t)gp * ck.NEcpad + eg * 64 +
                          2 * (l & 31);
#pragma unroll
      for (int r = 0; r < NHP_PAD / (2 * EM_WAVES); ++r) {
        const int c = 2 * (w + EM_WAVES * r);
        __builtin_amdgcn_global_load_lds((const void*)(src + (int64_t)(2 * EM_WAVES * r) * stride),
                                         (__attribute__((address_space(3))) void*)(Ds + c * 64), 16, 0, 0);
      }
      __builtin_amdgcn_s_waitcnt(0);
    }
    __syncthreads();
    const Shape sa = shape(gp, a), sb = shape(gp, b);
#define DV(pq) Ds[(pq) * 64 + l]
    // u-u: K[i3][k3] += h/8 sum_jl dNa_j dNb_l D(3 i3 + j, 3 k3 + l)
#pragma unroll
    for (int i3 = 0; i3 < 3; ++i3)
#pragma unroll
      for (int k3 = 0; k3 < 3; ++k3) {
        double sacc = 0.0;
#pragma unroll
        for (int jj = 0; jj < 3; ++jj)
#pragma unroll
          for (int ll = 0; ll < 3; ++ll) {
            const int pp = 3 * i3 + jj, rr = 3 * k3 + ll;
            const int pq = pp <= rr ? hidx(pp, rr) : hidx(rr, pp);
            sacc += sa.dN[jj] * sb.dN[ll] * DV(pq);
          }
        K[NDOF * i3 + k3] += cuu * sacc;
      }
    // u-eta and eta-u
#pragma unroll
    for (int m = 0; m < NV; ++m)
#pragma unroll
      for (int i3 = 0; i3 < 3; ++i3) {
        const double d0 = DV(hidx(3 * i3, 9 + m)), d1 = DV(hidx(3 * i3 + 1, 9 + m)), d2 = DV(hidx(3 * i3 + 2, 9 + m));
        K[NDOF * i3 + 3 + m] += cue * sb.N * (sa.dN[0] * d0 + sa.dN[1] * d1 + sa.dN[2] * d2);
        K[NDOF * (3 + m) + i3] += cue * sa.N * (sb.dN[0] * d0 + sb.dN[1] * d1 + sb.dN[2] * d2);
      }
    // eta-eta
    const double nn = cee * sa.N * sb.N;
#pragma unroll
    for (int m = 0; m < NV; ++m)
#pragma unroll
      for (int m2 = 0; m2 < NV; ++m2) {
        const int pq = m <= m2 ? hidx(9 + m, 9 + m2) : hidx(9 + m2, 9 + m);
        K[NDOF * (3 + m) + 3 + m2] += nn * DV(pq);
      }
#undef DV
  }
  // gradient energy: h * Lap_ab * Mg (exact under 2x2x2 Gauss)
  const double lap = g.h * lap_ref(a, b);
#pragma unroll
  for (int m = 0; m < NV; ++m)
#pragma unroll
    for (int m2 = 0; m2 < NV; ++m2) K[NDOF * (3 + m) + 3 + m2] += lap * cd->Mg[m][m2];
  if (e < ck.NEc) {
#pragma unroll
    for (int q = 0; q < NBLK; ++q) E[((int64_t)p * NBLK + q) * ck.NEcpad + e] = K[q];
  }
}
__global__ void __launch_bounds__(EM_WAVES * 64, EM_MINB) element_matrix_kernel(Grid g, Chunk ck,
                                                                          const double* __restrict__ qp,
                                                                          const DevCard* __restrict__ cd,
                                                                          double* __restrict__ E) {
  element_matrix_body(g, ck, qp, cd, E, blockIdx.x, gridDim.x);
}

void launch_element_matrices(const Grid& g, const Chunk& ck, const double* qp, const DevCard* cd, double* elem,
                             hipStream_t s) {
  const int nb = ck.NEcpad / 64 * (NPAIR / EM_WAVES);
  element_matrix_kernel<<<(nb + 7) / 8 * 8, EM_WAVES * 64, 0, s>>>(g, ck, qp, cd, elem);
}

// Stored block (n, n + off(13 + u)) = sum over the <= 8 elements containing
// both nodes of their element blocks, in a fixed order (bitwise reproducible);
// the second node never precedes the first, nor does its corner, so every
// element block is read as stored.
// Bound by reading the element blocks once and writing the rows.  A workgroup
// takes a (tile, u): coalesced element reads of 64 consecutive rows, each
// wavefront JG_E block entries, written as 16-byte words.  (One wavefront for
// the whole block, three rows of it at a time, is a chain of up to 24 rounds
// of loads.)  33^3 nodes: 470 -> 207 us (1.25 GB, 6 TB/s), 17^3 204 -> 27,
// 5^3 162 -> below 16; 15 unknowns per node, 10648 nodes: 1084 -> 286.
constexpr int JG_E = 12;  // whole 16-byte words of either type
constexpr int JG_CHUNKS = (Lay<float>::NE + JG_E - 1) / JG_E;  // the last one may be short
constexpr int JG_WAVES = JG_CHUNKS <= 16 ? JG_CHUNKS : (JG_CHUNKS + 1) / 2;
static_assert(JG_E % Lay<float>::V == 0 && JG_E % Lay<double>::V == 0 && JG_WAVES <= 16);
__device__ __forceinline__ void jacobian_gather_body(const Grid& g, const Chunk& ck, const double* __restrict__ E,
                                                     double* __restrict__ A64, float* __restrict__ A32,
                                                     double* __restrict__ diag64, int nblocks, int bid, int nblk) {
  const int L = xcd_logical(bid, nblk);
  if (L >= nblocks) return;
  const int t = ck.n0 / TILE + L / NUP, u = L % NUP;
  const int sten = 13 + u;
  const int l = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int n = t * TILE + l;
  if (n < ck.n0 || n >= ck.n1) return;  // rows of other slabs (no barriers below)
  const int dx = sten % 3 - 1, dy = (sten / 3) % 3 - 1, dz = sten / 9 - 1;
  const bool inside = n < g.N;
  const int i = n % g.nnx, j = (n / g.nnx) % g.nny, k = n / (g.nnx * g.nny);
  const int64_t es = ck.NEcpad;
  for (int ch = w; ch < JG_CHUNKS; ch += JG_WAVES) {
    const int q0 = ch * JG_E;
    double K[JG_E];
#pragma unroll
    for (int q = 0; q < JG_E; ++q) K[q] = 0.0;
    for (int a = 0; a < 8; ++a) {
      const int ax = a & 1, ay = (a >> 1) & 1, az = (a >> 2) & 1;
      const int bx = ax + dx, by = ay + dy, bz = az + dz;
      if (bx < 0 || bx > 1 || by < 0 || by > 1 || bz < 0 || bz > 1) continue;  // wave-uniform
      const int ex = i - ax, ey = j - ay, ez = k - az;
      if (!inside || ex < 0 || ex >= g.nx || ey < 0 || ey >= g.ny || ez < 0 || ez >= g.nz) continue;
      const int b = bx + 2 * by + 4 * bz;
      const int64_t e = ex + (int64_t)g.nx * (ey + (int64_t)g.ny * ez) - ck.e0;  // local, in [0, NEc)
      const double* src = E + ((int64_t)pair_index(a, b) * NBLK + q0) * es + e;
#pragma unroll
      for (int q = 0; q < JG_E; ++q)
        if (q0 + q < NBLK) K[q] += src[q * es];
    }
    auto put64 = [&](double* D) {
#pragma unroll
      for (int q = 0; q < JG_E; q += 2)
        if (q0 + q < Lay<double>::NE) *reinterpret_cast<double2*>(D + Lay<double>::off(q0 + q, l)) = double2{K[q], K[q + 1]};
    };
    if (A64) put64(A64 + (int64_t)(t * NUP + u) * Lay<double>::SLICE);
    if (u == 0 && diag64) put64(diag64 + (int64_t)t * Lay<double>::SLICE);
    if (A32) {
      float* D = A32 + (int64_t)(t * NUP + u) * Lay<float>::SLICE;
#pragma unroll
      for (int q = 0; q < JG_E; q += 4)
        if (q0 + q < Lay<float>::NE)
          *reinterpret_cast<float4*>(D + Lay<float>::off(q0 + q, l)) =
              float4{(float)K[q], (float)K[q + 1], (float)K[q + 2], (float)K[q + 3]};
    }
  }
}
__global__ void __launch_bounds__(64 * JG_WAVES) jacobian_gather_kernel(Grid g, Chunk ck, const double* __restrict__ E,
                                                                        double* __restrict__ A64,
                                                                        float* __restrict__ A32,
                                                                        double* __restrict__ diag64, int nblocks) {
  jacobian_gather_body(g, ck, E, A64, A32, diag64, nblocks, blockIdx.x, gridDim.x);
}

void launch_jacobian_gather(const Grid& g, const Chunk& ck, const double* elem, double* A64, float* A32,
                            double* diag64, hipStream_t s) {
  const int t0 = ck.n0 / TILE, t1 = (ck.n1 + TILE - 1) / TILE;
  const int nblocks = (t1 - t0) * NUP;
  const int nb_pad = (nblocks + 7) / 8 * 8;
  jacobian_gather_kernel<<<nb_pad, 64 * JG_WAVES, 0, s>>>(g, ck, elem, A64, A32, diag64, nblocks);
}

// Symmetric elimination on the stored blocks (nup = NUP; nup = 1: the diagonal
// blocks of a matrix-free level): entries in constrained rows of
// node n or constrained columns of node m are zeroed, the diagonal of a
// constrained dof is 1.
__device__ __forceinline__ void apply_dirichlet_body(const Grid& g, const uint16_t* __restrict__ mask,
                                                     double* __restrict__ A64, float* __restrict__ A32,
                                                     double* __restrict__ diag64, int nblocks, int nup, int bid,
                                                     int nblk) {
  const int L = xcd_logical(bid, nblk);
  if (L >= nblocks) return;
  const int t = L / nup, u = L - t * nup;
  const int sten = 13 + u;
  const int l = threadIdx.x;
  const int n = t * TILE + l;
  if (n >= g.N) return;
  const int dx = sten % 3 - 1, dy = (sten / 3) % 3 - 1, dz = sten / 9 - 1;
  const int i = n % g.nnx, j = (n / g.nnx) % g.nny, k = n / (g.nnx * g.nny);
  if (i + dx < 0 || i + dx >= g.nnx || j + dy < 0 || j + dy >= g.nny || k + dz < 0 || k + dz >= g.nnz) return;
  const int m = n + dx + g.nnx * (dy + g.nny * dz);
  const unsigned mr = mask[n], mc = mask[m];
  if ((mr | mc) == 0) return;
  const int64_t base64 = (int64_t)(t * NUP + u) * Lay<double>::SLICE;
  const int64_t base32 = (int64_t)(t * NUP + u) * Lay<float>::SLICE;
  const int64_t db = (int64_t)t * Lay<double>::SLICE;
  for (int e = 0; e < NBLK; ++e) {
    const int r = e / NDOF, c = e % NDOF;
    if (((mr >> r) & 1) || ((mc >> c) & 1)) {
      const double v = (u == 0 && r == c) ? 1.0 : 0.0;
      if (A64) A64[base64 + Lay<double>::off(e, l)] = v;
      if (A32) A32[base32 + Lay<float>::off(e, l)] = (float)v;
      if (u == 0 && diag64) diag64[db + Lay<double>::off(e, l)] = v;
    }
  }
}
__global__ void __launch_bounds__(64) apply_dirichlet_kernel(Grid g, const uint16_t* __restrict__ mask,
                                                             double* __restrict__ A64, float* __restrict__ A32,
                                                             double* __restrict__ diag64, int nblocks, int nup) {
  apply_dirichlet_body(g, mask, A64, A32, diag64, nblocks, nup, blockIdx.x, gridDim.x);
}

void launch_apply_dirichlet(const Grid& g, const uint16_t* mask, double* A64, float* A32, double* diag64,
                            hipStream_t s) {
  const int nup = (A64 || A32) ? NUP : 1;
  const int nblocks = g.ntiles * nup;
  const int nb_pad = (nblocks + 7) / 8 * 8;
  apply_dirichlet_kernel<<<nb_pad, TILE, 0, s>>>(g, mask, A64, A32, diag64, nblocks, nup);
}

// NDOF x NDOF inverse by Gauss-Jordan elimination with partial pivoting (the
// paper's point-block Jacobi inverts each block by LU with partial
// pivoting).  Pivot: the largest magnitude in the column among the rows not
// yet pivoted, ties to the lowest row.
//  * NDOF <= 9: one thread per block, the matrix in registers and inverted in
//    place (Gauss-Jordan on A itself: the pivot row is scaled with the
//    reciprocal on the diagonal, the other rows eliminated with the negated
//    multiples in the pivot column); the row interchanges are selects over
//    the rows below, and are undone as column interchanges in reverse order
//    (the steps invert P A, and A^-1 = (P A)^-1 P), applied as the columns'
//    store positions.
//  * larger blocks: 16 lanes per block, lane = row, inverted in place in the
//    lanes' registers with the pivot row sent to all of them; rows stay where
//    they are and the permutation is undone in the store.  (A thread per
//    block with [A | I] in LDS: 16 threads to a workgroup, a serial chain of
//    LDS accesses.  15 x 15, 10648 blocks: 600 -> 36 us, 1331 blocks 334 -> below 25.)
// DinvS32 (NDOF <= 9; null otherwise): the upper triangle of the FP32
// inverse, packed.  The blocks are symmetric (diagonal blocks of the Hessian
// of the potential, Sec. 3.4), so are their inverses up to rounding.
constexpr bool BI_REGS = NDOF <= 9;
constexpr int BI_NODES = BI_REGS ? 64 : 16;  // blocks per workgroup
constexpr int BI_THREADS = BI_REGS ? BI_NODES : BI_NODES * 16;
static_assert(BI_REGS || NDOF <= 16);

__device__ __forceinline__ void block_inverse_regs(const Grid& g, const double* __restrict__ diag64,
                                                   double* __restrict__ Dinv64, float* __restrict__ Dinv32,
                                                   float* __restrict__ DinvS32, int* status, int n) {
  const int t = n / TILE, l = n % TILE;
  const int64_t db = (int64_t)t * Lay<double>::SLICE;
  const int64_t db32 = (int64_t)t * Lay<float>::SLICE;
  const int64_t dbs = (int64_t)t * LaySym<float>::SLICE;
  bool ok = n < g.N;
  double A[NDOF][NDOF];
#pragma unroll
  for (int r = 0; r < NDOF; ++r)
#pragma unroll
    for (int c = 0; c < NDOF; ++c) A[r][c] = ok ? diag64[db + Lay<double>::off(NDOF * r + c, l)] : 0.0;
  int piv[NDOF];
#pragma unroll
  for (int k = 0; k < NDOF; ++k) {
    int p = k;
    double best = fabs(A[k][k]);
#pragma unroll
    for (int r = k + 1; r < NDOF; ++r) {
      const double v = fabs(A[r][k]);
      if (v > best) { best = v; p = r; }
    }
    piv[k] = p;
    ok = ok && best > 0.0;
#pragma unroll
    for (int r = k + 1; r < NDOF; ++r) {
      const bool sw = p == r;
#pragma unroll
      for (int c = 0; c < NDOF; ++c) {
        const double a = A[k][c], b = A[r][c];
        A[k][c] = sw ? b : a;
        A[r][c] = sw ? a : b;
      }
    }
    const double ip = 1.0 / (ok ? A[k][k] : 1.0);
#pragma unroll
    for (int c = 0; c < NDOF; ++c) A[k][c] = (c == k) ? ip : A[k][c] * ip;
#pragma unroll
    for (int r = 0; r < NDOF; ++r) {
      if (r == k) continue;
      const double f = A[r][k];
#pragma unroll
      for (int c = 0; c < NDOF; ++c) A[r][c] = (c == k) ? -f * ip : A[r][c] - f * A[k][c];
    }
  }
  // column interchanges k <-> piv[k] in reverse order, applied through the
  // store: column m of the registers goes to column dst[m] of the inverse
  int dst[NDOF];
#pragma unroll
  for (int m = 0; m < NDOF; ++m) dst[m] = m;
#pragma unroll
  for (int k = NDOF - 1; k >= 0; --k) {
    const int p = piv[k];
#pragma unroll
    for (int m = 0; m < NDOF; ++m) dst[m] = dst[m] == k ? p : (dst[m] == p ? k : dst[m]);
  }
  if (n < g.N && !ok) atomicOr(status, SETUP_SINGULAR);
#pragma unroll
  for (int r = 0; r < NDOF; ++r)
#pragma unroll
    for (int m = 0; m < NDOF; ++m) {
      const double v = ok ? A[r][m] : 0.0;
      if (Dinv64) Dinv64[db + Lay<double>::off(NDOF * r + dst[m], l)] = v;
      if (Dinv32) Dinv32[db32 + Lay<float>::off(NDOF * r + dst[m], l)] = (float)v;
      if (DinvS32 && r <= dst[m]) DinvS32[dbs + LaySym<float>::off(sym_index(r, dst[m]), l)] = (float)v;
    }
}

__device__ __forceinline__ void block_inverse_rows(const Grid& g, const double* __restrict__ diag64,
                                                   double* __restrict__ Dinv64, float* __restrict__ Dinv32,
                                                   int* status, int n) {
  const int t = n / TILE, l = n % TILE, r = threadIdx.x & 15;
  const int64_t db = (int64_t)t * Lay<double>::SLICE;
  const int64_t db32 = (int64_t)t * Lay<float>::SLICE;
  bool ok = n < g.N, act = r < NDOF;
  double a[NDOF];
#pragma unroll
  for (int c = 0; c < NDOF; ++c) a[c] = ok && act ? diag64[db + Lay<double>::off(NDOF * r + c, l)] : 0.0;
  int piv[NDOF], row = 0;  // row of the inverse that this lane ends with
#pragma unroll
  for (int k = 0; k < NDOF; ++k) {
    const double v = act ? fabs(a[k]) : -1.0;
    double m = v;
#pragma unroll
    for (int x = 1; x < 16; x *= 2) m = fmax(m, __shfl_xor(m, x, 16));
    const unsigned win = (unsigned)(__ballot(act && v == m) >> (threadIdx.x & 48)) & 0xFFFFu;
    ok = ok && m > 0.0 && win;
    const int p = win ? __ffs(win) - 1 : 0;
    piv[k] = p;
    const bool mine = r == p;
    if (mine) row = k;
    act = act && !mine;
    double s[NDOF];
#pragma unroll
    for (int c = 0; c < NDOF; ++c) s[c] = __shfl(a[c], p, 16);
    const double ip = 1.0 / (ok ? s[k] : 1.0), f = a[k];
#pragma unroll
    for (int c = 0; c < NDOF; ++c) {
      const double q = (c == k) ? ip : s[c] * ip;
      a[c] = mine ? q : (c == k ? 0.0 : a[c]) - f * q;
    }
  }
  if (n < g.N && !ok && r == 0) atomicOr(status, SETUP_SINGULAR);
  if (r >= NDOF) return;
  // A^-1[c][p_m] sits in lane p_c, column m
#pragma unroll
  for (int m = 0; m < NDOF; ++m) {
    const double v = ok ? a[m] : 0.0;
    const int e = NDOF * (ok ? row : r) + (ok ? piv[m] : m);
    if (Dinv64) Dinv64[db + Lay<double>::off(e, l)] = v;
    if (Dinv32) Dinv32[db32 + Lay<float>::off(e, l)] = (float)v;
  }
}

__device__ __forceinline__ void block_inverse_body(const Grid& g, const double* __restrict__ diag64,
                                                   double* __restrict__ Dinv64, float* __restrict__ Dinv32,
                                                   float* __restrict__ DinvS32, int* status, int bid) {
  const int n = bid * BI_NODES + threadIdx.x / (BI_THREADS / BI_NODES);
  if (n >= g.Npad) return;  // whole tiles, so whole wavefronts
  if constexpr (BI_REGS)
    block_inverse_regs(g, diag64, Dinv64, Dinv32, DinvS32, status, n);
  else
    block_inverse_rows(g, diag64, Dinv64, Dinv32, status, n);
}
__global__ void __launch_bounds__(BI_THREADS) block_inverse_kernel(Grid g, const double* __restrict__ diag64,
                                                                   double* __restrict__ Dinv64,
                                                                   float* __restrict__ Dinv32,
                                                                   float* __restrict__ DinvS32, int* status) {
  block_inverse_body(g, diag64, Dinv64, Dinv32, DinvS32, status, blockIdx.x);
}

void launch_block_inverse(const Grid& g, const double* diag64, double* Dinv64, float* Dinv32, float* DinvS32,
                          int* status, hipStream_t s) {
  block_inverse_kernel<<<(g.Npad + BI_NODES - 1) / BI_NODES, BI_THREADS, 0, s>>>(
      g, diag64, Dinv64, Dinv32, BI_REGS ? DinvS32 : nullptr, status);
}

// ---- batched assembly (jobs of many problems in one launch) --------------------
template <int PD, int MIX>
__global__ void __launch_bounds__(128) qp_hess_batch(const AJob* __restrict__ jobs, int njobs) {
  int bid;
  const AJob& j = find_job(jobs, njobs, bid);
  qp_body<PD, MIX>(j.g, j.ck, j.state, j.cd, j.qp, bid);
}
template <int PD, int MIX>
__global__ void __launch_bounds__(128) qp_mf_batch(const AJob* __restrict__ jobs, int njobs) {
  int bid;
  const AJob& j = find_job(jobs, njobs, bid);
  qp_mf_body<PD, MIX>(j.g, j.ck, j.state, j.cd, j.D64, j.D32, bid);
}
__global__ void __launch_bounds__(EM_WAVES * 64, EM_MINB) element_matrix_batch(const AJob* __restrict__ jobs, int njobs) {
  int bid;
  const AJob& j = find_job(jobs, njobs, bid);
  element_matrix_body(j.g, j.ck, j.qp, j.cd, j.elem, bid, j.nblk);
}
__global__ void __launch_bounds__(64 * JG_WAVES) jacobian_gather_batch(const AJob* __restrict__ jobs, int njobs) {
  int bid;
  const AJob& j = find_job(jobs, njobs, bid);
  jacobian_gather_body(j.g, j.ck, j.elem, j.A64, j.A32, j.diag64, j.nblocks, bid, j.nblk);
}
__global__ void __launch_bounds__(64) apply_dirichlet_batch(const AJob* __restrict__ jobs, int njobs) {
  int bid;
  const AJob& j = find_job(jobs, njobs, bid);
  apply_dirichlet_body(j.g, j.mask, j.A64, j.A32, j.diag64, j.nblocks, j.nup, bid, j.nblk);
}
__global__ void __launch_bounds__(BI_THREADS) block_inverse_batch(const AJob* __restrict__ jobs, int njobs) {
  int bid;
  const AJob& j = find_job(jobs, njobs, bid);
  block_inverse_body(j.g, j.diag64, j.Dinv64, j.Dinv32, BI_REGS ? j.DinvS32 : nullptr, j.status, bid);
}
template <int PD, int MIX>
__global__ void __launch_bounds__(256) residual_element_batch(const AJob* __restrict__ jobs, int njobs) {
  int bid;
  const AJob& j = find_job(jobs, njobs, bid);
  residual_element_body<PD, MIX>(j.g, j.ck, j.state, j.cd, j.out, bid, j.nblk);
}
__global__ void __launch_bounds__(256) residual_nodes_batch(const AJob* __restrict__ jobs, int njobs) {
  int bid;
  const AJob& j = find_job(jobs, njobs, bid);
  residual_nodes_body(j.g, j.ck, j.out, j.R, bid);
}

// the launch shapes of the single-problem launchers, per job
int assembly_job_blocks(int op, AJob& j) {
  const Grid& g = j.g;
  const Chunk& ck = j.ck;
  switch (op) {
    case AOP_QP_HESS: return (int)(((int64_t)8 * ck.NEcpad + 127) / 128);
    case AOP_QP_MF: return qp_mf_blocks(ck);
    case AOP_ELEMENT: return ((ck.NEcpad / 64) * (NPAIR / EM_WAVES) + 7) / 8 * 8;
    case AOP_GATHER: {
      const int t0 = ck.n0 / TILE, t1 = (ck.n1 + TILE - 1) / TILE;
      j.nblocks = (t1 - t0) * NUP;
      return (j.nblocks + 7) / 8 * 8;
    }
    case AOP_MF_DIAG: return mf_diag_blocks(ck);
    case AOP_MF_DIAG_GATHER: return mf_diag_gather_blocks(ck);
    case AOP_DIRICHLET:
      j.nup = (j.A64 || j.A32) ? NUP : 1;
      j.nblocks = g.ntiles * j.nup;
      return (j.nblocks + 7) / 8 * 8;
    case AOP_BLOCK_INVERSE: return (g.Npad + BI_NODES - 1) / BI_NODES;
    case AOP_RESIDUAL: return ck.NEcpad / SLAB_EPW;
    case AOP_RESIDUAL_NODES: return (ck.n1 - ck.n0 + 255) / 256 * NDOF;
    default: return 0;
  }
}

struct QpHessBatch {
  template <int PD, int MIX>
  static void run(const AJob* jobs, int njobs, int blocks, hipStream_t s) {
    qp_hess_batch<PD, MIX><<<blocks, 128, 0, s>>>(jobs, njobs);
  }
};
struct QpMfBatch {
  template <int PD, int MIX>
  static void run(const AJob* jobs, int njobs, int blocks, hipStream_t s) {
    qp_mf_batch<PD, MIX><<<blocks, 128, 0, s>>>(jobs, njobs);
  }
};
struct ResidualBatch {
  template <int PD, int MIX>
  static void run(const AJob* jobs, int njobs, int blocks, hipStream_t s) {
    residual_element_batch<PD, MIX><<<blocks, 256, 0, s>>>(jobs, njobs);
  }
};

// pade = Pade order + QP_LOG_MIX for logarithmic mixing
void launch_assembly_batch(int op, int pade, const AJob* jobs, int njobs, int blocks, hipStream_t s) {
  if (njobs <= 0 || blocks <= 0) return;
  const int order = pade % QP_LOG_MIX, mixing = pade >= QP_LOG_MIX ? MVPF_MIX_LOG : MVPF_MIX_LINEAR;
  switch (op) {
    case AOP_QP_HESS: run_card<QpHessBatch>(order, mixing, jobs, njobs, blocks, s); break;
    case AOP_QP_MF:
      if constexpr (MF_AVAILABLE) run_card<QpMfBatch>(order, mixing, jobs, njobs, blocks, s);
      break;
    case AOP_RESIDUAL: run_card<ResidualBatch>(order, mixing, jobs, njobs, blocks, s); break;
    case AOP_RESIDUAL_NODES: residual_nodes_batch<<<blocks, 256, 0, s>>>(jobs, njobs); break;
    case AOP_ELEMENT: element_matrix_batch<<<blocks, EM_WAVES * 64, 0, s>>>(jobs, njobs); break;
    case AOP_GATHER: jacobian_gather_batch<<<blocks, 64 * JG_WAVES, 0, s>>>(jobs, njobs); break;
    case AOP_DIRICHLET: apply_dirichlet_batch<<<blocks, TILE, 0, s>>>(jobs, njobs); break;
    case AOP_BLOCK_INVERSE: block_inverse_batch<<<blocks, BI_THREADS, 0, s>>>(jobs, njobs); break;
    case AOP_MF_DIAG:
    case AOP_MF_DIAG_GATHER: launch_mf_diag_batch(op, jobs, njobs, blocks, s); break;
    default: break;
  }
}

}  // namespace mvpf
