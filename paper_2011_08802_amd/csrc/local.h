// Local (quadrature-point) derivatives of the penalised incremental potential
// density with respect to q = (F_00..F_22 row-major, eta_1..eta_N).
//
// Density (Sec. 2.2-2.3, 3.1-3.2; gradient-energy part handled separately by
// the element kernels since it is a constant quadratic form):
//   psi = sum_i eta_i F_i + 1/2 J_t H : L(eta) H + sum_{i<j} w_ij eta_i eta_j
//         + sum_i rho/2 (eta_i - eta_in)^2 + sum_i eps/2 <eta_i>_-^2
//   F^t = I + sum_k eta_k dU_k  (Eq. LinMix with U_0 = I, condensed),
//   J_t = det F^t, G = (F^t)^-1, C = G F^T F G  (C^e of Eq. elasticEn),
//   H = A(C) B(C)^-1, the Pade approximant of 1/2 log C of order (1,1), (2,2)
//   or (3,3) (Eqs. pade11, pade22, pade33; A and B are matrix polynomials in
//   C, the leading factor folded into A), L = L_0 + sum eta_k dL_k.
//
// Derivatives are closed-form, in three spaces:
//  * C-space, along the symmetric basis E_v (xx,yy,zz,yz,xz,xy; the shear ones
//    are e_a e_b^T + e_b e_a^T).  A and B are polynomials in C, so dH along E
//    is a sum of products of functions of C around E,
//      dH[E] = sum_p A_p E C^p B^-1,  A_p = sum_{q > p} (a_q - H b_q) C^(q-1-p),
//    and every term of the second derivative w_CC besides dH : L dH is a form
//    tr(M E_u N E_v) of 3x3 matrices: with T = L H, Y = T B^-1,
//      T : d2H_uv = Y : (d2A - H d2B) - Y : (dH_u dB_v + dH_v dB_u),
//      d2(C^2) = E_u E_v + E_v E_u,
//      d2(C^3) = (E_u E_v + E_v E_u) C + C (E_u E_v + E_v E_u) + E_u C E_v + E_v C E_u.
//    A basis pair costs 1, 2 or 4 products per form instead of 3x3 products
//    with the basis matrices' zeros.
//  * F^t-space (6 components, G = (F^t)^-1): dC/dF^t[E] = -(G E C + C E G),
//    d J_t[E] = J_t tr(G E), and their second derivatives; the order parameters
//    enter through dF^t/deta_k (the constants U_k - I under Eq. LinMix) and
//    through L(eta), which is linear.
//  * Green-strain space: with eps = sym(F^T dF) in engineering components,
//    dC = 2 G eps G, so the density's dependence on F is through eps alone:
//    second derivatives D_ee (6x6), D_ek (6xN), the stress S (dpsi = S : eps)
//    and F itself give the derivatives with respect to F,
//      d2psi/dF_ij dF_kl = sum_ab F_ia D_(aj)(bl) F_kb + delta_ik S_jl,
//      d2psi/dF_ij deta_k = sum_a F_ia D_(aj)k,  dpsi/dF = F S.
#pragma once
#include <hip/hip_runtime.h>

// Number of martensite variants N: a compile-time constant of the library
// (each build is one instantiation; 6 for CuAlNi, Sec. 4.1; 12 for a
// NiTi-like card, the footnote of Sec. 4.4).
#ifndef MVPF_NVAR
#define MVPF_NVAR 6
#endif

namespace mvpf {

constexpr int NV = MVPF_NVAR;           // variants N (order parameters per node)
constexpr int NQ = 9 + NV;              // local variables of a Gauss point: F (9), eta_hat (N)
constexpr int NHP = NQ * (NQ + 1) / 2;  // packed upper triangle of their Hessian
static_assert(NV >= 1 && NV <= 13, "unknowns per node must fit the 16-bit constraint masks");

// Material card on the device, in the sample frame.
struct DevCard {
  double dU[NV][6];    // U_k - I (k = 1..N) as symmetric components
  double L0[6][6];     // austenite stiffness, Voigt (engineering shear strain)
  double dL[NV][6][6];  // L_k - L_0
  double dF0[NV];      // F_k - F_0
  double W[NV + 1][NV + 1];   // double-obstacle coefficients, zero diagonal
  double Sw[NV][NV];     // condensed Hessian of 1/2 eta^T W eta w.r.t. eta_hat
  double Mg[NV][NV];     // gradient-energy species matrix: psi_g = 1/2 Mg_kl grad eta_k . grad eta_l
  float Mg32[NV][NV];    // Mg rounded to FP32 (the FP32 matrix-free operator)
  double rho;
  double eps;
  int pade;
  int mixing;          // MVPF_MIX_LINEAR (Eq. LinMix) or MVPF_MIX_LOG
  double logU[NV][6];  // log U_k (logarithmic mixing rule, Sec. 2.1)
};

// Boundary of a computation phase: the values given are computed before it
// and their uses come after it, so that the unrolled phases' temporaries are
// not all live at once.
__device__ __forceinline__ void phase(double& x) {
#if defined(__HIP_DEVICE_COMPILE__)
  asm volatile("" : "+v"(x));
#endif
}
// The card as one phase reads it: its constants are loaded no earlier (all of
// them at once would not fit the scalar registers), by scalar loads.
#if defined(__HIP_DEVICE_COMPILE__)
typedef const DevCard __attribute__((address_space(4))) PhaseCard;
__device__ __forceinline__ PhaseCard& phase(const DevCard& cd) {
  PhaseCard* p = (PhaseCard*)&cd;
  asm volatile("" : "+s"(p));
  return *p;
}
#else
typedef const DevCard PhaseCard;
__host__ __device__ inline PhaseCard& phase(const DevCard& cd) { return cd; }
#endif
template <int N>
__device__ __forceinline__ void phase(double (&x)[N]) {
#pragma unroll
  for (int i = 0; i < N; ++i) phase(x[i]);
}
template <int N, int M>
__device__ __forceinline__ void phase(double (&x)[N][M]) {
#pragma unroll
  for (int i = 0; i < N; ++i) phase(x[i]);
}

// symmetric index map (xx,yy,zz,yz,xz,xy)
__host__ __device__ constexpr int SI(int a, int b) {
  return a == b ? a : (a + b == 3 ? 3 : (a + b == 2 ? 4 : 5));
}

__device__ __forceinline__ void full_from_sym(const double s[6], double m[9]) {
#pragma unroll
  for (int a = 0; a < 3; ++a)
#pragma unroll
    for (int b = 0; b < 3; ++b) m[3 * a + b] = s[SI(a, b)];
}

// symmetric part components of a full matrix
__device__ __forceinline__ void sym_of(const double m[9], double s[6]) {
  s[0] = m[0];
  s[1] = m[4];
  s[2] = m[8];
  s[3] = 0.5 * (m[5] + m[7]);
  s[4] = 0.5 * (m[2] + m[6]);
  s[5] = 0.5 * (m[1] + m[3]);
}

__device__ __forceinline__ void mm(const double a[9], const double b[9], double c[9]) {
#pragma unroll
  for (int i = 0; i < 3; ++i)
#pragma unroll
    for (int j = 0; j < 3; ++j)
      c[3 * i + j] = a[3 * i] * b[j] + a[3 * i + 1] * b[3 + j] + a[3 * i + 2] * b[6 + j];
}

// engineering (Voigt strain) form of symmetric components
__device__ __forceinline__ void eng(const double s[6], double e[6]) {
  e[0] = s[0]; e[1] = s[1]; e[2] = s[2];
  e[3] = 2.0 * s[3]; e[4] = 2.0 * s[4]; e[5] = 2.0 * s[5];
}

// inverse and determinant of a symmetric 3x3 (components)
__device__ __forceinline__ double sym_inv(const double s[6], double r[6]) {
  const double xx = s[0], yy = s[1], zz = s[2], yz = s[3], xz = s[4], xy = s[5];
  const double c0 = yy * zz - yz * yz;
  const double c5 = xz * yz - xy * zz;  // cofactor (0,1)
  const double c4 = xy * yz - xz * yy;  // cofactor (0,2)
  const double det = xx * c0 + xy * c5 + xz * c4;
  const double id = 1.0 / det;
  r[0] = c0 * id;
  r[5] = c5 * id;
  r[4] = c4 * id;
  r[1] = (xx * zz - xz * xz) * id;
  r[3] = (xy * xz - xx * yz) * id;
  r[2] = (xx * yy - xy * xy) * id;
  return det;
}

__host__ __device__ constexpr int hidx(int p, int q) {  // packed upper triangle, p <= q < NQ
  return p * NQ - (p * (p - 1)) / 2 + (q - p);
}

// Coefficients of H = A B^-1 with A = sum_p a_p C^p, B = sum_p b_p C^p.
template <int ORDER> struct Pade;
template <> struct Pade<11> {  // (C - I)(C + I)^-1
  static constexpr int deg = 1;
  __host__ __device__ static constexpr double a(int p) { return p == 0 ? -1.0 : (p == 1 ? 1.0 : 0.0); }
  __host__ __device__ static constexpr double b(int p) { return p <= 1 ? 1.0 : 0.0; }
};
template <> struct Pade<22> {  // 3/2 (C^2 - I)(C^2 + 4C + I)^-1
  static constexpr int deg = 2;
  __host__ __device__ static constexpr double a(int p) { return p == 0 ? -1.5 : (p == 2 ? 1.5 : 0.0); }
  __host__ __device__ static constexpr double b(int p) { return p == 1 ? 4.0 : (p <= 2 ? 1.0 : 0.0); }
};
template <> struct Pade<33> {  // 1/6 (11C^3 + 27C^2 - 27C - 11I)(C^3 + 9C^2 + 9C + I)^-1
  static constexpr int deg = 3;
  __host__ __device__ static constexpr double a(int p) {
    return p == 0 ? -11.0 / 6.0 : (p == 1 ? -4.5 : (p == 2 ? 4.5 : 11.0 / 6.0));
  }
  __host__ __device__ static constexpr double b(int p) { return (p == 0 || p == 3) ? 1.0 : 9.0; }
};

// x += c m, the term dropped at compile time when c is zero
template <int N>
__device__ __forceinline__ void axpy_c(double c, const double m[N], double x[N]) {
  if (c == 0.0) return;
#pragma unroll
  for (int i = 0; i < N; ++i) x[i] += c * m[i];
}

// Quantities shared by the gradient and the Hessian.
template <int PD>
struct LocalBase {
  double Jt;
  double G[9];     // (F^t)^-1, full symmetric
  double C[9];     // C^e, full symmetric
  double H[9];     // Hencky strain, full symmetric
  double Binv[9];  // B^-1, full symmetric
  double h[6];     // engineering H
  double T[9];     // L H, full symmetric
  double w;        // 1/2 H : L H
  double wEta[NV]; // dw/deta_k at fixed C: 1/2 h : dL_k h
  double Sf[9];    // dw/dC: dw = Sf : dC, full symmetric
  double B1[9];    // C Sf G
};

// Terms of the power series of exp: exact to rounding for ||M||_F <= 1
// (the omitted tail is below 1/19! ~ 8e-18 there; the order parameters of
// the workloads keep ||sum eta_k log U_k|| near 0.1).
constexpr int EXP_TERMS = 18;

__device__ __forceinline__ void log_mixing_matrix(const double eh[NV], const DevCard& cd, double M[9]) {
  double Ms[6];
#pragma unroll
  for (int v = 0; v < 6; ++v) {
    double s = 0.0;
#pragma unroll
    for (int k = 0; k < NV; ++k) s += eh[k] * cd.logU[k][v];
    Ms[v] = s;
  }
  full_from_sym(Ms, M);
}

// F^t = exp(M), M = sum_k eta_k log U_k (logarithmic mixing, Sec. 2.1), and
// dF^t/deta_k = sum_n 1/n! d(M^n)[log U_k], by the power series with the
// recurrences M^n = M^(n-1) M and d(M^n)[A] = d(M^(n-1))[A] M + M^(n-1) A.
__device__ __forceinline__ void log_mixing(const double eh[NV], const DevCard& cd, double Ft[6],
                                           double dFt[NV][6]) {
  double M[9], P[9], E[9];
  log_mixing_matrix(eh, cd, M);
  double D[NV][9], Sd[NV][9];
#pragma unroll
  for (int i = 0; i < 9; ++i) P[i] = E[i] = (i % 4 == 0) ? 1.0 : 0.0;
#pragma unroll
  for (int k = 0; k < NV; ++k)
#pragma unroll
    for (int i = 0; i < 9; ++i) D[k][i] = Sd[k][i] = 0.0;
  double c = 1.0;
#pragma unroll 1
  for (int n = 1; n <= EXP_TERMS; ++n) {
    c /= n;
    double T[9];
#pragma unroll
    for (int k = 0; k < NV; ++k) {
      double A[9], DM[9], PA[9];
      full_from_sym(cd.logU[k], A);
      mm(D[k], M, DM);
      mm(P, A, PA);
#pragma unroll
      for (int i = 0; i < 9; ++i) {
        D[k][i] = DM[i] + PA[i];
        Sd[k][i] += c * D[k][i];
      }
    }
    mm(P, M, T);
#pragma unroll
    for (int i = 0; i < 9; ++i) {
      P[i] = T[i];
      E[i] += c * P[i];
    }
  }
  sym_of(E, Ft);
#pragma unroll
  for (int k = 0; k < NV; ++k) sym_of(Sd[k], dFt[k]);
}

// d^2 F^t / deta_k deta_l = sum_n 1/n! d^2(M^n)[A_k, A_l] (A = log U) with
// d^2(M^n)[A_k, A_l] = d^2(M^(n-1))[A_k, A_l] M + d(M^(n-1))[A_l] A_k
//                      + d(M^(n-1))[A_k] A_l.
__device__ __forceinline__ void log_mixing_second(const double eh[NV], const DevCard& cd, int k, int l,
                                                  double out[9]) {
  double M[9], P[9], Dk[9], Dl[9], S[9], Ak[9], Al[9];
  log_mixing_matrix(eh, cd, M);
  full_from_sym(cd.logU[k], Ak);
  full_from_sym(cd.logU[l], Al);
#pragma unroll
  for (int i = 0; i < 9; ++i) {
    P[i] = (i % 4 == 0) ? 1.0 : 0.0;
    Dk[i] = Dl[i] = S[i] = out[i] = 0.0;
  }
  double c = 1.0;
#pragma unroll 1
  for (int n = 1; n <= EXP_TERMS; ++n) {
    c /= n;
    double SM[9], DlA[9], DkA[9], DkM[9], DlM[9], PAk[9], PAl[9], T[9];
    mm(S, M, SM);
    mm(Dl, Ak, DlA);
    mm(Dk, Al, DkA);
    mm(Dk, M, DkM);
    mm(Dl, M, DlM);
    mm(P, Ak, PAk);
    mm(P, Al, PAl);
    mm(P, M, T);
#pragma unroll
    for (int i = 0; i < 9; ++i) {
      S[i] = SM[i] + DlA[i] + DkA[i];
      Dk[i] = DkM[i] + PAk[i];
      Dl[i] = DlM[i] + PAl[i];
      P[i] = T[i];
      out[i] += c * S[i];
    }
  }
}

// d/deta_k of F^t: the constants U_k - I (Eq. LinMix), or per point with
// logarithmic mixing, where F^t depends nonlinearly on eta.
template <int MIX>
struct MixDerivative {
  template <class Card>
  __device__ __forceinline__ double operator()(Card& cd, int k, int v) const { return cd.dU[k][v]; }
};
template <>
struct MixDerivative<1> {
  double dFt[NV][6];
  template <class Card>
  __device__ __forceinline__ double operator()(Card&, int k, int v) const { return dFt[k][v]; }
};

// corners a <= b of basis element E_v (xx,yy,zz,yz,xz,xy)
__host__ __device__ constexpr int BA(int v) { return v < 3 ? v : (v == 3 ? 1 : 0); }
__host__ __device__ constexpr int BB(int v) { return v < 3 ? v : (v == 5 ? 1 : 2); }

// (M E_v N)_ij
__device__ __forceinline__ double sandwich(const double M[9], const double N[9], int v, int i, int j) {
  const int a = BA(v), b = BB(v);
  double r = M[3 * i + a] * N[3 * b + j];
  if (v >= 3) r += M[3 * i + b] * N[3 * a + j];
  return r;
}
// tr(M E_u N E_v)
__device__ __forceinline__ double bilinear(const double M[9], const double N[9], int u, int v) {
  const int a = BA(u), b = BB(u), c = BA(v), d = BB(v);
  double r = M[3 * d + a] * N[3 * b + c];
  if (u >= 3) r += M[3 * d + b] * N[3 * a + c];
  if (v >= 3) r += M[3 * c + a] * N[3 * b + d];
  if (u >= 3 && v >= 3) r += M[3 * c + b] * N[3 * a + d];
  return r;
}
// product of two symmetric matrices that commute (functions of C): symmetric
__device__ __forceinline__ void mm_sym(const double a[9], const double b[9], double c[9]) {
#pragma unroll
  for (int i = 0; i < 3; ++i)
#pragma unroll
    for (int j = i; j < 3; ++j)
      c[3 * i + j] = c[3 * j + i] = a[3 * i] * b[j] + a[3 * i + 1] * b[3 + j] + a[3 * i + 2] * b[6 + j];
}
__device__ __forceinline__ double ident(int i) { return i % 4 == 0 ? 1.0 : 0.0; }

// A_p of dH[E] = sum_p A_p E C^p B^-1 (p = 0 .. deg - 1): symmetric functions
// of C; Cp holds C and C^2
template <int PD>
__device__ __forceinline__ void hencky_factor(int p, const double C[9], const double C2[9], const double H[9],
                                              double A[9]) {
  using P = Pade<PD>;
  double b[9];
#pragma unroll
  for (int i = 0; i < 9; ++i) A[i] = P::a(p + 1) * ident(i), b[i] = P::b(p + 1) * ident(i);
  if (p + 2 <= P::deg) axpy_c<9>(P::a(p + 2), C, A), axpy_c<9>(P::b(p + 2), C, b);
  if (p + 3 <= P::deg) axpy_c<9>(P::a(p + 3), C2, A), axpy_c<9>(P::b(p + 3), C2, b);
  if (p + 1 == P::deg) {  // b is a multiple of the identity
#pragma unroll
    for (int i = 0; i < 9; ++i) A[i] -= P::b(P::deg) * H[i];
  } else {
    double Hb[9];
    mm_sym(H, b, Hb);
#pragma unroll
    for (int i = 0; i < 9; ++i) A[i] -= Hb[i];
  }
}

// y = L x of a Voigt stiffness (symmetric: its upper triangle is read)
template <class M>
__device__ __forceinline__ void voigt_product(M& L, const double x[6], double y[6]) {
#pragma unroll
  for (int i = 0; i < 6; ++i) {
    double s = 0.0;
#pragma unroll
    for (int j = 0; j < 6; ++j) s += (i <= j ? L[i][j] : L[j][i]) * x[j];
    y[i] = s;
  }
}

// Hencky energy (Pade order PD) and its first C-derivative; MIX: the mixing
// rule of F^t (0: Eq. LinMix, 1: logarithmic).
template <int PD, int MIX>
__device__ __forceinline__ void local_base(const double F[9], const double eh[NV], const DevCard& cd,
                                           LocalBase<PD>& b, MixDerivative<MIX>& dm) {
  using P = Pade<PD>;
  double Ft[6];
  if constexpr (MIX == 1) {
    log_mixing(eh, cd, Ft, dm.dFt);
  } else {
#pragma unroll
    for (int v = 0; v < 6; ++v) {
      double s = (v < 3) ? 1.0 : 0.0;
#pragma unroll
      for (int k = 0; k < NV; ++k) s += eh[k] * cd.dU[k][v];
      Ft[v] = s;
    }
  }
  double Gs[6], Fe[9], C2[9], C3[9];
  b.Jt = sym_inv(Ft, Gs);
  full_from_sym(Gs, b.G);
  mm(F, b.G, Fe);
#pragma unroll
  for (int a = 0; a < 3; ++a)
#pragma unroll
    for (int c = a; c < 3; ++c)
      b.C[3 * a + c] = b.C[3 * c + a] = Fe[a] * Fe[c] + Fe[3 + a] * Fe[3 + c] + Fe[6 + a] * Fe[6 + c];
  if constexpr (P::deg >= 2) mm_sym(b.C, b.C, C2);
  if constexpr (P::deg >= 3) mm_sym(C2, b.C, C3);
  double Am[9], Bf[9];
#pragma unroll
  for (int i = 0; i < 9; ++i) {
    Am[i] = P::a(0) * ident(i) + P::a(1) * b.C[i];
    Bf[i] = P::b(0) * ident(i) + P::b(1) * b.C[i];
  }
  if constexpr (P::deg >= 2) axpy_c<9>(P::a(2), C2, Am), axpy_c<9>(P::b(2), C2, Bf);
  if constexpr (P::deg >= 3) axpy_c<9>(P::a(3), C3, Am), axpy_c<9>(P::b(3), C3, Bf);
  double Bs[6], Bi[6], Hs[6], Ts[6];
  sym_of(Bf, Bs);
  sym_inv(Bs, Bi);
  full_from_sym(Bi, b.Binv);
  mm_sym(Am, b.Binv, b.H);
  sym_of(b.H, Hs);
  eng(Hs, b.h);
  // Hencky stress T = L h of the mixed stiffness, dw/deta_k at fixed C
  voigt_product(cd.L0, b.h, Ts);
#pragma unroll
  for (int k = 0; k < NV; ++k) {
    double d[6], e = 0.0;
    voigt_product(phase(cd).dL[k], b.h, d);
#pragma unroll
    for (int i = 0; i < 6; ++i) {
      Ts[i] += eh[k] * d[i];
      e += b.h[i] * d[i];
    }
    b.wEta[k] = 0.5 * e;
    phase(Ts);
    phase(b.wEta[k]);
  }
  double w = 0.0;
#pragma unroll
  for (int i = 0; i < 6; ++i) w += b.h[i] * Ts[i];
  b.w = 0.5 * w;
  full_from_sym(Ts, b.T);
  // dw/dC = sym sum_p C^p B^-1 T A_p
  double S[9], N[9];
#pragma unroll
  for (int i = 0; i < 9; ++i) S[i] = 0.0, N[i] = b.Binv[i];
#pragma unroll
  for (int p = 0; p < P::deg; ++p) {
    double A[9], TA[9], X[9];
    hencky_factor<PD>(p, b.C, C2, b.H, A);
    mm(b.T, A, TA);
    mm(N, TA, X);
#pragma unroll
    for (int i = 0; i < 9; ++i) S[i] += X[i];
    if (p + 1 < P::deg) {
      double Nn[9];
      mm_sym(b.C, N, Nn);
#pragma unroll
      for (int i = 0; i < 9; ++i) N[i] = Nn[i];
    }
  }
  double Ss[6], SG[9];
  sym_of(S, Ss);
  full_from_sym(Ss, b.Sf);
  mm(b.Sf, b.G, SG);
  mm(b.C, SG, b.B1);
}

__device__ __forceinline__ double neg_part(double x) { return x < 0.0 ? x : 0.0; }

// stress S (dpsi = S : sym(F^T dF), 6 components) and the derivative phi of
// the elastic energy along F^t (dpsi = sum_v phi_v dF^t_v at fixed L)
template <int PD>
__device__ __forceinline__ void local_first(const LocalBase<PD>& b, double S[6], double phi[6]) {
  double SG[9];
  mm(b.Sf, b.G, SG);
#pragma unroll
  for (int v = 0; v < 6; ++v) {
    const int i = BA(v), j = BB(v);
    S[v] = 2.0 * b.Jt * (b.G[3 * i] * SG[j] + b.G[3 * i + 1] * SG[3 + j] + b.G[3 * i + 2] * SG[6 + j]);
    // tr(G E_v) = G_ii or 2 G_ij; dC = -(G E C + C E G) gives -(B1 + B1^T) : E
    phi[v] = b.Jt * (v < 3 ? b.G[3 * i + j] * b.w - 2.0 * b.B1[3 * i + j]
                           : 2.0 * (b.G[3 * i + j] * b.w - b.B1[3 * i + j] - b.B1[3 * j + i]));
  }
}

// eta part of the gradient: elastic through F^t and L, chemical, double
// obstacle, viscous and penalty terms
template <int MIX>
__device__ __forceinline__ void eta_gradient(const double eh[NV], const double ehn[NV], const DevCard& cd, double Jt,
                                             const double wEta[NV], const MixDerivative<MIX>& dm, const double phi[6],
                                             double g[NV]) {
  double eta[NV + 1], etan[NV + 1];
  double s = 0.0, sn = 0.0;
#pragma unroll
  for (int k = 0; k < NV; ++k) { eta[k + 1] = eh[k]; etan[k + 1] = ehn[k]; s += eh[k]; sn += ehn[k]; }
  eta[0] = 1.0 - s;
  etan[0] = 1.0 - sn;
  double We[NV + 1];
#pragma unroll
  for (int i = 0; i < NV + 1; ++i) {
    double t = 0.0;
#pragma unroll
    for (int j = 0; j < NV + 1; ++j) t += cd.W[i][j] * eta[j];
    We[i] = t;
  }
  const double d0 = eta[0] - etan[0];
  const double n0 = neg_part(eta[0]);
#pragma unroll
  for (int k = 0; k < NV; ++k) {
    double t = Jt * wEta[k];
#pragma unroll
    for (int i = 0; i < 6; ++i) t += phi[i] * dm(cd, k, i);
    g[k] = t;
    g[k] += cd.dF0[k] + (We[k + 1] - We[0]) + cd.rho * ((eta[k + 1] - etan[k + 1]) - d0)
            + cd.eps * (neg_part(eta[k + 1]) - n0);
  }
}

// dpsi/dF = F S
__device__ __forceinline__ void first_piola(const double F[9], const double S[6], double g[9]) {
  double Sm[9];
  full_from_sym(S, Sm);
  mm(F, Sm, g);
}

// Gradient of the local density: g[NQ].
template <int PD, int MIX = 0>
__device__ __forceinline__ void local_gradient(const double F[9], const double eh[NV], const double ehn[NV],
                                               const DevCard& cd, double g[NQ]) {
  LocalBase<PD> b;
  MixDerivative<MIX> dm;
  double S[6], phi[6];
  local_base<PD, MIX>(F, eh, cd, b, dm);
  local_first<PD>(b, S, phi);
  first_piola(F, S, g);
  eta_gradient<MIX>(eh, ehn, cd, b.Jt, b.wEta, dm, phi, g + 9);
}

// index of D_ee entry (u, v) among its 21 upper entries
__host__ __device__ constexpr int eidx(int u, int v) {
  return u <= v ? u * 6 - u * (u - 1) / 2 + (v - u) : v * 6 - v * (v - 1) / 2 + (u - v);
}

// 2 G q G for the symmetric tensor whose contraction components are q
// (tensor components q_aa and q_ab / 2): sum_i (dC along eps_w)_i q_i
__device__ __forceinline__ void to_strain(const double G[9], const double q[6], double r[6]) {
  const double Q[9] = {q[0], 0.5 * q[5], 0.5 * q[4], 0.5 * q[5], q[1], 0.5 * q[3], 0.5 * q[4], 0.5 * q[3], q[2]};
  double GQ[9];
  mm(G, Q, GQ);
#pragma unroll
  for (int w = 0; w < 6; ++w) {
    const int i = BA(w), j = BB(w);
    r[w] = 2.0 * (GQ[3 * i] * G[j] + GQ[3 * i + 1] * G[3 + j] + GQ[3 * i + 2] * G[6 + j]);
  }
}

// Second derivatives of the local density in (eps, eta), handed to out as soon
// as they are known (so that few stay live): out.strain(S, D_ee) with the stress
// and the upper triangle, out.eps_eta(k, d) with the six entries D_(.)k,
// out.eta_eta(k, l, val) for l <= k.
template <int PD, int MIX, class Out>
__device__ __forceinline__ void local_hessian(const double F[9], const double eh[NV], const DevCard& cd, Out&& out) {
  using P = Pade<PD>;
  LocalBase<PD> b;
  MixDerivative<MIX> dm;
  double S[6], phi[6];
  local_base<PD, MIX>(F, eh, cd, b, dm);
  local_first<PD>(b, S, phi);
  // ---- second derivatives in C-space -------------------------------------
  double dh[6][6];  // engineering components of dH along E_v
  double wCC[21];   // upper triangle
  {
    constexpr int NF = 2 * P::deg - 1;  // forms tr(M_q E_u C^q B^-1 E_v), q < NF
    double C2[9], N[NF][9], M[NF][9], Y[9], Yt[9];
    if constexpr (P::deg >= 2) mm_sym(b.C, b.C, C2);
#pragma unroll
    for (int i = 0; i < 9; ++i) N[0][i] = b.Binv[i];
#pragma unroll
    for (int q = 1; q < NF; ++q) mm_sym(b.C, N[q - 1], N[q]);
    mm(b.T, b.Binv, Y);
#pragma unroll
    for (int i = 0; i < 9; ++i) Yt[i] = Y[3 * (i % 3) + i / 3];
#pragma unroll
    for (int q = 0; q < NF; ++q)
#pragma unroll
      for (int i = 0; i < 9; ++i) M[q][i] = 0.0;
#pragma unroll
    for (int v = 0; v < 6; ++v)
#pragma unroll
      for (int i = 0; i < 6; ++i) dh[v][i] = 0.0;
#pragma unroll
    for (int p = 0; p < P::deg; ++p) {
      double A[9], YA[9];
      hencky_factor<PD>(p, b.C, C2, b.H, A);
#pragma unroll
      for (int v = 0; v < 6; ++v)
#pragma unroll
        for (int i = 0; i < 6; ++i) dh[v][i] += sandwich(A, N[p], v, BA(i), BB(i));
      // Y : (dH_u dB_v), dB_v = sum_r Bc_r E_v C^r: M_(p+r) += Bc_r Y^T A_p
      mm(Yt, A, YA);
#pragma unroll
      for (int r = 0; r < P::deg; ++r) {
        axpy_c<9>(P::b(r + 1), YA, M[p + r]);
        if (r + 2 <= P::deg) {
          double X[9];
          mm(b.C, YA, X);
          axpy_c<9>(P::b(r + 2), X, M[p + r]);
        }
        if (r + 3 <= P::deg) {
          double X[9];
          mm(C2, YA, X);
          axpy_c<9>(P::b(r + 3), X, M[p + r]);
        }
      }
    }
#pragma unroll
    for (int v = 0; v < 6; ++v)
#pragma unroll
      for (int i = 3; i < 6; ++i) dh[v][i] *= 2.0;
    // Y : (d2A - H d2B) = Zt : (E_u E_v + E_v E_u) + Z3 : (E_u C E_v + E_v C E_u), Z_p = a_p Y - b_p H Y
    double Zt[9], Z3[9];  // transposed
    if constexpr (P::deg >= 2) {
      double YtH[9];
      mm(Yt, b.H, YtH);
#pragma unroll
      for (int i = 0; i < 9; ++i) Zt[i] = P::a(2) * Yt[i] - P::b(2) * YtH[i];
      if constexpr (P::deg >= 3) {
        double ZC[9], CZ[9];
#pragma unroll
        for (int i = 0; i < 9; ++i) Z3[i] = P::a(3) * Yt[i] - P::b(3) * YtH[i];
        mm(Z3, b.C, ZC);
        mm(b.C, Z3, CZ);
#pragma unroll
        for (int i = 0; i < 9; ++i) Zt[i] += ZC[i] + CZ[i];
      }
    }
    phase(dh);
    phase(M);
    double Lm[21];  // mixed stiffness
    PhaseCard& cl = phase(cd);
#pragma unroll
    for (int i = 0; i < 6; ++i)
#pragma unroll
      for (int j = i; j < 6; ++j) {
        double s = cl.L0[i][j];
#pragma unroll
        for (int k = 0; k < NV; ++k) s += eh[k] * cl.dL[k][i][j];
        Lm[eidx(i, j)] = s;
      }
#pragma unroll
    for (int u = 0; u < 6; ++u) {
      double LdH[6];
#pragma unroll
      for (int i = 0; i < 6; ++i) {
        double s = 0.0;
#pragma unroll
        for (int j = 0; j < 6; ++j) s += Lm[eidx(i, j)] * dh[u][j];
        LdH[i] = s;
      }
      phase(LdH);
#pragma unroll
      for (int v = 0; v <= u; ++v) {
        double s = 0.0;
#pragma unroll
        for (int i = 0; i < 6; ++i) s += dh[v][i] * LdH[i];
#pragma unroll
        for (int q = 0; q < NF; ++q) s -= bilinear(M[q], N[q], u, v) + bilinear(M[q], N[q], v, u);
        if constexpr (P::deg >= 2) {  // tr(Z^T (E_u E_v + E_v E_u)): one factor the identity
          const int a = BA(u), bb = BB(u), c = BA(v), d = BB(v);
          auto one = [&](int i, int j, int k2, int l) {  // tr(Zt e_i e_j^T e_k e_l^T)
            if (j == k2) s += Zt[3 * l + i];
          };
          auto prod = [&](int i, int j, int k2, int l, bool ss, bool tt) {
            one(i, j, k2, l);
            if (ss) one(j, i, k2, l);
            if (tt) one(i, j, l, k2);
            if (ss && tt) one(j, i, l, k2);
          };
          prod(a, bb, c, d, u >= 3, v >= 3);
          prod(c, d, a, bb, v >= 3, u >= 3);
        }
        if constexpr (P::deg >= 3) s += bilinear(Z3, b.C, u, v) + bilinear(Z3, b.C, v, u);
        wCC[eidx(v, u)] = s;
      }
    }
  }
  phase(wCC);
  // ---- Green-strain space: D_ee = J_t dC_u : w_CC : dC_v along eps --------------
  {
    double Me[6][6], Dee[21];  // Me[w]: dC along eps_w (2 G E_w G, shear G E_w G)
#pragma unroll
    for (int w = 0; w < 6; ++w)
#pragma unroll
      for (int i = 0; i < 6; ++i) {
        const double m = sandwich(b.G, b.G, w, BA(i), BB(i));
        Me[w][i] = w < 3 ? 2.0 * m : m;
      }
#pragma unroll
    for (int w = 0; w < 6; ++w) {
      double col[6];
#pragma unroll
      for (int u = 0; u < 6; ++u) {
        double s = 0.0;
#pragma unroll
        for (int i = 0; i < 6; ++i) s += wCC[eidx(u, i)] * Me[w][i];
        col[u] = b.Jt * s;
      }
#pragma unroll
      for (int u = 0; u <= w; ++u) {
        double s = 0.0;
#pragma unroll
        for (int i = 0; i < 6; ++i) s += Me[u][i] * col[i];
        Dee[eidx(u, w)] = s;
      }
#pragma unroll
      for (int u = 0; u <= w; ++u) phase(Dee[eidx(u, w)]);
    }
    out.strain(S, Dee);
  }
  // ---- F^t space ---------------------------------------------------------------
  double X[21];     // second derivative along F^t at fixed L, / J_t
  double Te[6][6];  // [v][w]: mixed (F^t_v, eps_w), / J_t
  double gam[6];    // tr(G E_v)
  {
    double Nv[6][6];  // [v]: dC along F^t_v, -(G E_v C + C E_v G)
    double A1[9], P2[9], wC[6], wq[6];
    mm(b.Sf, b.G, A1);
    mm_sym(b.G, A1, P2);
#pragma unroll
    for (int v = 0; v < 6; ++v) {
      const int a = BA(v), c = BB(v);
      gam[v] = v < 3 ? b.G[3 * a + c] : 2.0 * b.G[3 * a + c];
      wC[v] = v < 3 ? b.Sf[3 * a + c] : 2.0 * b.Sf[3 * a + c];
      wq[v] = v < 3 ? -2.0 * b.B1[3 * a + c] : -2.0 * (b.B1[3 * a + c] + b.B1[3 * c + a]);
#pragma unroll
      for (int i = 0; i < 6; ++i)
        Nv[v][i] = -(sandwich(b.G, b.C, v, BA(i), BB(i)) + sandwich(b.C, b.G, v, BA(i), BB(i)));
    }
    phase(Nv);
#pragma unroll
    for (int v = 0; v < 6; ++v) {
      double wN[6];
#pragma unroll
      for (int u = 0; u < 6; ++u) {
        double s = 0.0;
#pragma unroll
        for (int i = 0; i < 6; ++i) s += wCC[eidx(u, i)] * Nv[v][i];
        wN[u] = s;
      }
#pragma unroll
      for (int u = 0; u <= v; ++u) {
        double s = 0.0;
#pragma unroll
        for (int i = 0; i < 6; ++i) s += Nv[u][i] * wN[i];
        s += 2.0 * (bilinear(b.B1, b.G, u, v) + bilinear(b.B1, b.G, v, u) + bilinear(P2, b.C, u, v));
        s += gam[u] * wq[v] + gam[v] * wq[u] + (gam[u] * gam[v] - bilinear(b.G, b.G, u, v)) * b.w;
        X[eidx(u, v)] = s;
      }
      // w_CC dC_v - 2 (Sf G E_v) : E_u + tr(G E_v) w_C
#pragma unroll
      for (int u = 0; u < 6; ++u) {
        const int a = BA(u), c = BB(u), p = BA(v), q = BB(v);
        double t = 0.0;  // (A1 E_v)_ij = A1_ip [j == q] (+ A1_iq [j == p])
        if (c == q) t += A1[3 * a + p];
        if (v >= 3 && c == p) t += A1[3 * a + q];
        if (u >= 3) {
          if (a == q) t += A1[3 * c + p];
          if (v >= 3 && a == p) t += A1[3 * c + q];
        }
        wN[u] += gam[v] * wC[u] - 2.0 * t;
      }
      to_strain(b.G, wN, Te[v]);
      phase(Te[v]);
#pragma unroll
      for (int u = 0; u <= v; ++u) phase(X[eidx(u, v)]);
    }
  }
  // ---- order parameters ----------------------------------------------------
  const double eta0 = [&] {
    double s = 0.0;
#pragma unroll
    for (int k = 0; k < NV; ++k) s += eh[k];
    return 1.0 - s;
  }();
  const double pen0 = (eta0 < 0.0) ? cd.eps : 0.0;
  double Y[NV][6];  // mixed (F^t_v, L through eta_k), / J_t
#pragma unroll
  for (int k = 0; k < NV; ++k) {
    double wCe[6], d[6], z[6];  // wCe: mixed (C along E_v, L through eta_k)
    PhaseCard& ck = phase(cd);
    {
      double dLh[6];
      voigt_product(ck.dL[k], b.h, dLh);
#pragma unroll
      for (int v = 0; v < 6; ++v) {
        double s = 0.0;
#pragma unroll
        for (int i = 0; i < 6; ++i) s += dLh[i] * dh[v][i];
        wCe[v] = s;
      }
    }
    to_strain(b.G, wCe, d);
#pragma unroll
    for (int w = 0; w < 6; ++w) {
      double s = d[w];
#pragma unroll
      for (int v = 0; v < 6; ++v) s += Te[v][w] * dm(ck, k, v);
      d[w] = b.Jt * s;
    }
    out.eps_eta(k, d);
    {  // sum_i (dC along F^t_v)_i wCe_i = -2 sym(G q C) : E_v
      const double Q[9] = {wCe[0], 0.5 * wCe[5], 0.5 * wCe[4], 0.5 * wCe[5], wCe[1],
                           0.5 * wCe[3], 0.5 * wCe[4], 0.5 * wCe[3], wCe[2]};
      double GQ[9], R[9];
      mm(b.G, Q, GQ);
      mm(GQ, b.C, R);
#pragma unroll
      for (int v = 0; v < 6; ++v) {
        const int i = BA(v), j = BB(v);
        Y[k][v] = b.wEta[k] * gam[v] - 2.0 * (v < 3 ? R[3 * i + j] : R[3 * i + j] + R[3 * j + i]);
      }
    }
#pragma unroll
    for (int v = 0; v < 6; ++v) {
      double s = Y[k][v];
#pragma unroll
      for (int i = 0; i < 6; ++i) s += X[eidx(v, i)] * dm(ck, k, i);
      z[v] = s;
    }
#pragma unroll
    for (int l = 0; l <= k; ++l) {
      double s = 0.0;
#pragma unroll
      for (int v = 0; v < 6; ++v) s += dm(ck, l, v) * z[v] + dm(ck, k, v) * Y[l][v];
      double val = b.Jt * s;
      if constexpr (MIX == 1) {  // second derivative of F^t
        double S2[9], S2s[6];
        log_mixing_second(eh, cd, k, l, S2);
        sym_of(S2, S2s);
#pragma unroll
        for (int v = 0; v < 6; ++v) val += phi[v] * S2s[v];
      }
      val += ck.Sw[k][l] + ck.rho * ((k == l ? 1.0 : 0.0) + 1.0) + pen0;
      if (k == l && eh[k] < 0.0) val += ck.eps;
      out.eta_eta(k, l, val);
    }
    phase(Y[k]);
  }
}

// Packed upper triangle of the Hessian in (F, eta), entry hidx(p, q) stored to
// D[hidx(p, q) * ds + off]: D and ds uniform over the wavefront and a 32-bit
// lane offset, so that the 120 addresses are scalar.
struct PackedOut {
  const double* F;
  double* D;
  int64_t ds;
  uint32_t off;
  __device__ __forceinline__ void eps_eta(int k, const double d[6]) const {
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
      for (int j = 0; j < 3; ++j)
        (D + hidx(3 * i + j, 9 + k) * ds)[off] =
            F[3 * i] * d[SI(0, j)] + F[3 * i + 1] * d[SI(1, j)] + F[3 * i + 2] * d[SI(2, j)];
  }
  __device__ __forceinline__ void eta_eta(int k, int l, double v) const { (D + hidx(9 + l, 9 + k) * ds)[off] = v; }
  // F-F block from D_ee and the stress
  __device__ __forceinline__ void strain(const double S[6], const double Dee[21]) const {
#pragma unroll
    for (int k = 0; k < 3; ++k)
#pragma unroll
      for (int l = 0; l < 3; ++l) {
        double t[6];
#pragma unroll
        for (int u = 0; u < 6; ++u)
          t[u] = Dee[eidx(u, SI(0, l))] * F[3 * k] + Dee[eidx(u, SI(1, l))] * F[3 * k + 1] +
                 Dee[eidx(u, SI(2, l))] * F[3 * k + 2];
#pragma unroll
        for (int i = 0; i <= k; ++i)
#pragma unroll
          for (int j = 0; j < 3; ++j) {
            if (3 * i + j > 3 * k + l) continue;
            double s = F[3 * i] * t[SI(0, j)] + F[3 * i + 1] * t[SI(1, j)] + F[3 * i + 2] * t[SI(2, j)];
            if (i == k) s += S[SI(j, l)];
            (D + hidx(3 * i + j, 3 * k + l) * ds)[off] = s;
          }
      }
  }
};

}  // namespace mvpf
