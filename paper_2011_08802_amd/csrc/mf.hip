// Matrix-free application of the finest-level tangent from its Gauss-point
// Hessians (Sec. 3.4: K = d^2 Pi / dU^2, here never assembled on the finest
// level).  With v_g = B_g x_e the 15 local variables of Gauss point g
// (reference-cube gradients of u, h * eta) and D_g the 15 x 15 Hessian of the
// density,
//   (K x)_a = h/8 sum_g B_{g,a}^T D_g v_g  +  the gradient-energy term
//             h/8 sum_g dN_a . (Mg (x) I) grad_ref eta,
// which is the element matrix of the assembled path applied to x_e (same
// 2x2x2 rule; the Laplacian term is exact under it).
//
// D_g is stored in Green-strain form, 93 values padded to 96 (the density
// depends on F through F^T F only): D v costs the same number of operations as
// with the 120 packed entries of D_g, and the product is bound by streaming
// them.  64^3, FP32: 188 -> 156 us per product (0.81 GB, 5.2 TB/s); 128x128x64:
// FP32 750 -> 611 us, FP64 1513 -> 1212 us (5.3 TB/s).
// eps and sigma are intermediate results that a product with the packed entries
// does not round, so the sums of D v are taken in 64 bits for either storage
// type.  Error of the FP32 product against 64 bits at 64^3: 6.1e-8 with the packed
// entries, 6.4e-8 in this form with 32-bit sums, 5.7e-8 so; evaluated on the CPU,
// also where one kind of unknown dominates the input (32-bit sums of the parts
// that hold the other kind exceed the packed entries' error there by 1 %).  The
// 108 conversions per lane cost the FP32 sweep 2 % (41^3 nodes 53.3 -> 54.4 us).
// Stored per element: 3 KB in FP32 instead of the half-stencil blocks of its
// node (4.7 KB) plus the assembled path's transposed contributions (0.9 KB
// written and read per sweep).
//
// Kernel layout: a wavefront covers 8 elements x 8 Gauss points (lane =
// 8 * element + j).  Lane j loads the 9 unknowns of corner j of its element
// and evaluates Gauss point j: since the Q1 shape functions and the 2x2x2
// points are tensor products, v_g follows from three one-dimensional
// interpolation stages over lane pairs (sum factorisation; lanes exchange
// values by DPP moves, xor 1, 2, 4), and the contributions B^T [w; z] go
// back to the corners through the transposed stages, so that lane j ends
// with the element's part for corner j.  The workgroup merges the parts of
// neighbouring elements along x that meet at a node and writes them to the
// element-output buffer (layout in common.h); a node gather sums its <= 4
// merged element rows in a fixed order and applies the epilogue (product,
// defect or damped point-block Jacobi update), so results are reproducible
// bit for bit.
//
// The lane layout (9 unknowns per corner, 15 local variables, 96 tangent
// values streamed as 24 16-byte vectors) is that of the six-variant card:
// a library built for another number of variants never enables the
// matrix-free level (its finest level is assembled like the others) and
// launches none of these kernels.
#include "pair.h"

namespace mvpf {

// elements per workgroup of the element kernels: 8, 16 or 32
constexpr int MF_MAX_EPW = 32;

// gradient-energy coefficient Mg[m][m2] in the arithmetic type
template <typename T>
__device__ __forceinline__ T mg_coef(const DevCard* __restrict__ cd, int m, int m2) {
  if constexpr (sizeof(T) == 4) return cd->Mg32[m][m2];
  else return cd->Mg[m][m2];
}

// E = element parts of K x_e (x masked on constrained dofs when mask != null).
// Lane = 8 * element + j: the lane loads the unknowns of corner j of its
// element and evaluates Gauss point j; the 15 local variables of every
// point come from three interpolation stages over lane pairs (x, y, z), and
// its contributions go back to the corners through the transposed stages
// (z, y, x), so that lane j ends with the element's part for corner j.
// SPARSE: x has few nonzero entries (the lifting of a prescribed increment):
// an element whose unknowns are all zero reads no Hessians; otherwise the
// Hessian loads are issued before the unknowns arrive.
// PF: Hessian vectors loaded ahead of the contraction (the rest are loaded
// PF vectors ahead of their use); MINB: minimum waves per SIMD the register
// budget is sized for.
template <typename TD, typename TX, typename T, int PF, bool SPARSE>
__device__ __forceinline__ void mf_element_body(const Grid& g, const TD* __restrict__ D, const TX* __restrict__ x,
                                                const uint16_t* __restrict__ mask, const DevCard* __restrict__ cd,
                                                T* __restrict__ E, int wg, int nb) {
  // workgroups are dealt to the 8 XCDs in turn: renumber them so that each
  // XCD takes one contiguous range of elements (corner unknowns shared by
  // neighbouring elements then hit that XCD's L2)
  const int xcd = wg & 7;
  const int bid = xcd * (nb >> 3) + min(xcd, nb & 7) + (wg >> 3);
  const int64_t t = (int64_t)bid * blockDim.x + threadIdx.x;
  const int lane = threadIdx.x & 63;
  const int gp = lane & 7;
  const int64_t e = (t >> 6) * 8 + (lane >> 3);
  const bool active = e < g.NE;  // inactive lanes hold zeros and still take part in the exchanges
  const bool b0 = gp & 1, b1 = (gp >> 1) & 1, b2 = (gp >> 2) & 1;
  // weight of the partner in the interpolation, of the own and the partner's
  // part in the transposed stages (the points sit symmetrically: the same for
  // both sides), and the sign of the derivative per direction
  const T one = (T)1, lo = (T)MGQ0, hi = (T)MGQ1;
  const T sg0 = b0 ? -one : one, sg1 = b1 ? -one : one, sg2 = b2 ? -one : one;
  const T h = (T)g.h, c1 = (T)(0.125 * g.h);
  // the unknowns of corner gp
  T xa[9];
#pragma unroll
  for (int c = 0; c < 9; ++c) xa[c] = 0;
  int node = 0;
  if (active) {
    const int ex = (int)(e % g.nx), ey = (int)((e / g.nx) % g.ny), ez = (int)(e / ((int64_t)g.nx * g.ny));
    node = (ex + b0) + g.nnx * ((ey + b1) + g.nny * (ez + b2));
    const unsigned mb = mask ? mask[node] : 0u;
    TX xl[9];
#pragma unroll
    for (int c = 0; c < 9; ++c) xl[c] = x[(int64_t)c * g.Npad + node];
#pragma unroll
    for (int c = 0; c < 9; ++c) xa[c] = ((mb >> c) & 1) ? (T)0 : (T)xl[c];
  }
  // tangent of Gauss point gp in Green-strain form (MF_G ... of common.h),
  // 16-byte non-temporal loads (streamed once per product: x and the element
  // outputs stay in the caches)
  constexpr int V = 16 / (int)sizeof(TD);
  constexpr int NV = MF_NK / V;
  typedef TD VT __attribute__((ext_vector_type(V)));
  const VT* Dp = reinterpret_cast<const VT*>(D) + ((e >> 3) * NV * 64 + gp * 8 + (e & 7));
  constexpr int64_t ks = 64;
  VT dq[NV];
  if (!SPARSE && active) {
#pragma unroll
    for (int k = 0; k < PF; ++k) dq[k] = __builtin_nontemporal_load(Dp + k * ks);
  }
  // interpolation to Gauss point gp: x, then y, then z
  T s1[9], d1[9];
  interp_pair<1>(xa, lo, sg0, s1, d1);
  T sd1[18], s2[18], d2[9];
#pragma unroll
  for (int c = 0; c < 9; ++c) sd1[c] = s1[c], sd1[9 + c] = d1[c];
  interp_pair<2>(sd1, lo, sg1, s2, d2);  // s2 = (value, d/dx) at (q0, q1); d2 = d/dy
  T sd2[27], s3[27], d3[9];
#pragma unroll
  for (int c = 0; c < 18; ++c) sd2[c] = s2[c];
#pragma unroll
  for (int c = 0; c < 9; ++c) sd2[18 + c] = d2[c];
  interp_pair<4>(sd2, lo, sg2, s3, d3);  // s3 = (value, d/dx, d/dy); d3 = d/dz
  // v: reference gradients of u (3 x 3), h * eta (6); ge: reference gradients of eta
  T v[15], ge[18];
#pragma unroll
  for (int c = 0; c < 3; ++c) v[3 * c] = s3[9 + c], v[3 * c + 1] = s3[18 + c], v[3 * c + 2] = d3[c];
#pragma unroll
  for (int m = 0; m < 6; ++m) {
    v[9 + m] = h * s3[3 + m];
    ge[3 * m] = s3[12 + m], ge[3 * m + 1] = s3[21 + m], ge[3 * m + 2] = d3[3 + m];
  }
  // w = D v: with F = I + G, eps = sym(F^T dF) (engineering shears),
  // sigma = D_ee eps + D_ek eta, t = D_ek^T eps + D_kk eta, and back through
  // dF: F sigma + dF S.  All sums in 64 bits (see the head of the file); G and
  // S wait in the storage type for their use at the end.
  T w[15];
#pragma unroll
  for (int k = 0; k < 15; ++k) w[k] = 0;
  bool load = active;
  if (SPARSE) {  // the element is zero iff the unknowns of its 8 corners (lanes) are
    bool nz = false;
#pragma unroll
    for (int c = 0; c < 9; ++c) nz = nz || xa[c] != (T)0;
    const unsigned long long bal = __ballot(nz);
    load = active && ((bal >> (lane & ~7)) & 0xFFull) != 0;
    if (load) {
#pragma unroll
      for (int k = 0; k < NV; ++k) dq[k] = __builtin_nontemporal_load(Dp + k * ks);
    }
  }
  if (load) {
    // entry k of the stream (each taken once, in order): its vector's first
    // entry issues the load PF vectors ahead
    auto entry = [&](int k) -> TD {
      if (!SPARSE && k % V == 0 && k / V + PF < NV) dq[k / V + PF] = __builtin_nontemporal_load(Dp + (k / V + PF) * ks);
      return dq[k / V][k % V];
    };
    TD G[9], S[6];
    double eps[6], sig[6], t[6];
#pragma unroll
    for (int k = 0; k < 9; ++k) G[k] = entry(MF_G + k);
#pragma unroll
    for (int u = 0; u < 6; ++u) {
      const int j = BA(u), l = BB(u);
      double s = j == l ? (double)v[4 * j] : (double)v[3 * j + l] + (double)v[3 * l + j];
#pragma unroll
      for (int i = 0; i < 3; ++i) {
        s += (double)G[3 * i + j] * (double)v[3 * i + l];
        if (j != l) s += (double)G[3 * i + l] * (double)v[3 * i + j];
      }
      eps[u] = s;
      sig[u] = t[u] = 0;
    }
#pragma unroll
    for (int u = 0; u < 6; ++u) S[u] = entry(MF_S + u);
#pragma unroll
    for (int p = 0, k = MF_EE; p < 6; ++p)
#pragma unroll
      for (int q = p; q < 6; ++q, ++k) {
        const double d = entry(k);
        sig[p] += d * eps[q];
        if (q != p) sig[q] += d * eps[p];
      }
#pragma unroll
    for (int m = 0; m < 6; ++m)
#pragma unroll
      for (int u = 0; u < 6; ++u) {
        const double d = entry(MF_EK + 6 * m + u);
        sig[u] += d * (double)v[9 + m];
        t[m] += d * eps[u];
      }
#pragma unroll
    for (int m = 0, k = MF_KK; m < 6; ++m)
#pragma unroll
      for (int l = 0; l <= m; ++l, ++k) {
        const double d = entry(k);
        t[m] += d * (double)v[9 + l];
        if (l != m) t[l] += d * (double)v[9 + m];
      }
#pragma unroll
    for (int m = 0; m < 6; ++m) w[9 + m] = (T)t[m];
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
      for (int j = 0; j < 3; ++j) {
        double s = sig[SI(i, j)];
#pragma unroll
        for (int l = 0; l < 3; ++l)
          s += (double)G[3 * i + l] * sig[SI(l, j)] + (double)S[SI(l, j)] * (double)v[3 * i + l];
        w[3 * i + j] = (T)s;
      }
  }
  // gradient energy: z = (Mg (x) I) grad_ref eta
  T z[18];
#pragma unroll
  for (int m = 0; m < 6; ++m)
#pragma unroll
    for (int j = 0; j < 3; ++j) {
      T sum = 0;
#pragma unroll
      for (int m2 = 0; m2 < 6; ++m2) sum += mg_coef<T>(cd, m, m2) * ge[3 * m2 + j];
      z[3 * m + j] = sum;
    }
  // coefficients of point gp: a = of the shape-function values, (bx, by, bz)
  // = of their reference derivatives, per component, each derivative
  // coefficient carrying the transposed stage's sign of its direction (the
  // x and y coefficients keep it through the z and y stages, whose lane
  // partners share the lane's x and y bits)
  const T cx = b0 ? c1 : -c1, cy = b1 ? c1 : -c1, cz = b2 ? c1 : -c1;
  T a3[27], bz[27];
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    a3[c] = 0, a3[9 + c] = cx * w[3 * c], a3[18 + c] = cy * w[3 * c + 1];
    bz[c] = cz * w[3 * c + 2];
  }
#pragma unroll
  for (int m = 0; m < 6; ++m) {
    a3[3 + m] = c1 * h * w[9 + m], a3[12 + m] = cx * z[3 * m], a3[21 + m] = cy * z[3 * m + 1];
    bz[3 + m] = cz * z[3 * m + 2];
  }
#pragma unroll
  for (int c = 0; c < 9; ++c) bz[9 + c] = 0, bz[18 + c] = 0;
  // back to the corners: z (27 sums: value, x, y coefficients), then y, then x
  T r3[27];
  interp_pair_t<4>(a3, bz, hi, lo, r3);
  T a2[18], by[18], r2[18];
#pragma unroll
  for (int c = 0; c < 18; ++c) a2[c] = r3[c], by[c] = 0;
#pragma unroll
  for (int c = 0; c < 9; ++c) by[c] = r3[18 + c];
  interp_pair_t<2>(a2, by, hi, lo, r2);
  T a1[9], bx[9], out[9];
#pragma unroll
  for (int c = 0; c < 9; ++c) a1[c] = r2[c], bx[c] = r2[9 + c];
  interp_pair_t<1>(a1, bx, hi, lo, out);
  __shared__ T eo[72 * (MF_MAX_EPW + 1)];
  store_corners<T, 9>(eo, out, gp, threadIdx.x >> 3, blockDim.x >> 3, bid, g.nx, g.NE, E, g.NEpad, mf_nw(g), mf_nr(g));
}
template <typename TD, typename TX, typename T, int MINB, int PF, bool SPARSE>
__global__ void __launch_bounds__(256, MINB) mf_element_kernel(Grid g, const TD* __restrict__ D, const TX* __restrict__ x,
                                                               const uint16_t* __restrict__ mask,
                                                               const DevCard* __restrict__ cd, T* __restrict__ E) {
  mf_element_body<TD, TX, T, PF, SPARSE>(g, D, x, mask, cd, E, blockIdx.x, gridDim.x);
}

// Node gather with epilogue.  MODE 0: y = K x; 1: r = b - K x;
// 2: xo = x + omega Dinv (b - K x), Dinv packed symmetric (LaySym) in FP32,
// full (Lay) in FP64.  Constrained rows (mask) act as the identity, as in the
// eliminated assembled operator.  E: the element outputs of a launch with
// epw elements per workgroup; Cf: the contact face outputs, or null.
template <int MODE, typename T, typename TX, typename TY>
__device__ __forceinline__ void mf_gather_body(const Grid& g, const T* __restrict__ E, const T* __restrict__ Cf,
                                               int epw, const uint16_t* __restrict__ mask,
                                               const TX* __restrict__ x, const T* __restrict__ b,
                                               const T* __restrict__ Dinv, T omega, TY* __restrict__ y, int bid) {
  const int n = bid * 256 + threadIdx.x;
  if (n >= g.Npad) return;
  if (n >= g.N) {
#pragma unroll
    for (int c = 0; c < 9; ++c) y[(int64_t)c * g.Npad + n] = (TY)0;
    return;
  }
  const int i = n % g.nnx, j = (n / g.nnx) % g.nny, k = n / (g.nnx * g.nny);
  T s[9] = {0, 0, 0, 0, 0, 0, 0, 0, 0};
  const T* __restrict__ W = E + mf_w_offset(g);
  const T* __restrict__ Rr = E + mf_r_offset(g);
#pragma unroll
  for (int q = 3; q >= 0; --q) {  // element row r = (j - by) + ny (k - bz) holds this node at (by, bz)
    const int ey = j - (q & 1), ez = k - (q >> 1);
    if (ey < 0 || ey >= g.ny || ez < 0 || ez >= g.nz) continue;
    const int64_t r = ey + (int64_t)g.ny * ez;
    T t[9];
    if (i < g.nx) {
      const int64_t e = i + g.nx * r;
#pragma unroll
      for (int c = 0; c < 9; ++c) t[c] = E[(int64_t)(9 * q + c) * g.NEpad + e];
      if (i > 0 && (e & (epw - 1)) == 0) {  // element e - 1 ended the previous workgroup
        const int64_t w = e / epw - 1;
#pragma unroll
        for (int c = 0; c < 9; ++c) t[c] = t[c] + W[(int64_t)(9 * q + c) * mf_nw(g) + w];
      }
    } else {
#pragma unroll
      for (int c = 0; c < 9; ++c) t[c] = Rr[(int64_t)(9 * q + c) * mf_nr(g) + r];
    }
#pragma unroll
    for (int c = 0; c < 9; ++c) s[c] += t[c];
  }
  if (Cf && k == g.nz) {  // penalty contact: the top faces around the node
    const int64_t nf = mf_nf(g);
#pragma unroll
    for (int a = 3; a >= 0; --a) {
      const int fi = i - (a & 1), fj = j - (a >> 1);
      if (fi < 0 || fi >= g.nx || fj < 0 || fj >= g.ny) continue;
      const int64_t f = fi + (int64_t)g.nx * fj;
#pragma unroll
      for (int c = 0; c < 3; ++c) s[c] += Cf[(3 * a + c) * nf + f];
    }
  }
  const unsigned mb = mask ? mask[n] : 0u;
  T r[9];
#pragma unroll
  for (int c = 0; c < 9; ++c) {
    const T xv = (T)x[(int64_t)c * g.Npad + n];
    const T kx = ((mb >> c) & 1) ? xv : s[c];
    r[c] = (MODE == 0) ? kx : b[(int64_t)c * g.Npad + n] - kx;
  }
  if (MODE == 2 && sizeof(T) == 4) {  // FP32: the packed upper triangles of the symmetric block inverses
    const int t = n >> 6, l = n & 63;
    const T* Db = Dinv + (int64_t)t * LaySym<T>::SLICE;
    T dv[NSYM];
#pragma unroll
    for (int e = 0; e < NSYM; ++e) dv[e] = Db[LaySym<T>::off(e, l)];
#pragma unroll
    for (int rr = 0; rr < 9; ++rr) {
      T acc = 0;
#pragma unroll
      for (int c = 0; c < 9; ++c) acc += dv[sym_index(rr, c)] * r[c];
      y[(int64_t)rr * g.Npad + n] = (TY)((T)x[(int64_t)rr * g.Npad + n] + omega * acc);
    }
  } else if (MODE == 2) {
    const int t = n >> 6, l = n & 63;
    const T* Db = Dinv + (int64_t)t * Lay<T>::SLICE;
#pragma unroll
    for (int rr = 0; rr < 9; ++rr) {
      T acc = 0;
#pragma unroll
      for (int c = 0; c < 9; ++c) acc += Db[Lay<T>::off(rr * 9 + c, l)] * r[c];
      y[(int64_t)rr * g.Npad + n] = (TY)((T)x[(int64_t)rr * g.Npad + n] + omega * acc);
    }
  } else {
#pragma unroll
    for (int c = 0; c < 9; ++c) y[(int64_t)c * g.Npad + n] = (TY)r[c];
  }
}
template <int MODE, typename T, typename TX, typename TY>
__global__ void __launch_bounds__(256) mf_gather_kernel(Grid g, const T* __restrict__ E, const T* __restrict__ Cf,
                                                        int epw, const uint16_t* __restrict__ mask,
                                                        const TX* __restrict__ x, const T* __restrict__ b,
                                                        const T* __restrict__ Dinv, T omega, TY* __restrict__ y) {
  mf_gather_body<MODE, T, TX, TY>(g, E, Cf, epw, mask, x, b, Dinv, omega, y, blockIdx.x);
}

// The same for small grids, where a thread per node leaves most of the chip
// idle and walks its loads in turn: a workgroup takes a tile of 64 nodes, one
// wavefront per component, with the tile's block inverses staged in LDS while
// the element outputs arrive.  Sums and rounding as above.
constexpr int GT = 9 * TILE;
template <int MODE, typename T, typename TX, typename TY>
__global__ void __launch_bounds__(GT) mf_gather_tile_kernel(Grid g, const T* __restrict__ E, const T* __restrict__ Cf,
                                                            int epw, const uint16_t* __restrict__ mask,
                                                            const TX* __restrict__ x, const T* __restrict__ b,
                                                            const T* __restrict__ Dinv, T omega, TY* __restrict__ y) {
  using LD = std::conditional_t<sizeof(T) == 4, LaySym<T>, Lay<T>>;
  using VT = typename Vec16<T>::type;
  constexpr int ND = MODE == 2 && MF_AVAILABLE ? LD::NE / LD::V * TILE : 1, ROUNDS = (ND + GT - 1) / GT;
  __shared__ VT sd[ND];
  __shared__ T sr[9][TILE];
  const int t = blockIdx.x, l = threadIdx.x & 63, c = threadIdx.x >> 6;
  const int n = t * TILE + l;
  VT dv[ROUNDS];
  if constexpr (MODE == 2) {
    const VT* Db = reinterpret_cast<const VT*>(Dinv + (int64_t)t * LD::SLICE);
#pragma unroll
    for (int u = 0; u < ROUNDS; ++u) {
      const int i = u * GT + threadIdx.x;
      if (i < ND) dv[u] = Db[i];
    }
  }
  const T* __restrict__ W = E + mf_w_offset(g);
  const T* __restrict__ Rr = E + mf_r_offset(g);
  T xv = 0, r = 0;
  if (n < g.N) {
    xv = (T)x[(int64_t)c * g.Npad + n];
    const T bv = MODE == 0 ? (T)0 : b[(int64_t)c * g.Npad + n];
    const unsigned mb = mask ? mask[n] : 0u;
    const int i = n % g.nnx, j = (n / g.nnx) % g.nny, k = n / (g.nnx * g.nny);
    T a[4], w[4];
    bool in[4];
#pragma unroll
    for (int q = 3; q >= 0; --q) {
      const int ey = j - (q & 1), ez = k - (q >> 1);
      in[q] = ey >= 0 && ey < g.ny && ez >= 0 && ez < g.nz;
      const int64_t row = in[q] ? ey + (int64_t)g.ny * ez : 0;
      const int64_t e = i + g.nx * row;
      a[q] = *(i < g.nx ? E + (int64_t)(9 * q + c) * g.NEpad + e : Rr + (int64_t)(9 * q + c) * mf_nr(g) + row);
      w[q] = 0;
      if (i > 0 && i < g.nx && (e & (epw - 1)) == 0) w[q] = W[(int64_t)(9 * q + c) * mf_nw(g) + e / epw - 1];
    }
    T s = 0;
#pragma unroll
    for (int q = 3; q >= 0; --q)
      if (in[q]) s += a[q] + w[q];
    if (Cf && c < 3 && k == g.nz) {
      const int64_t nf = mf_nf(g);
#pragma unroll
      for (int q = 3; q >= 0; --q) {
        const int fi = i - (q & 1), fj = j - (q >> 1);
        if (fi < 0 || fi >= g.nx || fj < 0 || fj >= g.ny) continue;
        s += Cf[(3 * q + c) * nf + fi + (int64_t)g.nx * fj];
      }
    }
    const T kx = ((mb >> c) & 1) ? xv : s;
    r = (MODE == 0) ? kx : bv - kx;
  }
  if constexpr (MODE == 2) {
    sr[c][l] = r;
#pragma unroll
    for (int u = 0; u < ROUNDS; ++u) {
      const int i = u * GT + threadIdx.x;
      if (i < ND) sd[i] = dv[u];
    }
    __syncthreads();
    const T* D = reinterpret_cast<const T*>(sd);
    T acc = 0;
#pragma unroll
    for (int d = 0; d < 9; ++d) {
      int o;
      if constexpr (sizeof(T) == 4)
        o = (int)LD::off(c <= d ? c * NDOF - c * (c - 1) / 2 + (d - c) : d * NDOF - d * (d - 1) / 2 + (c - d), l);
      else
        o = (int)LD::off(9 * c + d, l);
      acc += D[o] * sr[d][l];
    }
    r = n < g.N ? xv + omega * acc : (T)0;
  }
  y[(int64_t)c * g.Npad + n] = (TY)r;
}

size_t mf_hessian_values(const Grid& g) { return MF_AVAILABLE ? (size_t)MF_NK * 8 * g.NEpad : 0; }

// ---- diagonal blocks from the Gauss-point tangents ----------------------------
// One direction of a diagonal block's quadrature by lane pairs: a lane holds a
// coefficient at its Gauss point and ends with both points' sum for its own
// corner, weighted by phi^2 (VV), phi phi' (VD) or phi'^2 = 1 (DD).
enum PairType { PAIR_VV, PAIR_VD, PAIR_DD };
struct PairWeights {
  double mv, tv, md, td;  // own and partner's weight of VV, of VD
};
__device__ __forceinline__ PairWeights pair_weights(bool b) {
  const double mq = MGQ1, tq = MGQ0;  // a corner's shape value at the nearer and the farther point
  const double sg = b ? 1.0 : -1.0;
  return PairWeights{mq * mq, tq * tq, mq * sg, -tq * sg};
}
template <int X, int TYPE>
__device__ __forceinline__ double pair_sum(double a, const PairWeights& w) {
  if constexpr (TYPE == PAIR_VV) return a * w.mv + lane_xor<X>(a * w.tv);
  else if constexpr (TYPE == PAIR_VD) return a * w.md + lane_xor<X>(a * w.td);
  else return a + lane_xor<X>(a);
}

// Merged element parts of the 9x9 diagonal blocks (45 symmetric entries per
// corner), straight from the FP64 Gauss-point tangents: lane = 8 * element +
// Gauss point as in the element product.  Every coefficient of B^T D B on the
// diagonal is a product of one-dimensional weights, so the eight points are
// summed by three pair exchanges per coefficient (297 in all) instead of one
// 9x9 product per corner and point.  Elements of one slab (whole layers),
// chunk-local index el; streams as for the element outputs, 45 values instead
// of 9, each group of nine stored as soon as it is complete.  Bound: the
// tangents' 0.77 KB per point, read once (64^3: 1.6 GB), at the 3 wavefronts
// per SIMD that 168 registers allow: 698 -> 442 us against one wavefront with
// all 45 results live.
constexpr int DG_EPW = SLAB_EPW;
constexpr int DG_ENTRIES = 45;
// position of entry (r, c) of the symmetric block among the 45: u-u, then u-eta by
// eta component, then eta-eta
__host__ __device__ constexpr int diag_stream(int r, int c) {
  if (r > c) { const int x = r; r = c; c = x; }
  return c < 3 ? c * (c + 1) / 2 + r : r < 3 ? 6 + 3 * (c - 3) + r : 24 + (c - 3) * (c - 2) / 2 + r - 3;
}

__device__ __forceinline__ void mf_diag_body(const Grid& g, const Chunk& ck, const double* __restrict__ D,
                                             const DevCard* __restrict__ cd, double* __restrict__ E, int wg, int nb) {
  __shared__ double eo[72 * (DG_EPW + 1)];
  const int xcd = wg & 7;
  const int bid = xcd * (nb >> 3) + min(xcd, nb & 7) + (wg >> 3);
  const int lane = threadIdx.x & 63, gp = lane & 7, jw = threadIdx.x >> 3;
  const int el = bid * DG_EPW + jw;
  const bool active = el < ck.NEc;
  const int64_t e = ck.e0 + (active ? el : 0);
  const double2* Dp = reinterpret_cast<const double2*>(D) + ((e >> 3) * (MF_NK / 2) * 64 + gp * 8 + (e & 7));
  const PairWeights wx = pair_weights(gp & 1), wy = pair_weights((gp >> 1) & 1), wz = pair_weights((gp >> 2) & 1);
  const double h = g.h, cuu = 0.125 * h, cue = 0.125 * h * h, cee = 0.125 * h * h * h;
  // entry `next` (order of diag_stream), nine to a stream group: a full group
  // leaves at once, so that nine results, not 45, are live
  double part[9];
  int next = 0;
  auto emit = [&](double v) {
    part[next % 9] = v;
    if (++next % 9) return;
    const int r = next / 9 - 1;
    if (r > 0) __syncthreads();
    store_corners<double, 9>(eo, part, gp, jw, DG_EPW, bid, g.nx, ck.NEc, E + r * slab_values(ck, g.nx, 9), ck.NEcpad,
                             slab_nw(ck), ck.NEc / g.nx);
  };
  double F[9];
  {
    double2 v[(MF_EK) / 2];
#pragma unroll
    for (int k = 0; k < MF_EK / 2; ++k) v[k] = Dp[k * 64];
    auto at = [&](int k) { return (k & 1) ? v[k >> 1].y : v[k >> 1].x; };
#pragma unroll
    for (int i = 0; i < 9; ++i) F[i] = at(MF_G + i) + (i % 4 == 0 ? 1.0 : 0.0);
    // u-u: D(ij, kl) = sum_ab F_ia F_kb D_(aj)(bl) + delta_ik S_jl, weights dN_j dN_l
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      double t[6][3];  // [aj][l]: sum_b D_(aj)(bl) F_kb
#pragma unroll
      for (int u = 0; u < 6; ++u)
#pragma unroll
        for (int l = 0; l < 3; ++l)
          t[u][l] = at(MF_EE + eidx(u, SI(0, l))) * F[3 * k] + at(MF_EE + eidx(u, SI(1, l))) * F[3 * k + 1] +
                    at(MF_EE + eidx(u, SI(2, l))) * F[3 * k + 2];
#pragma unroll
      for (int i = 0; i <= k; ++i) {
        double d[6];  // coefficients of dN_j dN_l, j <= l (xx, yy, zz, yz, xz, xy)
#pragma unroll
        for (int u = 0; u < 6; ++u) {
          const int j = BA(u), l = BB(u);
          double s = F[3 * i] * t[SI(0, j)][l] + F[3 * i + 1] * t[SI(1, j)][l] + F[3 * i + 2] * t[SI(2, j)][l];
          if (j != l)
            s += F[3 * i] * t[SI(0, l)][j] + F[3 * i + 1] * t[SI(1, l)][j] + F[3 * i + 2] * t[SI(2, l)][j];
          if (i == k) s += (j != l ? 2.0 : 1.0) * at(MF_S + u);
          d[u] = cuu * s;
        }
        // z, y, x
        const double xx = pair_sum<2, PAIR_VV>(pair_sum<4, PAIR_VV>(d[0], wz), wy);
        const double yy = pair_sum<2, PAIR_DD>(pair_sum<4, PAIR_VV>(d[1], wz), wy);
        const double zz = pair_sum<2, PAIR_VV>(pair_sum<4, PAIR_DD>(d[2], wz), wy);
        const double yz = pair_sum<2, PAIR_VD>(pair_sum<4, PAIR_VD>(d[3], wz), wy);
        const double xz = pair_sum<2, PAIR_VV>(pair_sum<4, PAIR_VD>(d[4], wz), wy);
        const double xy = pair_sum<2, PAIR_VD>(pair_sum<4, PAIR_VV>(d[5], wz), wy);
        emit(pair_sum<1, PAIR_DD>(xx, wx) + pair_sum<1, PAIR_VV>(yy + zz + yz, wx) +
             pair_sum<1, PAIR_VD>(xz + xy, wx));
      }
    }
  }
#pragma unroll
  for (int m = 0; m < 6; ++m) {  // u-eta, weights dN_j N
    double d[6];
#pragma unroll
    for (int u = 0; u < 3; ++u) {
      const double2 v = Dp[(MF_EK / 2 + 3 * m + u) * 64];
      d[2 * u] = v.x, d[2 * u + 1] = v.y;
    }
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      double c[3];
#pragma unroll
      for (int j = 0; j < 3; ++j)
        c[j] = cue * (F[3 * i] * d[SI(0, j)] + F[3 * i + 1] * d[SI(1, j)] + F[3 * i + 2] * d[SI(2, j)]);
      const double x = pair_sum<2, PAIR_VV>(pair_sum<4, PAIR_VV>(c[0], wz), wy);
      const double y = pair_sum<2, PAIR_VD>(pair_sum<4, PAIR_VV>(c[1], wz), wy);
      const double z = pair_sum<2, PAIR_VV>(pair_sum<4, PAIR_VD>(c[2], wz), wy);
      emit(pair_sum<1, PAIR_VD>(x, wx) + pair_sum<1, PAIR_VV>(y + z, wx));
    }
  }
  {
    double2 v[(MF_NK - MF_KK) / 2];
#pragma unroll
    for (int k = 0; k < (MF_NK - MF_KK) / 2; ++k) v[k] = Dp[(MF_KK / 2 + k) * 64];
    // eta-eta, weight N^2, and the gradient energy h Lap_aa Mg with Lap_aa = 1/3
#pragma unroll
    for (int m = 0, k = 0; m < 6; ++m)
#pragma unroll
      for (int l = 0; l <= m; ++l, ++k) {
        const double d = cee * ((k & 1) ? v[k >> 1].y : v[k >> 1].x);
        emit(pair_sum<1, PAIR_VV>(pair_sum<2, PAIR_VV>(pair_sum<4, PAIR_VV>(d, wz), wy), wx) + h / 3.0 * cd->Mg[l][m]);
      }
  }
}
// Node sums of the merged parts -> full diagonal blocks.  A workgroup takes a
// tile of 64 nodes, each wavefront five of the 45 entries with all their loads
// in flight; the tile's blocks then leave LDS in whole 16-byte words.  (A thread
// per node and block row, single values stored: 250 -> 153 us at 65^3 nodes, 560 MB.)
constexpr int DG_WAVES = 9, DG_PER = DG_ENTRIES / DG_WAVES;
__device__ __forceinline__ void mf_diag_gather_body(const Grid& g, const Chunk& ck, const double* __restrict__ E,
                                                    double* __restrict__ diag64, int bid) {
  __shared__ double sh[DG_ENTRIES * TILE];
  const int t = ck.n0 / TILE + bid;
  {
    const int l = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), n = t * TILE + l;
    double s[DG_PER];
#pragma unroll
    for (int u = 0; u < DG_PER; ++u) s[u] = 0.0;
    if (n >= ck.n0 && n < ck.n1 && n < g.N) {
      const int nz = ck.NEc / (g.nx * g.ny);
      const int64_t nw = slab_nw(ck), nr = ck.NEc / g.nx, se = ck.NEcpad;
      const int i = n % g.nnx, j = (n / g.nnx) % g.nny, k = n / (g.nnx * g.nny) - (int)(ck.e0 / ((int64_t)g.nx * g.ny));
      double a[4][DG_PER], b[4][DG_PER];
      bool in[4];
#pragma unroll
      for (int q = 3; q >= 0; --q) {  // element row (j - by, k - bz) holds the node at (by, bz)
        const int ey = j - (q & 1), ez = k - (q >> 1);
        in[q] = ey >= 0 && ey < g.ny && ez >= 0 && ez < nz;
        const int64_t r = in[q] ? ey + (int64_t)g.ny * ez : 0, e = i + g.nx * r;
        const bool cut = i > 0 && i < g.nx && (e & (DG_EPW - 1)) == 0;  // element e - 1 ended a workgroup
#pragma unroll
        for (int u = 0; u < DG_PER; ++u) {
          const int x = w + DG_WAVES * u;  // stream x / 9 * 9 + x % 9
          const double* G = E + x / 9 * slab_values(ck, g.nx, 9);
          const int64_t st = 9 * q + x % 9;
          const double* W = G + 36 * se;
          a[q][u] = *(i < g.nx ? G + st * se + e : W + 36 * nw + st * nr + r);
          b[q][u] = 0.0;
          if (cut) b[q][u] = W[st * nw + e / DG_EPW - 1];
        }
      }
#pragma unroll
      for (int q = 3; q >= 0; --q)
        if (in[q]) {
#pragma unroll
          for (int u = 0; u < DG_PER; ++u) s[u] += a[q][u] + b[q][u];
        }
    }
#pragma unroll
    for (int u = 0; u < DG_PER; ++u) sh[(w + DG_WAVES * u) * TILE + l] = s[u];
  }
  __syncthreads();
  double2* db = reinterpret_cast<double2*>(diag64 + (int64_t)t * Lay<double>::SLICE);
  for (int x = threadIdx.x; x < (82 / 2) * TILE; x += DG_WAVES * 64) {
    const int e = x / TILE * 2, l = x % TILE, n = t * TILE + l;
    if (n < ck.n0 || n >= ck.n1) continue;
    double2 v;
    v.x = sh[diag_stream(e / 9, e % 9) * TILE + l];
    v.y = e + 1 < 81 ? sh[diag_stream((e + 1) / 9, (e + 1) % 9) * TILE + l] : 0.0;
    db[x] = v;
  }
}
__global__ void __launch_bounds__(256, 3) mf_diag_kernel(Grid g, Chunk ck, const double* __restrict__ D,
                                                      const DevCard* __restrict__ cd, double* __restrict__ E) {
  mf_diag_body(g, ck, D, cd, E, blockIdx.x, gridDim.x);
}
__global__ void __launch_bounds__(64 * DG_WAVES) mf_diag_gather_kernel(Grid g, Chunk ck, const double* __restrict__ E,
                                                             double* __restrict__ diag64) {
  mf_diag_gather_body(g, ck, E, diag64, blockIdx.x);
}
__global__ void __launch_bounds__(256, 3) mf_diag_batch(const AJob* __restrict__ jobs, int njobs) {
  int bid;
  const AJob& j = find_job(jobs, njobs, bid);
  mf_diag_body(j.g, j.ck, j.D64, j.cd, j.elem, bid, j.nblk);
}
__global__ void __launch_bounds__(64 * DG_WAVES) mf_diag_gather_batch(const AJob* __restrict__ jobs, int njobs) {
  int bid;
  const AJob& j = find_job(jobs, njobs, bid);
  mf_diag_gather_body(j.g, j.ck, j.elem, j.diag64, bid);
}
// values of the element buffer a slab of ne elements (padded) in rows of nx uses
int64_t mf_diag_values(int64_t ne, int nx) { return 4 * DG_ENTRIES * (ne + ne / SLAB_EPW + ne / nx + 1); }
int mf_diag_blocks(const Chunk& ck) { return ck.NEcpad / DG_EPW; }
int mf_diag_gather_blocks(const Chunk& ck) { return (ck.n1 + TILE - 1) / TILE - ck.n0 / TILE; }
void launch_mf_diag(const Grid& g, const Chunk& ck, const double* D64, const DevCard* cd, double* elem, double* diag64,
                    hipStream_t s) {
  if constexpr (!MF_AVAILABLE) return;
  mf_diag_kernel<<<mf_diag_blocks(ck), 256, 0, s>>>(g, ck, D64, cd, elem);
  mf_diag_gather_kernel<<<mf_diag_gather_blocks(ck), 64 * DG_WAVES, 0, s>>>(g, ck, elem, diag64);
}
void launch_mf_diag_batch(int op, const AJob* jobs, int njobs, int blocks, hipStream_t s) {
  if constexpr (!MF_AVAILABLE) return;
  if (op == AOP_MF_DIAG) mf_diag_batch<<<blocks, 256, 0, s>>>(jobs, njobs);
  else mf_diag_gather_batch<<<blocks, 64 * DG_WAVES, 0, s>>>(jobs, njobs);
}

// Register budgets (measured equal within 1 % for prefetch depths 12 and more
// at 2 ... 4 waves per SIMD): FP64 tangents 16 vectors ahead at >= 2 waves per
// SIMD.  FP32 8 ahead at >= 3 waves (160 registers): 12 ahead take 1 to 2 %
// longer, from 14 on registers spill (41^3 nodes: 54 and 60 us), and 16 ahead at
// 2 waves take 57.
constexpr int MF_PF32 = 8, MF_MINB32 = 3, MF_PF64 = 16, MF_MINB64 = 2;
template <typename TD, typename TX, typename T>
void launch_mf_element(const Grid& g, const TD* D, const TX* x, const uint16_t* mask, const DevCard* cd, T* E,
                       hipStream_t s, bool sparse_x, int elems_per_wg) {
  if constexpr (!MF_AVAILABLE) return;
  const int64_t threads = (int64_t)g.NEpad * 8;  // NEpad is a multiple of 64: whole wavefronts
  constexpr bool f64 = sizeof(TD) == 8;
  constexpr int MINB = f64 ? MF_MINB64 : MF_MINB32, PF = f64 ? MF_PF64 : MF_PF32;
  const int wg = 8 * mf_epw_of(elems_per_wg);  // divides threads
  const int blocks = (int)(threads / wg);
  if (sparse_x)
    mf_element_kernel<TD, TX, T, MINB, PF, true><<<blocks, wg, 0, s>>>(g, D, x, mask, cd, E);
  else
    mf_element_kernel<TD, TX, T, MINB, PF, false><<<blocks, wg, 0, s>>>(g, D, x, mask, cd, E);
}

// Tiles up to which a grid is gathered by tiles.  A tile per CU where that is
// ahead (V-cycle or product, us by tile and by node): FP64 V-cycle 9^3 nodes 106
// and 121, 21^3 148 and 167, 25^3 (245 tiles) 202 and 216, 33^3 (562 tiles) 346
// and 326; products in either type 33 and 36, 41 and 44 (25^3), 45.7 and 47.6
// (329 tiles).  The FP32 sweep reads its packed blocks back from LDS in words
// four apart, at a quarter of the banks: 17 x 17 x 13 (59 tiles) 127 to 136 and
// 132, 17^3 140 and 135, 21^3 163 and 142, 25^3 202 and 169.
template <int MODE, typename T>
constexpr int MF_GATHER_TILES = MODE == 2 && sizeof(T) == 4 ? 64 : 256;
template <int MODE, typename T, typename TX, typename TY>
void launch_mf_gather(const Grid& g, const T* E, bool contact, int elems_per_wg, const uint16_t* mask, const TX* x,
                      const T* b, const T* Dinv, T omega, TY* y, hipStream_t s) {
  if constexpr (!MF_AVAILABLE) return;
  const T* Cf = contact ? E + mf_cf_offset(g) : nullptr;
  const int epw = mf_epw_of(elems_per_wg);
  if (g.ntiles <= MF_GATHER_TILES<MODE, T>)
    mf_gather_tile_kernel<MODE, T, TX, TY><<<g.ntiles, GT, 0, s>>>(g, E, Cf, epw, mask, x, b, Dinv, omega, y);
  else
    mf_gather_kernel<MODE, T, TX, TY><<<(g.Npad + 255) / 256, 256, 0, s>>>(g, E, Cf, epw, mask, x, b, Dinv, omega, y);
}

template void launch_mf_element<float, float, float>(const Grid&, const float*, const float*, const uint16_t*,
                                                     const DevCard*, float*, hipStream_t, bool, int);
template void launch_mf_element<double, float, double>(const Grid&, const double*, const float*, const uint16_t*,
                                                       const DevCard*, double*, hipStream_t, bool, int);
template void launch_mf_element<double, double, double>(const Grid&, const double*, const double*, const uint16_t*,
                                                        const DevCard*, double*, hipStream_t, bool, int);
template void launch_mf_gather<0, float, float, float>(const Grid&, const float*, bool, int, const uint16_t*,
                                                       const float*, const float*, const float*, float, float*,
                                                       hipStream_t);
template void launch_mf_gather<1, float, float, float>(const Grid&, const float*, bool, int, const uint16_t*,
                                                       const float*, const float*, const float*, float, float*,
                                                       hipStream_t);
template void launch_mf_gather<2, float, float, float>(const Grid&, const float*, bool, int, const uint16_t*,
                                                       const float*, const float*, const float*, float, float*,
                                                       hipStream_t);
template void launch_mf_gather<0, double, float, double>(const Grid&, const double*, bool, int, const uint16_t*,
                                                         const float*, const double*, const double*, double, double*,
                                                         hipStream_t);
template void launch_mf_gather<0, double, double, double>(const Grid&, const double*, bool, int, const uint16_t*,
                                                          const double*, const double*, const double*, double,
                                                          double*, hipStream_t);
template void launch_mf_gather<1, double, double, double>(const Grid&, const double*, bool, int, const uint16_t*,
                                                          const double*, const double*, const double*, double,
                                                          double*, hipStream_t);
template void launch_mf_gather<2, double, double, double>(const Grid&, const double*, bool, int, const uint16_t*,
                                                          const double*, const double*, const double*, double,
                                                          double*, hipStream_t);

// ---- batched launches (FP32 or FP64 smoothing on matrix-free finest levels) ----
template <typename T, int MINB, int PF>
__global__ void __launch_bounds__(256, MINB) mf_element_batch(const BJob* __restrict__ jobs, int njobs) {
  int bid;
  const BJob& j = find_job(jobs, njobs, bid);
  mf_element_body<T, T, T, PF, false>(j.g, (const T*)j.A, (const T*)j.x, j.mask, j.cd, (T*)j.C, bid, j.nblk);
}
template <int MODE, typename T>
__global__ void __launch_bounds__(256) mf_gather_batch(const BJob* __restrict__ jobs, int njobs) {
  int bid;
  const BJob& j = find_job(jobs, njobs, bid);
  mf_gather_body<MODE, T, T, T>(j.g, (const T*)j.C, j.contact ? (const T*)j.C + mf_cf_offset(j.g) : nullptr, j.epw,
                                j.mask, (const T*)j.x, (const T*)j.b, (const T*)j.D, (T)j.omega,
                                (T*)j.y, bid);
}
template <typename T>
void launch_mf_batch(int op, const BJob* jobs, int njobs, int blocks, hipStream_t s, int threads) {
  if constexpr (!MF_AVAILABLE) return;
  constexpr bool f64 = sizeof(T) == 8;
  if (op == BOP_MF_ELEMENT)
    mf_element_batch<T, f64 ? MF_MINB64 : MF_MINB32, f64 ? MF_PF64 : MF_PF32><<<blocks, threads, 0, s>>>(jobs, njobs);
  else if (op == BOP_MF_GATHER_PBJ)
    mf_gather_batch<2, T><<<blocks, 256, 0, s>>>(jobs, njobs);
  else if (op == BOP_MF_GATHER_DEFECT)
    mf_gather_batch<1, T><<<blocks, 256, 0, s>>>(jobs, njobs);
}
template void launch_mf_batch<float>(int, const BJob*, int, int, hipStream_t, int);
template void launch_mf_batch<double>(int, const BJob*, int, int, hipStream_t, int);
// element kernels: threads (64, 128 or 256) divide the 8 NEpad lanes exactly
int mf_job_blocks(int op, const Grid& g, int threads) {
  return (op == BOP_MF_ELEMENT || op == BOP_MF_OUTER_ELEMENT) ? (int)((int64_t)g.NEpad * 8 / threads)
                                                             : (g.Npad + 255) / 256;
}

// batched FGMRES operator product on matrix-free finest levels: FP64
// Hessians, input z of type TZ (the preconditioned vector), FP64 output
template <typename TZ>
__global__ void __launch_bounds__(256, MF_MINB64) mf_outer_element_batch(const BJob* __restrict__ jobs, int njobs) {
  int bid;
  const BJob& j = find_job(jobs, njobs, bid);
  mf_element_body<double, TZ, double, MF_PF64, false>(j.g, (const double*)j.A, (const TZ*)j.x, j.mask, j.cd,
                                                      (double*)j.C, bid, j.nblk);
}
template <typename TZ>
__global__ void __launch_bounds__(256) mf_outer_gather_batch(const BJob* __restrict__ jobs, int njobs) {
  int bid;
  const BJob& j = find_job(jobs, njobs, bid);
  mf_gather_body<0, double, TZ, double>(j.g, (const double*)j.C,
                                        j.contact ? (const double*)j.C + mf_cf_offset(j.g) : nullptr, j.epw, j.mask,
                                        (const TZ*)j.x, nullptr, nullptr, 0.0,
                                        (double*)j.y, bid);
}
template <typename TZ>
void launch_mf_outer_batch(int op, const BJob* jobs, int njobs, int blocks, hipStream_t s, int threads) {
  if constexpr (!MF_AVAILABLE) return;
  if (op == BOP_MF_OUTER_ELEMENT)
    mf_outer_element_batch<TZ><<<blocks, threads, 0, s>>>(jobs, njobs);
  else if (op == BOP_MF_OUTER_GATHER)
    mf_outer_gather_batch<TZ><<<blocks, 256, 0, s>>>(jobs, njobs);
}
template void launch_mf_outer_batch<float>(int, const BJob*, int, int, hipStream_t, int);
template void launch_mf_outer_batch<double>(int, const BJob*, int, int, hipStream_t, int);

}  // namespace mvpf
