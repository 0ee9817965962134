// Galerkin coarse operators, an alternative to the rediscretised coarse
// levels of Sec. 3.4 (opts.coarse = MVPF_COARSE_GALERKIN):
//   A_{l+1} = P~^T A_l P~,
// with P the trilinear prolongation of the V-cycle and P~ = P with the rows of
// constrained level-l unknowns set to zero (the V-cycle never adds a
// correction there), followed by the symmetric elimination of the constrained
// level-(l+1) unknowns.  Where the penalty of the order parameters is active
// on a pattern finer than a coarse element (a state the injected coarse state
// cannot represent), the two constructions differ and only this one keeps the
// coarse correction A-orthogonal to the coarse space.
//
// Built element by element on the nested structured levels: parent element E
// of level l+1 has the 8 children s of level l, and
//   K_E = sum_s W~_s^T K_s W~_s,
//   W~_s[(a, c), (A, c)] = w(a, A) * free_l(node of child corner a, c),
// K_s the child's element matrix (its 36 stored node pairs), w(a, A) the
// trilinear weight of parent corner A at child corner a (a tensor product of
// the 1D weights 1, 1/2, 0 at child positions 0, 1, 2 halves of the parent).
// Summing K_E over the parents that share two nodes (jacobian_gather) gives
// P~^T K P~, which equals P~^T A_l P~ because P~ removes every constrained
// row and column.  Level 0's element matrices come from the Gauss-point
// Hessians (element_matrix, contact included), so the whole hierarchy
// inherits the finest tangent exactly.
#include <utility>

#include "common.h"

namespace mvpf {

// 1D weight of parent corner bit A at child-level position p (0, 1, 2)
__host__ __device__ constexpr double gal_w1(int p, int A) {
  return p == 1 ? 0.5 : ((p == 0) == (A == 0) ? 1.0 : 0.0);
}
// weight of parent corner A at corner a of child s
__host__ __device__ constexpr double gal_w(int s, int a, int A) {
  return gal_w1((s & 1) + (a & 1), A & 1) * gal_w1(((s >> 1) & 1) + ((a >> 1) & 1), (A >> 1) & 1) *
         gal_w1((s >> 2) + (a >> 2), A >> 2);
}
// index of corner a of child s among the parent's 3 x 3 x 3 child-level nodes
__host__ __device__ constexpr int gal_node(int s, int a) {
  return ((s & 1) + (a & 1)) + 3 * (((s >> 1) & 1) + ((a >> 1) & 1)) + 9 * ((s >> 2) + (a >> 2));
}

// acc[pair(A, B)] += w(a, A) w(b, B) k for parent pair I = 8 A + B, A <= B;
// the weights are compile-time constants, zero terms are not generated
template <int S, int a, int b, int I>
__device__ __forceinline__ void gal_term(double k, double (&acc)[NPAIR]) {
  constexpr int A = I >> 3, B = I & 7;
  if constexpr (A <= B) {
    constexpr double w = gal_w(S, a, A) * gal_w(S, b, B);
    if constexpr (w != 0.0) acc[pair_index(A, B)] += w * k;
  }
}
template <int S, int a, int b, int... I>
__device__ __forceinline__ void gal_terms(double k, double (&acc)[NPAIR], std::integer_sequence<int, I...>) {
  (gal_term<S, a, b, I>(k, acc), ...);
}
// the ordered child corner pair (a, b) contributes entry (c, c2) of K_ab to
// entry (c, c2) of the parent blocks, zero where dof c of corner a or dof c2
// of corner b is constrained (fa, fb: free bits of dofs c and c2)
template <int S, int a, int b>
__device__ __forceinline__ void gal_add(double k, uint32_t fa, uint32_t fb, double (&acc)[NPAIR]) {
  const bool keep = ((fa >> gal_node(S, a)) & (fb >> gal_node(S, b)) & 1u) != 0u;
  gal_terms<S, a, b>(keep ? k : 0.0, acc, std::make_integer_sequence<int, 64>{});
}
// stored child pair P (a <= b): its entries q = (c, c2) and qt = (c2, c),
// i.e. K_ab[c][c2] and K_ab[c2][c], are also K_ba[c2][c] and K_ba[c][c2];
// the lane accumulates entry q (accq) and, off the diagonal of the blocks,
// entry qt (acct) of the parent pairs, so each child entry is read once
template <int S, bool DIAG, int P>
__device__ __forceinline__ void gal_child_pair(const double* __restrict__ Ee, int64_t es, int q, int qt, uint32_t fc,
                                               uint32_t fc2, double (&accq)[NPAIR], double (&acct)[NPAIR]) {
  constexpr int a = pair_a(P), b = pair_b(P);
  const double kq = Ee[((int64_t)P * NBLK + q) * es];
  if constexpr (DIAG) {  // c == c2: K_ab[c][c] = K_ba[c][c]
    gal_add<S, a, b>(kq, fc, fc, accq);
    if constexpr (a != b) gal_add<S, b, a>(kq, fc, fc, accq);
  } else {
    const double kt = Ee[((int64_t)P * NBLK + qt) * es];
    gal_add<S, a, b>(kq, fc, fc2, accq);   // K_ab[c][c2]
    gal_add<S, a, b>(kt, fc2, fc, acct);   // K_ab[c2][c]
    if constexpr (a != b) {
      gal_add<S, b, a>(kt, fc, fc2, accq);  // K_ba[c][c2] = K_ab[c2][c]
      gal_add<S, b, a>(kq, fc2, fc, acct);  // K_ba[c2][c] = K_ab[c][c2]
    }
  }
}
template <int S, bool DIAG, int... P>
__device__ __forceinline__ void gal_child(const double* __restrict__ Ee, int64_t es, int q, int qt, uint32_t fc,
                                          uint32_t fc2, double (&accq)[NPAIR], double (&acct)[NPAIR],
                                          std::integer_sequence<int, P...>) {
  (gal_child_pair<S, DIAG, P>(Ee, es, q, qt, fc, fc2, accq, acct), ...);
}

// Block entries handled together: the diagonal ones (c, c) alone, the others
// as the pairs (c, c2), (c2, c) with c < c2: NDOF (NDOF + 1) / 2 tasks.
constexpr int GAL_TASKS = NDOF * (NDOF + 1) / 2;
__device__ __forceinline__ void gal_task(int task, int& c, int& c2) {
  c = 0;
  while (task >= NDOF - c) { task -= NDOF - c; ++c; }
  c2 = c + task;
}

template <bool DIAG>
__device__ __forceinline__ void gal_parent(const Grid& gc, const Chunk& ckc, const double* __restrict__ Ec,
                                           const Grid& gp, int64_t E, int c, int c2, uint32_t fc, uint32_t fc2,
                                           double* __restrict__ Ep) {
  const int q = NDOF * c + c2, qt = NDOF * c2 + c;
  const int X = (int)(E % gp.nx), Y = (int)((E / gp.nx) % gp.ny), Z = (int)(E / ((int64_t)gp.nx * gp.ny));
  double accq[NPAIR], acct[NPAIR];
#pragma unroll
  for (int p = 0; p < NPAIR; ++p) accq[p] = acct[p] = 0.0;
  const int64_t es = ckc.NEcpad;
  const int64_t nxc = gc.nx, nxyc = (int64_t)gc.nx * gc.ny;
  const int64_t e00 = 2 * X + nxc * 2 * Y + nxyc * 2 * Z - ckc.e0;  // child 0, chunk-local
  const std::make_integer_sequence<int, NPAIR> pairs{};
  gal_child<0, DIAG>(Ec + e00, es, q, qt, fc, fc2, accq, acct, pairs);
  gal_child<1, DIAG>(Ec + e00 + 1, es, q, qt, fc, fc2, accq, acct, pairs);
  gal_child<2, DIAG>(Ec + e00 + nxc, es, q, qt, fc, fc2, accq, acct, pairs);
  gal_child<3, DIAG>(Ec + e00 + nxc + 1, es, q, qt, fc, fc2, accq, acct, pairs);
  gal_child<4, DIAG>(Ec + e00 + nxyc, es, q, qt, fc, fc2, accq, acct, pairs);
  gal_child<5, DIAG>(Ec + e00 + nxyc + 1, es, q, qt, fc, fc2, accq, acct, pairs);
  gal_child<6, DIAG>(Ec + e00 + nxyc + nxc, es, q, qt, fc, fc2, accq, acct, pairs);
  gal_child<7, DIAG>(Ec + e00 + nxyc + nxc + 1, es, q, qt, fc, fc2, accq, acct, pairs);
#pragma unroll
  for (int p = 0; p < NPAIR; ++p) Ep[((int64_t)p * NBLK + q) * gp.NEpad + E] = accq[p];
  if constexpr (!DIAG) {
#pragma unroll
    for (int p = 0; p < NPAIR; ++p) Ep[((int64_t)p * NBLK + qt) * gp.NEpad + E] = acct[p];
  }
}

// One wavefront per 64 consecutive parents and one task: block entry (c, c)
// or the entry pair (c, c2), (c2, c).  Each lane accumulates those entries of
// its parent's 36 node pairs over the 8 children and their corner pairs, in
// a fixed order (bitwise reproducible), reading each child entry it needs
// once.  The tasks of one parent group are consecutive logical workgroups on
// one XCD.  Child element matrices: chunk-local, Ec[(p NBLK + q) es + e - e0];
// parents: whole level, Ep[(P NBLK + q) NEpad + E], E in [E0, E1).
__global__ void __launch_bounds__(64) galerkin_coarsen_kernel(Grid gc, Chunk ckc, const double* __restrict__ Ec,
                                                             const uint16_t* __restrict__ maskc, Grid gp,
                                                             int64_t E0, int64_t E1, int nwork, double* __restrict__ Ep) {
  const int L = xcd_logical(blockIdx.x, gridDim.x);
  if (L >= nwork) return;
  int c, c2;
  gal_task(L % GAL_TASKS, c, c2);
  const int64_t E = E0 + (int64_t)(L / GAL_TASKS) * 64 + threadIdx.x;
  if (E >= E1) return;
  const int X = (int)(E % gp.nx), Y = (int)((E / gp.nx) % gp.ny), Z = (int)(E / ((int64_t)gp.nx * gp.ny));
  // free bits of dofs c (fc) and c2 (fc2) of the parent's 27 child-level nodes
  uint32_t fc = 0, fc2 = 0;
#pragma unroll
  for (int k = 0; k < 27; ++k) {
    const int64_t node = (2 * X + k % 3) + (int64_t)gc.nnx * ((2 * Y + (k / 3) % 3) + (int64_t)gc.nny * (2 * Z + k / 9));
    const uint32_t m = maskc[node];
    fc |= ((~m >> c) & 1u) << k;
    fc2 |= ((~m >> c2) & 1u) << k;
  }
  if (c == c2)
    gal_parent<true>(gc, ckc, Ec, gp, E, c, c2, fc, fc2, Ep);
  else
    gal_parent<false>(gc, ckc, Ec, gp, E, c, c2, fc, fc2, Ep);
}

void launch_galerkin_coarsen(const Grid& gc, const Chunk& ckc, const double* Ec, const uint16_t* maskc,
                             const Grid& gp, int Z0, int Z1, double* Ep, hipStream_t s) {
  const int64_t nxy = (int64_t)gp.nx * gp.ny;
  const int64_t E0 = Z0 * nxy, E1 = Z1 * nxy;
  if (E1 <= E0) return;
  const int64_t nwork = (E1 - E0 + 63) / 64 * GAL_TASKS;
  const int blocks = (int)((nwork + 7) / 8 * 8);
  galerkin_coarsen_kernel<<<blocks, 64, 0, s>>>(gc, ckc, Ec, maskc, gp, E0, E1, (int)nwork, Ep);
}


// ---- level 1 straight from a matrix-free finest level's Gauss points -----------
// On a matrix-free finest level the child element matrices exist nowhere else:
// K_E = sum over the parent's 4 x 4 x 4 Gauss points g of W~^T B^T D_g B W~, and
// the columns of B W~ are the parent's own shape functions at those points
// (trilinear functions are interpolated exactly), so
//   K_E[(A, c), (B, c2)] = sum_g sum_(p, q) f_A^p(g) f_B^q(g) D_g(p, q)
// with f the parent's shape values (order parameters) or derivatives (F), each
// a product of one-dimensional factors.  The sums are taken one direction at a
// time: 4 points -> the 4 corner combinations (a, b), x then y then z, with
// entries of equal remaining factors added up on the way.  Against the element
// matrices (2916 values per child written and read back) this reads 768 values
// per child and writes the parents only.
//
// A constrained plane z = 0 of the child level (all u of its nodes, the bottom
// face) keeps the tensor product: P~ zeroes the plane's nodes, so the u-functions
// of the bottom parents are the same in x and y and piecewise linear in z with
// the value 0 at the plane.  The parents of the top layer, whose constraints and
// contact follow no such pattern, go through galerkin_coarsen.
//
// A workgroup holds 8 parents of a row, i.e. 16 children in x, and takes their
// 4 child rows (y, z) in turn: its first 128 threads read one Gauss point each
// (the layout's own order) and put the entries of D in (F, eta) into LDS, from
// there every thread accumulates the 64 corner combinations of one block entry
// (c, c2) of one parent.  ROLE 0: u-u (6 block entries of 9 entries of D each),
// 1: u-eta (18 of 3), 2: eta-eta (21 of 1, plus the gradient energy).
// Bound: FP64 issue and LDS at one to two wavefronts per SIMD; 64^3: 0.30 + 0.38
// + 0.16 ms, against 3.45 ms for the element matrices and 2.5 ms for their
// coarsening.
constexpr int GD_PARENTS = 8, GD_POINTS = 8 * 2 * GD_PARENTS;
template <int ROLE>
struct GalRole {
  static constexpr int tasks = ROLE == 0 ? 6 : ROLE == 1 ? 18 : 21;
  static constexpr int entries = ROLE == 0 ? 9 : ROLE == 1 ? 3 : 1;  // per task
  static constexpr int ztypes = ROLE == 0 ? 4 : ROLE == 1 ? 2 : 1;   // derivative along z of (A, B): none, A, B, both
  static constexpr int stride = entries * GD_POINTS + 16;            // LDS values per task (16: spreads the tasks' banks)
  static constexpr int threads = ROLE == 0 ? 128 : 192;
  // direction of the derivative of A's and B's factor for entry e (-1: a value)
  __host__ __device__ static constexpr int dA(int e) { return ROLE == 0 ? e / 3 : ROLE == 1 ? e : -1; }
  __host__ __device__ static constexpr int dB(int e) { return ROLE == 0 ? e % 3 : -1; }
};
// abscissae of the four points of a direction on the parent's unit interval
__host__ __device__ constexpr double gd_point(int t) {
  return 0.5 * ((t >> 1) + ((t & 1) ? 0.78867513459481288225 : 0.21132486540518711775));
}
__host__ __device__ constexpr double gd_value(int t, int a) { return a ? gd_point(t) : 1.0 - gd_point(t); }

template <int ROLE>
__global__ void __launch_bounds__(GalRole<ROLE>::threads)
    galerkin_direct_kernel(Grid gc, const double* __restrict__ D, const DevCard* __restrict__ cd, Grid gp, int Z0,
                           int nwork, double* __restrict__ Ep) {
  using R = GalRole<ROLE>;
  __shared__ __attribute__((aligned(16))) double T[R::tasks * R::stride];
  const int L = xcd_logical(blockIdx.x, gridDim.x);
  if (L >= nwork) return;  // uniform
  const int nbx = (gp.nx + GD_PARENTS - 1) / GD_PARENTS;
  const int bx = L % nbx, Y = (L / nbx) % gp.ny, Z = Z0 + L / (nbx * gp.ny);
  const int tid = threadIdx.x;
  // the Gauss point this thread reads
  const int el = 8 * (tid >> 6) + (tid & 7), g = (tid >> 3) & 7, x = 2 * GD_PARENTS * bx + el;
  const bool reads = tid < GD_POINTS, inside = reads && x < gc.nx;
  double* const Tp = T + g * 16 + el;
  // the block entry and parent it sums
  const int task = tid >> 3, X = tid & 7;
  const bool sums = task < R::tasks;
  const double* const Ts = T + (sums ? task : 0) * R::stride + 2 * X;
  double acc[64];
#pragma unroll
  for (int i = 0; i < 64; ++i) acc[i] = 0.0;
#pragma unroll 1
  for (int row = 0; row < 4; ++row) {
    const int dy = row & 1, dz = row >> 1;
    if (row > 0) __syncthreads();
    if (reads) {
      const int64_t e = x + (int64_t)gc.nx * ((2 * Y + dy) + (int64_t)gc.ny * (2 * Z + dz));
      const double2* Dp = reinterpret_cast<const double2*>(D) + ((e >> 3) * (MF_NK / 2) * 64 + g * 8 + (e & 7));
      auto put = [&](int t, int k, double v) { Tp[t * R::stride + k * GD_POINTS] = v; };
      if constexpr (ROLE < 2) {
        constexpr int n = ROLE == 0 ? MF_EK / 2 : 5;
        double2 v[n];
#pragma unroll
        for (int k = 0; k < n; ++k) v[k] = inside ? Dp[k * 64] : make_double2(0.0, 0.0);
        auto at = [&](int k) { return (k & 1) ? v[k >> 1].y : v[k >> 1].x; };
        double F[9];
#pragma unroll
        for (int i = 0; i < 9; ++i) F[i] = at(MF_G + i) + (i % 4 == 0 ? 1.0 : 0.0);
        if constexpr (ROLE == 0) {
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
            for (int i = 0; i <= k; ++i)
#pragma unroll
              for (int j = 0; j < 3; ++j)
#pragma unroll
                for (int l = 0; l < 3; ++l) {
                  double s = F[3 * i] * t[SI(0, j)][l] + F[3 * i + 1] * t[SI(1, j)][l] + F[3 * i + 2] * t[SI(2, j)][l];
                  if (i == k) s += at(MF_S + SI(j, l));
                  put(k * (k + 1) / 2 + i, 3 * j + l, s);
                }
          }
        } else {
#pragma unroll
          for (int m = 0; m < 6; ++m) {
            double d[6];
#pragma unroll
            for (int u = 0; u < 3; ++u) {
              const double2 w = inside ? Dp[(MF_EK / 2 + 3 * m + u) * 64] : make_double2(0.0, 0.0);
              d[2 * u] = w.x, d[2 * u + 1] = w.y;
            }
#pragma unroll
            for (int i = 0; i < 3; ++i)
#pragma unroll
              for (int j = 0; j < 3; ++j)
                put(3 * m + i, j, F[3 * i] * d[SI(0, j)] + F[3 * i + 1] * d[SI(1, j)] + F[3 * i + 2] * d[SI(2, j)]);
          }
        }
      } else {
        double2 v[(MF_NK - MF_KK) / 2];
#pragma unroll
        for (int k = 0; k < (MF_NK - MF_KK) / 2; ++k) v[k] = inside ? Dp[(MF_KK / 2 + k) * 64] : make_double2(0.0, 0.0);
#pragma unroll
        for (int t = 0; t < 21; ++t) put(t, 0, (t & 1) ? v[t >> 1].y : v[t >> 1].x);
      }
    }
    __syncthreads();
    if (!sums) continue;
#pragma unroll
    for (int gz = 0; gz < 2; ++gz) {
      double Yv[R::ztypes][16];  // [derivatives along z][4 (ay, by) + (ax, bx)]
#pragma unroll
      for (int zt = 0; zt < R::ztypes; ++zt)
#pragma unroll
        for (int i = 0; i < 16; ++i) Yv[zt][i] = 0.0;
#pragma unroll
      for (int gy = 0; gy < 2; ++gy) {
        double yv[2];  // the corner values at this y
#pragma unroll
        for (int a = 0; a < 2; ++a) yv[a] = dy ? gd_value(2 + gy, a) : gd_value(gy, a);
#pragma unroll
        for (int e = 0; e < R::entries; ++e) {
          const bool ax = R::dA(e) == 0, bxd = R::dB(e) == 0, ay = R::dA(e) == 1, by = R::dB(e) == 1;
          const int zt = (R::dA(e) == 2 ? 1 : 0) + (R::dB(e) == 2 ? 2 : 0);
          const double2 r0 = *reinterpret_cast<const double2*>(Ts + e * GD_POINTS + (4 * gz + 2 * gy) * 16);
          const double2 r1 = *reinterpret_cast<const double2*>(Ts + e * GD_POINTS + (4 * gz + 2 * gy + 1) * 16);
          const double d[4] = {r0.x, r1.x, r0.y, r1.y};  // points t = 2 child + gx
#pragma unroll
          for (int xc = 0; xc < 4; ++xc) {
            const int a = xc >> 1, b = xc & 1;
            double s = 0.0;
#pragma unroll
            for (int t = 0; t < 4; ++t) s += (ax ? 1.0 : gd_value(t, a)) * (bxd ? 1.0 : gd_value(t, b)) * d[t];
            if ((ax && a == 0) != (bxd && b == 0)) s = -s;  // derivatives -1, +1
#pragma unroll
            for (int yc = 0; yc < 4; ++yc) {
              const int c = yc >> 1, f = yc & 1;
              const double w = (ay ? 1.0 : yv[c]) * (by ? 1.0 : yv[f]);
              const double sw = ((ay && c == 0) != (by && f == 0)) ? -w : w;
              Yv[zt][4 * yc + xc] += sw * s;
            }
          }
        }
      }
      // values and derivatives along z: of u (A, and B in role 0) and of eta
      const bool plane = Z == 0;  // the constrained plane z = 0
      double uv[2], ud[2], ev[2];
#pragma unroll
      for (int a = 0; a < 2; ++a) {
        ev[a] = dz ? gd_value(2 + gz, a) : gd_value(gz, a);
        // with the plane's value 0 the lower child interpolates 0 and 1/2
        uv[a] = plane && !dz ? gd_point(gz) : ev[a];
        ud[a] = plane && !dz ? 1.0 : (a ? 1.0 : -1.0);
      }
#pragma unroll
      for (int zc = 0; zc < 4; ++zc) {
        const int a = zc >> 1, b = zc & 1;
#pragma unroll
        for (int zt = 0; zt < R::ztypes; ++zt) {
          const double wa = ROLE == 2 ? ev[a] : (zt & 1) ? ud[a] : uv[a];
          const double wb = ROLE != 0 ? ev[b] : (zt & 2) ? ud[b] : uv[b];
          const double w = wa * wb;
#pragma unroll
          for (int i = 0; i < 16; ++i) acc[16 * zc + i] += w * Yv[zt][i];
        }
      }
    }
  }
  const int PX = GD_PARENTS * bx + X;
  if (!sums || PX >= gp.nx) return;
  int c = 0, c2 = 0;  // the block entry
  if constexpr (ROLE == 0) {
    c2 = task == 0 ? 0 : task < 3 ? 1 : 2;
    c = task - c2 * (c2 + 1) / 2;
  } else if constexpr (ROLE == 1) {
    c = task % 3;
    c2 = 3 + task / 3;
  } else {
    int k = 0;
    while ((k + 1) * (k + 2) / 2 <= task) ++k;
    c = 3 + task - k * (k + 1) / 2;
    c2 = 3 + k;
  }
  const double h = gc.h;
  const double scale = ROLE == 0 ? h / 32.0 : ROLE == 1 ? h * h / 16.0 : h * h * h / 8.0;
  const double mg = ROLE == 2 ? 2.0 * h * cd->Mg[c - 3][c2 - 3] : 0.0;
  double* out = Ep + PX + (int64_t)gp.nx * (Y + (int64_t)gp.ny * Z);
  auto store = [&](int P, int q, double v) { out[((int64_t)P * NBLK + q) * gp.NEpad] = v; };
  const int q = NDOF * c + c2, qt = NDOF * c2 + c;
#pragma unroll
  for (int A = 0; A < 8; ++A)
#pragma unroll
    for (int B = 0; B < 8; ++B) {
      if (ROLE == 2 && A > B) continue;
      const int ic = 16 * (2 * (A >> 2) + (B >> 2)) + 4 * (2 * ((A >> 1) & 1) + ((B >> 1) & 1)) + 2 * (A & 1) + (B & 1);
      double v = scale * acc[ic];
      if constexpr (ROLE == 2) {
        // Laplacian of the unit cube: stiffness +-1 along one direction, mass 1/3 or 1/6 along the others
        const bool sx = (A & 1) == (B & 1), sy = ((A ^ B) & 2) == 0, sz = (A >> 2) == (B >> 2);
        const double mx = sx ? 1.0 / 3.0 : 1.0 / 6.0, my = sy ? 1.0 / 3.0 : 1.0 / 6.0, mz = sz ? 1.0 / 3.0 : 1.0 / 6.0;
        v += mg * ((sx ? 1.0 : -1.0) * my * mz + mx * (sy ? 1.0 : -1.0) * mz + mx * my * (sz ? 1.0 : -1.0));
        store(pair_index(A, B), q, v);
        if (c != c2) store(pair_index(A, B), qt, v);
      } else {
        // K_AB[c][c2], which is K_BA[c2][c]
        if (A <= B) store(pair_index(A, B), q, v);
        if (A >= B && c != c2) store(pair_index(B, A), qt, v);
      }
    }
}

void launch_galerkin_direct(const Grid& gc, const double* D64, const DevCard* cd, const Grid& gp, int Z0, int Z1,
                            double* Ep, hipStream_t s) {
  if constexpr (!MF_AVAILABLE) return;
  if (Z1 <= Z0) return;
  const int nwork = (gp.nx + GD_PARENTS - 1) / GD_PARENTS * gp.ny * (Z1 - Z0);
  const int blocks = (nwork + 7) / 8 * 8;
  galerkin_direct_kernel<0><<<blocks, GalRole<0>::threads, 0, s>>>(gc, D64, cd, gp, Z0, nwork, Ep);
  galerkin_direct_kernel<1><<<blocks, GalRole<1>::threads, 0, s>>>(gc, D64, cd, gp, Z0, nwork, Ep);
  galerkin_direct_kernel<2><<<blocks, GalRole<2>::threads, 0, s>>>(gc, D64, cd, gp, Z0, nwork, Ep);
}

}  // namespace mvpf
