// Coarsest-level direct solve (Sec. 3.4: the V-cycle bottoms out in a sparse
// LU factorisation).  The coarsest operator (at most 8192 unknowns) is
// gathered into a dense FP64 matrix and inverted once per Newton system by
// blocked Gauss-Jordan elimination (pivoting inside 64 x 64 blocks and a check
// of the result; pivoting over all rows where the check fails); each V-cycle then applies
// the inverse with one dense matrix-vector product (fully parallel, instead
// of two latency-bound triangular solves).
//
// Dense unknown ordering: d = c * N + n (component-major, no padding).
#include "common.h"

namespace mvpf {

// one thread per (node, stored block, block row): the NDOF entries of that row
// and, for off-diagonal blocks, their transposes (the lower half)
__global__ void __launch_bounds__(256) dense_from_bsr_kernel(Grid g, const double* __restrict__ A,
                                                             double* __restrict__ D) {
  const int idx = blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= g.N * NUP * NDOF) return;
  const int r = idx % NDOF, u = (idx / NDOF) % NUP, n = idx / (NDOF * NUP);
  const int64_t nd = (int64_t)NDOF * g.N;
  const int t = n >> 6, l = n & 63;
  const int i = n % g.nnx, j = (n / g.nnx) % g.nny, k = n / (g.nnx * g.nny);
  const int s = 13 + u;
  const int dx = s % 3 - 1, dy = (s / 3) % 3 - 1, dz = s / 9 - 1;
  if (i + dx < 0 || i + dx >= g.nnx || j + dy < 0 || j + dy >= g.nny || k + dz < 0 || k + dz >= g.nnz) return;
  const int m = n + dx + g.nnx * (dy + g.nny * dz);
  const double* Ab = A + (int64_t)(t * NUP + u) * Lay<double>::SLICE;
#pragma unroll
  for (int c = 0; c < NDOF; ++c) {
    const double v = Ab[Lay<double>::off(r * NDOF + c, l)];
    D[((int64_t)r * g.N + n) * nd + (int64_t)c * g.N + m] = v;
    if (u > 0) D[((int64_t)c * g.N + m) * nd + (int64_t)r * g.N + n] = v;  // lower half by symmetry
  }
}

__global__ void zero_kernel_d(int64_t n, double* p) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
    p[i] = 0.0;
}

void launch_dense_from_bsr(const Grid& g, const double* A64, double* dense, hipStream_t s) {
  const int64_t nd = (int64_t)NDOF * g.N;
  zero_kernel_d<<<1024, 256, 0, s>>>(nd * nd, dense);
  dense_from_bsr_kernel<<<(g.N * NUP * NDOF + 255) / 256, 256, 0, s>>>(g, A64, dense);
}

// Two-level blocked Gauss-Jordan inversion with partial pivoting over all rows
// (dense_invert_pivoted).
//
// M = [A | Y] is n x 2n, row-major.  Y starts at zero; the k-th pivot row
// p_k (the row chosen for column k) gets its unit vector e_{p_k} placed in
// column n + k at the moment it is chosen, so the right half ends up holding
// T e_{p_k}, where T is the product of all elimination steps.  Since
// T A = E with E[p_k][k] = 1, row k of A^-1 is row p_k of T, i.e.
// A^-1[k][p_m] = M[p_k][n + m].
//
// Outer panels of NB columns c0 .. c0 + nbw - 1.  Inside a panel, sub-panels
// of PB columns are eliminated with partial pivoting by
//   0. gj_fetch: copies the sub-panel F = M[:, sub-panel] (row-major F and
//      column-major Wc);
//   1. gj_panel: one workgroup holds the sub-panel in registers, chooses the
//      pivot rows by elimination with partial pivoting restricted to the
//      sub-panel (rows pivoted earlier are excluded), places the unit
//      columns and inverts the pivot block Mp = F[P, :] (Gauss-Jordan in
//      LDS, rows in pivot order); beyond 4 GJ_THREADS rows the same is done
//      by tournament pivoting (gj_tourn0, gj_tourn1);
//   2. gj_rows: R = Mp^-1 M[P, active] (the new pivot rows);
//   3. gj_update: rows in P become R, every other row i becomes
//      M[i, active] - F[i, :] R,
// where "active" is only the outer panel's 2 nbw columns [c0, c0 + nbw) and
// [n + c0, n + c0 + nbw).  Columns outside the active set are either
// untouched by these steps (eliminated unit columns, zero columns of Y) or
// are updated once per outer panel: with T_o the panel's accumulated
// transformation, T_o - I is non-zero only in the columns p_k, whose values
// T_o e_{p_k} - e_{p_k} =: Yo[:, k] sit in the right half, so
//   M[:, rest] += Yo * M_old[P, rest],   rest = [c0 + nbw, n + c0)
// (gj_gather copies Yo and the old pivot rows; gj_gemm does the product).
constexpr int BG = 64;    // block of the block elimination (below)
constexpr int GJB = 32;   // widest sub-panel
constexpr int GJ_NB = 128;  // outer panel width
constexpr int GJ_THREADS = 512;

// Several inversions can run as one: every kernel of either elimination works on
// job z of a device table, or on the one job passed by value (a type of its own:
// a choice at run time puts the job's pointers behind vector loads, 1125
// unknowns with pivoting over all rows 4.4 -> 4.8 ms).  Each job keeps its own
// panel widths and kernel variants, so it computes the same numbers alone or in
// a batch.
struct GJOne {
  GJJob job;
  __device__ __forceinline__ const GJJob& get() const { return job; }
};
struct GJTab {
  const GJJob* tab;
  __device__ __forceinline__ const GJJob& get() const { return tab[blockIdx.z]; }
};

// sub-panel width: up to 4 rows per thread the sub-panel is factored in one
// workgroup's registers, beyond that by tournament pivoting
__host__ __device__ inline int gj_pbw(int n) { return (n > 4 * GJ_THREADS || n <= 2 * GJ_THREADS) ? GJB : 16; }
// how a job's sub-panels are factored: gj_panel_kernel with 1 to 4 rows per
// thread (0 ... 3) or 5 rows per thread of a half-size workgroup (4), or by
// tournament pivoting (5); a launch leaves the jobs of other variants alone
constexpr int GJ_VARIANTS = 6;
__host__ __device__ inline int gj_variant(int n) {
  return n > 4 * GJ_THREADS ? 5 : n > 2 * GJ_THREADS && n <= 5 * 256 ? 4 : (n - 1) / GJ_THREADS;
}
// the job's sub-panel at (c0, s0), if it has one: outer-panel width nbw, width B
__device__ __forceinline__ bool gj_step(int n, int c0, int s0, int& nbw, int& B) {
  if (c0 >= n) return false;
  nbw = min(GJ_NB, n - c0);
  const int pb = gj_pbw(n);
  if (s0 >= c0 + nbw || (s0 - c0) % pb) return false;
  B = min(pb, c0 + nbw - s0);
  return true;
}

// Inverse of the pivot block Mp = F[pr[a], b] (B x B, B <= PB), rows in
// pivot order, by Gauss-Jordan on [Mp | I] in LDS.  No pivot search: each
// pivot was the largest remaining entry of its column over all candidate
// rows, these rows included, so in pivot order the diagonal is the
// partial-pivoting choice.  Needs blockDim.x >= 2 B; 2 barriers per column.
template <int PB>
__device__ void pivot_block_inverse(int B, const double* __restrict__ F, const int* pr, double* __restrict__ Pinv,
                                    int* status, double (*Mp)[2 * PB], double* fr, double* rowc) {
  const int tid = threadIdx.x;
  for (int idx = tid; idx < B * B; idx += blockDim.x) {
    const int a = idx / B, b = idx % B;
    Mp[a][b] = F[(int64_t)pr[a] * B + b];
    Mp[a][B + b] = (a == b) ? 1.0 : 0.0;
  }
  __syncthreads();
  for (int c = 0; c < B; ++c) {
    const double piv = Mp[c][c];
    if (!(fabs(piv) > 0.0)) {
      if (tid == 0) atomicOr(status, SETUP_SINGULAR);
      return;  // uniform
    }
    if (tid < 2 * B) rowc[tid] = Mp[c][tid] / piv;
    if (tid < B) fr[tid] = Mp[tid][c];
    __syncthreads();
    for (int idx = tid; idx < B * 2 * B; idx += blockDim.x) {
      const int r = idx / (2 * B), cc = idx % (2 * B);
      Mp[r][cc] = (r == c) ? rowc[cc] : Mp[r][cc] - fr[r] * rowc[cc];
    }
    __syncthreads();
  }
  for (int idx = tid; idx < B * B; idx += blockDim.x) Pinv[idx] = Mp[idx / B][B + idx % B];
}

// Elimination with partial pivoting over the rows a workgroup holds in its
// registers: W[q][.] is the sub-panel window of row rid[q] (act[q]: still a
// candidate).  After each step the windows shift left by one, so the active
// column is always W[q][0] (all register indices static).  One barrier per
// column: every wavefront's best row publishes its value, index and window
// in LDS slots (double-buffered by column parity), and every wavefront picks
// the block's winner from the slots itself; ties go to the lowest row.
// Candidates are ordered by |entry|, then by the lower row; the order is
// total, so the winner does not depend on the order in which pairs are
// compared.  Inside a wavefront the comparisons run over DPP lane exchanges
// and scalar lane reads (no LDS round trips).
// on_pivot(jj, p) runs in the thread that holds the chosen row p; it writes
// LDS only, since a global store in the loop would hold up the next barrier
// (flat stores count against the LDS wait counter).
// strict: a column without a non-zero candidate makes the block singular
// (returns -1); otherwise such a column takes its lowest candidate row without
// elimination, and the loop ends early (returns the count) when no candidate
// rows are left.
constexpr int NWV = GJ_THREADS / 64;
static_assert(NWV == 8, "the slot reduction covers one group of 8 lanes");

// (ov, oi) beats (v, idx): a candidate (row >= 0) beats none, then the larger
// value, then the lower row
__device__ __forceinline__ bool cand_better(double ov, int oi, double v, int idx) {
  return oi >= 0 && (idx < 0 || ov > v || (ov == v && oi < idx));
}
template <int CTRL>
__device__ __forceinline__ void cand_step(double& v, int& idx, int& slot) {
  const double ov = dpp_t<CTRL>(v);
  const int oi = dpp_i<CTRL>(idx), os = dpp_i<CTRL>(slot);
  if (cand_better(ov, oi, v, idx)) { v = ov; idx = oi; slot = os; }
}
// the best of groups of 8 lanes in each of their lanes: xor 1, xor 2, then the
// half-row mirror (lane i <-> 7 - i) joins the two quads
__device__ __forceinline__ void cand_best8(double& v, int& idx, int& slot) {
  cand_step<0xB1>(v, idx, slot);
  cand_step<0x4E>(v, idx, slot);
  cand_step<0x141>(v, idx, slot);
}
// the best of lane `src` of the wavefront, in every lane
__device__ __forceinline__ void cand_read(double& v, int& idx, int& slot, int src) {
  v = read_lane(v, src);
  idx = __builtin_amdgcn_readlane(idx, src);
  slot = __builtin_amdgcn_readlane(slot, src);
}
// the best of the wavefront in every lane: rows of 16 lanes by DPP (groups of
// 8, then the row mirror lane i <-> 15 - i), then the four rows from scalar
// reads of lanes 0, 16, 32 and 48
__device__ __forceinline__ void cand_best64(double& v, int& idx, int& slot) {
  cand_best8(v, idx, slot);
  cand_step<0x140>(v, idx, slot);
  double bv = v;
  int bi = idx, bs = slot;
  cand_read(bv, bi, bs, 0);
#pragma unroll
  for (int r = 16; r < 64; r += 16) {
    double ov = v;
    int oi = idx, os = slot;
    cand_read(ov, oi, os, r);
    if (cand_better(ov, oi, bv, bi)) { bv = ov; bi = oi; bs = os; }
  }
  v = bv;
  idx = bi;
  slot = bs;
}

// NW: wavefronts of the workgroup (at most NWV)
template <int RPT, int PB, int NW, typename OnPivot>
__device__ int window_eliminate(double (&W)[RPT][PB], bool (&act)[RPT], const int (&rid)[RPT], int B, bool strict,
                                OnPivot on_pivot, double (*cv)[NWV], int (*ci)[NWV], double (*crow)[NWV][PB]) {
  static_assert(NW >= 1 && NW <= NWV, "one slot per wavefront");
  const int tid = threadIdx.x, wid = tid >> 6, lane = tid & 63;
#pragma unroll 1
  for (int jj = 0; jj < B; ++jj) {
    double v = -1.0;
    int idx = -1;
#pragma unroll
    for (int q = 0; q < RPT; ++q) {
      const double cand = fabs(W[q][0]);
      if (act[q] && (cand > v || (cand == v && rid[q] < idx))) { v = cand; idx = rid[q]; }
    }
    int unused = 0;
    cand_best64(v, idx, unused);
    const int par = jj & 1;
    bool mine = false;
#pragma unroll
    for (int q = 0; q < RPT; ++q) mine = mine || (act[q] && rid[q] == idx);
    if (lane == 0) {
      cv[par][wid] = v;
      ci[par][wid] = idx;
    }
    if (idx >= 0 && mine) {
#pragma unroll
      for (int q = 0; q < RPT; ++q)
        if (act[q] && rid[q] == idx) {
#pragma unroll
          for (int b = 0; b < PB; ++b) crow[par][wid][b] = W[q][b];
        }
    }
    __syncthreads();
    // lanes 0 .. NW - 1 take one slot each; the best of them, in every lane
    double bv = -1.0;
    int p = -1, pw = 0;
    if (lane < NW) {
      bv = cv[par][lane];
      p = ci[par][lane];
      pw = lane;
    }
    cand_best8(bv, p, pw);
    cand_read(bv, p, pw, 0);
    if (p < 0) return strict ? -1 : jj;  // uniform: no candidate rows left
    if (strict && !(bv > 0.0)) return -1;  // uniform: singular
#pragma unroll
    for (int q = 0; q < RPT; ++q)
      if (act[q] && rid[q] == p) {
        act[q] = false;
        on_pivot(jj, p);
      }
    const double* prw = crow[par][pw];
    const double ip = bv > 0.0 ? 1.0 / prw[0] : 0.0;
#pragma unroll
    for (int q = 0; q < RPT; ++q) {
      const double f = act[q] ? W[q][0] * ip : 0.0;
#pragma unroll
      for (int b = 1; b < PB; ++b) W[q][b - 1] = W[q][b] - f * prw[b];
      W[q][PB - 1] = 0.0;
    }
  }
  return B;
}

// Sub-panel factorisation (columns c0 .. c0 + B - 1) in one workgroup of NT
// threads.  Thread t owns rows t, t + NT, ... (RPT of them); n <= NT * RPT.
// A column costs every wavefront the same pivot search whatever its row
// count, so fewer, fuller wavefronts (NT = 256, 5 rows per thread) take less
// time per column than 512 threads with 3 rows each.
template <int RPT, int PB, int NT, class Jobs>
__global__ void __launch_bounds__(NT) gj_panel_kernel(Jobs jobs, int variant, int oc0, int c0) {
  const GJJob& jb = jobs.get();
  const int n = jb.n;
  int nbw_, B;
  if (gj_variant(n) != variant || !gj_step(n, oc0, c0, nbw_, B)) return;  // uniform
  double* __restrict__ M = jb.M;
  const double* __restrict__ F = jb.F;
  const double* __restrict__ Wc = jb.Wc;
  int* __restrict__ done = jb.done;
  int* __restrict__ prow = jb.prow;
  double* __restrict__ Pinv = jb.Pinv;
  int* status = jb.status;
  __shared__ double Mp[PB][2 * PB];
  __shared__ double fr[PB];
  __shared__ double rowc[2 * PB];
  __shared__ int pr[PB];
  __shared__ double cv[2][NWV];
  __shared__ int ci[2][NWV];
  __shared__ double crow[2][NWV][PB];
  const int tid = threadIdx.x;
  const int64_t w = 2 * (int64_t)n;
  double W[RPT][PB];
  bool act[RPT];
  int rid[RPT];
  // The sub-panel comes column-major from gj_fetch (Wc[b][i], F = its
  // row-major copy), so the loads of a wavefront are 64 consecutive rows.
  // Addresses are clamped and loaded unconditionally (all in flight at
  // once); window entries of rows i >= n or columns b >= B are never used
  // (such rows are inactive, and window positions at or beyond B - jj never
  // become the active column).
#pragma unroll
  for (int q = 0; q < RPT; ++q) {
    const int i = tid + q * NT;
    const bool ok = i < n;
    const int ic = ok ? i : 0;
    rid[q] = i;
    act[q] = !done[ic] && ok;
#pragma unroll
    for (int b = 0; b < PB; ++b) W[q][b] = Wc[(int64_t)(b < B ? b : B - 1) * n + ic];
  }
  // the pivots go to LDS during the elimination and to global memory after it
  // (a global store inside the column loop would hold up every barrier)
  const int got =
      window_eliminate<RPT, PB, NT / 64>(W, act, rid, B, true, [&](int jj, int p) { pr[jj] = p; }, cv, ci, crow);
  if (got < 0) {
    if (tid == 0) atomicOr(status, SETUP_SINGULAR);
    return;  // uniform
  }
  __syncthreads();  // pr[] complete
  pivot_block_inverse<PB>(B, F, pr, Pinv, status, Mp, fr, rowc);
  if (tid < B) {  // after the inverse's barriers, which would wait for these stores
    const int p = pr[tid];
    done[p] = 1;
    prow[c0 + tid] = p;
    M[(int64_t)p * w + n + c0 + tid] = 1.0;  // unit column of the new pivot
  }
}

// active column j (0 .. 2 nbw - 1) of the outer panel at c0
__device__ __forceinline__ int64_t gj_col(int n, int c0, int nbw, int j) {
  return j < nbw ? (int64_t)c0 + j : (int64_t)n + c0 + (j - nbw);
}

// R[a][j] = sum_b Pinv[a][b] M[prow[s0 + b]][col(j)] over the active columns
template <class Jobs>
__global__ void __launch_bounds__(256) gj_rows_kernel(Jobs jobs, int c0, int s0) {
  const GJJob& jb = jobs.get();
  const int n = jb.n;
  int nbw, B;
  if (!gj_step(n, c0, s0, nbw, B)) return;
  const double* __restrict__ M = jb.M;
  const int* __restrict__ prow = jb.prow;
  const double* __restrict__ Pinv = jb.Pinv;
  double* __restrict__ R = jb.R;
  const int64_t w = 2 * (int64_t)n;
  const int a = blockIdx.y;
  const int j = blockIdx.x * blockDim.x + threadIdx.x;
  if (a >= B || j >= 2 * nbw) return;
  const int64_t c = gj_col(n, c0, nbw, j);
  double mv[GJB];
#pragma unroll
  for (int b = 0; b < GJB; ++b) mv[b] = M[(int64_t)prow[s0 + (b < B ? b : B - 1)] * w + c];  // all loads at once
  double s = 0.0;
#pragma unroll
  for (int b = 0; b < GJB; ++b)
    if (b < B) s += Pinv[a * B + b] * mv[b];
  R[(int64_t)a * 2 * nbw + j] = s;
}

// Over the active columns: rows pivoted in this sub-panel become R, every
// other row i becomes M[i] - F[i, :] R.  Block: UPR rows x 256 columns.
constexpr int UPR = 8;
template <class Jobs>
__global__ void __launch_bounds__(256) gj_update_kernel(Jobs jobs, int c0, int s0) {
  const GJJob& jb = jobs.get();
  __shared__ double Fs[UPR][GJB];
  __shared__ int sub[UPR];  // sub-panel position of each row, or -1
  const int n = jb.n;
  int nbw, B;
  if (!gj_step(n, c0, s0, nbw, B)) return;  // uniform
  const int r0 = blockIdx.y * UPR;
  if (r0 >= n || blockIdx.x * 256 >= 2 * nbw) return;  // uniform, before the barriers
  double* __restrict__ M = jb.M;
  const double* __restrict__ F = jb.F;
  const double* __restrict__ R = jb.R;
  const int* __restrict__ prow = jb.prow;
  const int64_t w = 2 * (int64_t)n;
  const int j = blockIdx.x * 256 + threadIdx.x;
  for (int idx = threadIdx.x; idx < UPR * GJB; idx += 256) {
    const int rr = idx / GJB, b = idx % GJB;
    Fs[rr][b] = (r0 + rr < n && b < B) ? F[(int64_t)(r0 + rr) * B + b] : 0.0;
  }
  if (threadIdx.x < UPR) sub[threadIdx.x] = -1;
  __syncthreads();
  if (threadIdx.x < B) {
    const int pr = prow[s0 + threadIdx.x];
    if (pr >= r0 && pr < r0 + UPR) sub[pr - r0] = threadIdx.x;
  }
  __syncthreads();
  if (j >= 2 * nbw) return;
  const int64_t c = gj_col(n, c0, nbw, j);
  // unconditional clamped loads; entries b >= B meet zero padding in Fs and
  // are never selected as a pivot row's value
  double Rc[GJB];
#pragma unroll
  for (int b = 0; b < GJB; ++b) Rc[b] = R[(int64_t)(b < B ? b : B - 1) * 2 * nbw + j];
  // all rows' old values are loaded before the first store (each store would
  // otherwise complete before the next row's load is waited for)
  int sr[UPR];
#pragma unroll
  for (int rr = 0; rr < UPR; ++rr) sr[rr] = sub[rr];
  double old[UPR];
#pragma unroll
  for (int rr = 0; rr < UPR; ++rr) {
    const int i = r0 + rr;
    old[rr] = (i < n && sr[rr] < 0) ? M[(int64_t)i * w + c] : 0.0;
  }
#pragma unroll
  for (int rr = 0; rr < UPR; ++rr) {
    const int i = r0 + rr;
    if (i >= n) break;
    const int pi = sr[rr];
    double v;
    if (pi >= 0) {
      v = Rc[0];
#pragma unroll
      for (int b = 1; b < GJB; ++b)
        if (b == pi) v = Rc[b];
    } else {
      v = old[rr];
#pragma unroll
      for (int b = 0; b < GJB; ++b) v -= Fs[rr][b] * Rc[b];
    }
    M[(int64_t)i * w + c] = v;
  }
}

// ---- wide sub-panels (n > 4 GJ_THREADS): tournament pivoting -------------
// Beyond 4 rows per thread a sub-panel (B = GJB columns) no longer fits one
// workgroup's registers.  Its pivot rows are chosen by tournament pivoting
// (communication-avoiding LU, Grigori, Demmel and Xiang 2011) in two rounds:
//   gj_tourn0: each block of GJ_THREADS rows eliminates the sub-panel over its
//              own candidate rows and nominates the rows it pivoted on;
//   gj_tourn1: one workgroup eliminates the original sub-panel rows of all
//              nominees (at most 16 x GJB <= GJ_THREADS of them) and takes its
//              pivots as the sub-panel's, then inverts the pivot block.
// The pivots differ from column-by-column partial pivoting over all rows
// (each is the largest among the nominees); the inverse is the same up to
// rounding.  Two launches per sub-panel instead of one per column.

// F[i][b] = Wc[b][i] = M[i][s0 + b]
template <class Jobs>
__global__ void __launch_bounds__(256) gj_fetch_kernel(Jobs jobs, int c0, int s0) {
  const GJJob& jb = jobs.get();
  const int n = jb.n;
  int nbw, B;
  if (!gj_step(n, c0, s0, nbw, B)) return;
  const double* __restrict__ M = jb.M;
  double* __restrict__ F = jb.F;
  double* __restrict__ Wc = jb.Wc;
  const int64_t w = 2 * (int64_t)n;
  const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= (int64_t)n * B) return;
  const int i = (int)(idx / B), b = (int)(idx - (int64_t)i * B);
  const double v = M[(int64_t)i * w + s0 + b];
  F[idx] = v;
  Wc[(int64_t)b * n + i] = v;
}

template <class Jobs>
__global__ void __launch_bounds__(GJ_THREADS) gj_tourn0_kernel(Jobs jobs, int c0, int s0) {
  const GJJob& jb = jobs.get();
  __shared__ double cv[2][NWV];
  __shared__ int ci[2][NWV];
  __shared__ double crow[2][NWV][GJB];
  __shared__ int pv[GJB];  // the block's pivot rows (written to global memory after the elimination)
  const int n = jb.n;
  int nbw, B;
  if (gj_variant(n) != 5 || !gj_step(n, c0, s0, nbw, B)) return;  // uniform
  const double* __restrict__ Wc = jb.Wc;
  const int* __restrict__ done = jb.done;
  int* __restrict__ cand = jb.cand;
  const int i = blockIdx.x * GJ_THREADS + threadIdx.x;
  const bool ok = i < n;
  const int ic = ok ? i : 0;
  double W[1][GJB];
  bool act[1] = {!done[ic] && ok};
  const int rid[1] = {i};
#pragma unroll
  for (int b = 0; b < GJB; ++b) W[0][b] = Wc[(int64_t)(b < B ? b : B - 1) * n + ic];
  int* mine = cand + blockIdx.x * GJB;
  const int got =
      window_eliminate<1, GJB, NWV>(W, act, rid, B, false, [&](int jj, int p) { pv[jj] = p; }, cv, ci, crow);
  __syncthreads();  // pv[] complete
  for (int jj = threadIdx.x; jj < GJB; jj += blockDim.x) mine[jj] = jj < got ? pv[jj] : -1;
}

template <class Jobs>
__global__ void __launch_bounds__(GJ_THREADS) gj_tourn1_kernel(Jobs jobs, int c0, int s0) {
  const GJJob& jb = jobs.get();
  __shared__ double Mp[GJB][2 * GJB];
  __shared__ double fr[GJB];
  __shared__ double rowc[2 * GJB];
  __shared__ int pr[GJB];
  __shared__ double cv[2][NWV];
  __shared__ int ci[2][NWV];
  __shared__ double crow[2][NWV][GJB];
  const int n = jb.n;
  int nbw, B;
  if (gj_variant(n) != 5 || !gj_step(n, c0, s0, nbw, B)) return;  // uniform
  const int nblk = (n + GJ_THREADS - 1) / GJ_THREADS;
  double* __restrict__ M = jb.M;
  const double* __restrict__ F = jb.F;
  const int* __restrict__ cand = jb.cand;
  int* __restrict__ done = jb.done;
  int* __restrict__ prow = jb.prow;
  double* __restrict__ Pinv = jb.Pinv;
  int* status = jb.status;
  const int tid = threadIdx.x;
  const int64_t w = 2 * (int64_t)n;
  const int r = tid < nblk * GJB ? cand[tid] : -1;
  const int rc = r >= 0 ? r : 0;
  double W[1][GJB];
  bool act[1] = {r >= 0};
  const int rid[1] = {r >= 0 ? r : n + tid};  // distinct ids for empty slots (never active)
#pragma unroll
  for (int b = 0; b < GJB; ++b) W[0][b] = F[(int64_t)rc * B + (b < B ? b : B - 1)];
  const int got =
      window_eliminate<1, GJB, NWV>(W, act, rid, B, true, [&](int jj, int p) { pr[jj] = p; }, cv, ci, crow);
  if (got < 0) {
    if (tid == 0) atomicOr(status, SETUP_SINGULAR);
    return;  // uniform
  }
  __syncthreads();  // pr[] complete
  pivot_block_inverse<GJB>(B, F, pr, Pinv, status, Mp, fr, rowc);
  if (tid < B) {
    const int p = pr[tid];
    done[p] = 1;
    prow[s0 + tid] = p;
    M[(int64_t)p * w + n + s0 + tid] = 1.0;
  }
}

// Yo[i][k] = M[i][n + c0 + k] - [i == p_{c0+k}];  Rb[k][j] = M[p_{c0+k}][c0 + nbw + j]
template <class Jobs>
__global__ void __launch_bounds__(256) gj_gather_kernel(Jobs jobs, int c0) {
  const GJJob& jb = jobs.get();
  const int n = jb.n;
  if (c0 >= n) return;
  const int nbw = min(GJ_NB, n - c0);
  const double* __restrict__ M = jb.M;
  const int* __restrict__ prow = jb.prow;
  double* __restrict__ Yo = jb.Yo;
  double* __restrict__ Rb = jb.Rb;
  const int64_t w = 2 * (int64_t)n;
  const int64_t nr = n - nbw;
  const int64_t ny = (int64_t)n * nbw, nrb = (int64_t)nbw * nr;
  for (int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; idx < ny + nrb;
       idx += (int64_t)gridDim.x * blockDim.x) {
    if (idx < ny) {
      const int64_t i = idx / nbw;
      const int k = (int)(idx - i * nbw);
      Yo[idx] = M[i * w + n + c0 + k] - ((int)i == prow[c0 + k] ? 1.0 : 0.0);
    } else {
      const int64_t t = idx - ny;
      const int k = (int)(t / nr);
      const int64_t jj = t - (int64_t)k * nr;
      Rb[t] = M[(int64_t)prow[c0 + k] * w + c0 + nbw + jj];
    }
  }
}

// M[i][c0 + nbw + j] += sum_k Yo[i][k] Rb[k][j]  (i < n, j < n - nbw).
// 64 x 64 output tile per workgroup, 4 x 4 per thread, K staged in LDS by 16.
constexpr int GT = 64, GK = 16;
template <class Jobs>
__global__ void __launch_bounds__(256) gj_gemm_kernel(Jobs jobs, int c0) {
  const GJJob& jb = jobs.get();
  __shared__ double Ys[GK][GT + 1];
  __shared__ double Rs[GK][GT + 1];
  const int n = jb.n;
  if (c0 >= n) return;  // uniform
  const int nbw = min(GJ_NB, n - c0);
  const int nr = n - nbw;
  const int i0 = blockIdx.y * GT, j0 = blockIdx.x * GT;
  if (i0 >= n || j0 >= nr) return;  // uniform, before the barriers
  const double* __restrict__ Yo = jb.Yo;
  const double* __restrict__ Rb = jb.Rb;
  double* __restrict__ M = jb.M;
  const int64_t w = 2 * (int64_t)n;
  const int tx = threadIdx.x & 15, ty = threadIdx.x >> 4;
  double acc[4][4];
#pragma unroll
  for (int a = 0; a < 4; ++a)
#pragma unroll
    for (int b = 0; b < 4; ++b) acc[a][b] = 0.0;
  for (int k0 = 0; k0 < nbw; k0 += GK) {
    for (int idx = threadIdx.x; idx < GK * GT; idx += 256) {
      const int kk = idx % GK, ii = idx / GK;   // Yo: consecutive threads walk k
      const int i = i0 + ii, k = k0 + kk;
      Ys[kk][ii] = (i < n && k < nbw) ? Yo[(int64_t)i * nbw + k] : 0.0;
      const int jj = idx % GT, kr = idx / GT;   // Rb: consecutive threads walk j
      const int jc = j0 + jj, k2 = k0 + kr;
      Rs[kr][jj] = (jc < nr && k2 < nbw) ? Rb[(int64_t)k2 * nr + jc] : 0.0;
    }
    __syncthreads();
#pragma unroll
    for (int kk = 0; kk < GK; ++kk) {
      double a[4], b[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) { a[q] = Ys[kk][ty + 16 * q]; b[q] = Rs[kk][tx + 16 * q]; }
#pragma unroll
      for (int x = 0; x < 4; ++x)
#pragma unroll
        for (int y = 0; y < 4; ++y) acc[x][y] += a[x] * b[y];
    }
    __syncthreads();
  }
#pragma unroll
  for (int x = 0; x < 4; ++x) {
    const int i = i0 + ty + 16 * x;
    if (i >= n) continue;
#pragma unroll
    for (int y = 0; y < 4; ++y) {
      const int jc = j0 + tx + 16 * y;
      if (jc < nr) M[(int64_t)i * w + c0 + nbw + jc] += acc[x][y];
    }
  }
}

template <class Jobs>
__global__ void __launch_bounds__(256) gj_init_kernel(Jobs jobs) {
  const GJJob& jb = jobs.get();
  const int n = jb.n;
  const double* __restrict__ a = jb.a;
  double* __restrict__ M = jb.M;
  int* __restrict__ done = jb.done;
  int* __restrict__ prow = jb.prow;
  int* __restrict__ cand = jb.cand;
  const int64_t w = 2 * (int64_t)n;
  for (int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; idx < (int64_t)n * w;
       idx += (int64_t)gridDim.x * blockDim.x) {
    const int64_t i = idx / w, c = idx - i * w;
    M[idx] = (c < n) ? a[i * n + c] : 0.0;
    if (c == 0) {
      done[i] = 0;
      prow[i] = 0;  // any valid row until the pivot is chosen
      if (i < 16 * GJB) cand[i] = -1;
    }
  }
}

// A^-1[k][p_m] = M[p_k][n + m]
template <class Jobs>
__global__ void __launch_bounds__(256) gj_extract_kernel(Jobs jobs) {
  const GJJob& jb = jobs.get();
  const int n = jb.n;
  const double* __restrict__ M = jb.M;
  const int* __restrict__ prow = jb.prow;
  double* __restrict__ inv = jb.inv;
  const int64_t w = 2 * (int64_t)n;
  for (int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; idx < (int64_t)n * n;
       idx += (int64_t)gridDim.x * blockDim.x) {
    const int64_t k = idx / n, m = idx - k * n;
    inv[k * n + prow[m]] = M[(int64_t)prow[k] * w + n + m];
  }
}

// Scratch of one inversion, in doubles: the block elimination's two padded
// copies of the matrix, its diagonal-block inverses (2), its pivot row panel
// and the check's vector; the pivoted elimination lays its own buffers over
// the same memory.
static int64_t bgj_pad(int n) { return ((int64_t)n + BG - 1) / BG * BG; }
size_t dense_invert_work(int n) {
  const int64_t np = bgj_pad(n);
  // pivoted: M (2n^2), F and Wc (n*GJB each), R (GJB*2*GJ_NB), Pinv (GJB^2), Yo and Rb (n*GJ_NB each);
  // then 16*GJB tournament candidates and 2n ints
  const size_t pivoted = (size_t)(2 * (int64_t)n * n + 2 * (int64_t)n * GJB + 2 * (int64_t)GJB * GJ_NB + GJB * GJB +
                                  2 * (int64_t)n * GJ_NB) * sizeof(double) +
                         (size_t)(16 * GJB + 2 * n) * sizeof(int);
  const size_t block = (size_t)(2 * np * np + 2 * BG * BG + BG * np + np + 1) * sizeof(double);
  return std::max(pivoted, block);
}

GJJob gj_make_job(int n, const double* a, double* inv, double* work, int* status, int* rejected) {
  GJJob j;
  const int64_t np = bgj_pad(n);
  j.n = n;
  j.a = a;
  j.inv = inv;
  j.status = status;
  j.rejected = rejected;
  j.b0 = (double*)(((uintptr_t)work + 15) / 16 * 16);  // 16-byte loads
  j.b1 = j.b0 + np * np;
  j.dinv = j.b1 + np * np;
  j.rp = j.dinv + 2 * BG * BG;
  j.xv = j.rp + BG * np;
  j.M = work;
  j.F = j.M + 2 * (int64_t)n * n;
  j.Wc = j.F + (int64_t)n * GJB;
  j.R = j.Wc + (int64_t)n * GJB;
  j.Pinv = j.R + 2 * (int64_t)GJB * GJ_NB;
  j.Yo = j.Pinv + GJB * GJB;
  j.Rb = j.Yo + (int64_t)n * GJ_NB;
  j.cand = (int*)(j.Rb + (int64_t)GJ_NB * n);
  j.done = j.cand + 16 * GJB;
  j.prow = j.done + n;
  return j;
}

// Inversions with partial pivoting over all rows, for the matrices the block
// elimination's check rejects: jobs of sizes ns, n <= 16 GJ_THREADS
// (MVPF_MAX_COARSE_DOF).
template <class Jobs>
static int gj_run(const Jobs& jobs, const std::vector<int>& ns, hipStream_t s) {
  const int nj = (int)ns.size();
  const int nmax = *std::max_element(ns.begin(), ns.end());
  if (nmax > 16 * GJ_THREADS) return -1;  // at most 16 tournament blocks
  bool have[GJ_VARIANTS] = {};
  for (int n : ns) have[gj_variant(n)] = true;
  gj_init_kernel<<<dim3(1024, 1, nj), 256, 0, s>>>(jobs);
  for (int c0 = 0; c0 < nmax; c0 += GJ_NB) {
    for (int s0 = c0; s0 < std::min(nmax, c0 + GJ_NB); s0 += 16) {  // every sub-panel width is a multiple
      bool any = false;
      for (int n : ns) any = any || (c0 < n && s0 < std::min(n, c0 + GJ_NB) && (s0 - c0) % gj_pbw(n) == 0);
      if (!any) continue;
      gj_fetch_kernel<<<dim3((nmax * GJB + 255) / 256, 1, nj), 256, 0, s>>>(jobs, c0, s0);
      for (int v = 0; v < GJ_VARIANTS; ++v) {
        if (!have[v]) continue;
        const dim3 z(1, 1, nj);
        switch (v) {
          case 0: gj_panel_kernel<1, 32, GJ_THREADS><<<z, GJ_THREADS, 0, s>>>(jobs, v, c0, s0); break;
          case 1: gj_panel_kernel<2, 32, GJ_THREADS><<<z, GJ_THREADS, 0, s>>>(jobs, v, c0, s0); break;
          case 2: gj_panel_kernel<3, 16, GJ_THREADS><<<z, GJ_THREADS, 0, s>>>(jobs, v, c0, s0); break;
          case 3: gj_panel_kernel<4, 16, GJ_THREADS><<<z, GJ_THREADS, 0, s>>>(jobs, v, c0, s0); break;
          case 4: gj_panel_kernel<5, 16, 256><<<z, 256, 0, s>>>(jobs, v, c0, s0); break;
          default:
            gj_tourn0_kernel<<<dim3((nmax + GJ_THREADS - 1) / GJ_THREADS, 1, nj), GJ_THREADS, 0, s>>>(jobs, c0, s0);
            gj_tourn1_kernel<<<z, GJ_THREADS, 0, s>>>(jobs, c0, s0);
        }
      }
      gj_rows_kernel<<<dim3((2 * GJ_NB + 255) / 256, GJB, nj), 256, 0, s>>>(jobs, c0, s0);
      gj_update_kernel<<<dim3((2 * GJ_NB + 255) / 256, (nmax + UPR - 1) / UPR, nj), 256, 0, s>>>(jobs, c0, s0);
    }
    gj_gather_kernel<<<dim3(1024, 1, nj), 256, 0, s>>>(jobs, c0);
    gj_gemm_kernel<<<dim3((nmax + GT - 1) / GT, (nmax + GT - 1) / GT, nj), 256, 0, s>>>(jobs, c0);
  }
  gj_extract_kernel<<<dim3(1024, 1, nj), 256, 0, s>>>(jobs);
  return hipGetLastError() == hipSuccess ? 0 : -1;
}
int dense_invert_pivoted(const GJJob& job, hipStream_t s) { return gj_run(GJOne{job}, {job.n}, s); }
int dense_invert_pivoted_batch(const GJJob* tab_dev, const std::vector<int>& ns, hipStream_t s) {
  return ns.empty() ? 0 : gj_run(GJTab{tab_dev}, ns, s);
}

// ---- block elimination with pivoting inside the diagonal blocks -----------
// The matrix is a symmetric Hessian, near-definite: rows need not be searched
// over the whole matrix.  In-place Gauss-Jordan by blocks of BG = 64: with
// D = A_kk^-1 (partial pivoting inside the block), step k replaces
//   A_kj -> D A_kj,  A_ij -> A_ij - A_ik D A_kj,  A_ik -> -A_ik D,  A_kk -> D.
// Throughout, A_ij = A_ji^T where both or neither of i, j < k are eliminated and
// A_ij = -A_ji^T where one is: only the tiles i >= j are held and computed.
// A step is one launch over these tiles, reading one copy of the matrix and
// writing the other (every tile changes anyway); the workgroup of the next
// diagonal tile, the first of the launch, inverts it at once, beside the other
// tiles' products, so that the chain per 64 columns is one tile product and
// one block inversion.
//
// Stability is not assumed: the finished inverse is checked (bgj_check), and a
// matrix that fails is inverted again by the elimination with pivoting over
// all rows above.
//
// Bound: up to ~2000 unknowns the chain of block inversions (64 columns in
// registers, one barrier per column; 37 us per step, launch and tile products
// included), beyond that the tiles' traffic.  8 wavefronts per tile: the one
// that publishes the next column has half the columns to update after it
// (against 4 wavefronts: 1125 unknowns 0.81 -> 0.66 ms, 3645 4.2 -> 3.1 ms).
// Measured against four launches per 16 or 32 columns of the elimination
// above: 576 unknowns 2.07 -> 0.32 ms, 1125 4.23 -> 0.65, 2187 12.1 -> 1.6,
// 3645 22.7 -> 3.0 ms.
typedef double bg_vec4 __attribute__((ext_vector_type(4)));
constexpr int BGT = 512;  // threads of a tile's workgroup
constexpr int BG_LDA = 66, BG_LDB = 72;  // LDS strides: the matrix instructions' operand reads meet every bank evenly
// up to this many blocks a step forms D A_kj in every tile's workgroup; beyond,
// a launch of its own forms the row panel and the column panel once, and the
// tiles change in place (half the operations and less than half the traffic,
// one launch more per step).  The same sums either way.  A Newton system (us)
// with the one launch and with two: 576 unknowns 567 and 600, 1125 903 and 987;
// 2268 1732 and 1814; 3087 2610 and 2588, 4608 5680 and 4734, 6561 16.9 and 12.1
// ms.  Several at once fill the chip, and the operations count sooner: ten of
// 1125 2193 and 2268, of 1620 (26 blocks) 4157 and 3610, of 2268 8815 and 7370.
constexpr int BG_FUSED_MAX = 24;

// 64 x 64 x 64 product into acc: T1 (rows x k, stride BG_LDA) times T2 (k x
// columns, stride BG_LDB); 8 wavefronts, 32 x 16 each as two matrix
// instructions of 16 x 16 x 4 (lane l: A row l % 16, k l / 16; B k l / 16,
// column l % 16; result rows 4 r + l / 16, column l % 16)
__device__ __forceinline__ void bgj_product(const double* T1, const double* T2, bg_vec4 (&acc)[2]) {
  const int l = threadIdx.x & 63, w = threadIdx.x >> 6;
  const double* pa = T1 + (32 * (w >> 2) + (l & 15)) * BG_LDA + (l >> 4);
  const double* pb = T2 + (l >> 4) * BG_LDB + 16 * (w & 3) + (l & 15);
#pragma unroll
  for (int k = 0; k < 16; ++k) {
    const double a0 = pa[4 * k], a1 = pa[16 * BG_LDA + 4 * k];
    const double b0 = pb[4 * k * BG_LDB];
    acc[0] = __builtin_amdgcn_mfma_f64_16x16x4f64(a0, b0, acc[0], 0, 0, 0);
    acc[1] = __builtin_amdgcn_mfma_f64_16x16x4f64(a1, b0, acc[1], 0, 0, 0);
  }
}
// row and column of entry r of acc[x] in this lane
__device__ __forceinline__ int bgj_row(int x, int r) {
  return 32 * (threadIdx.x >> 8) + 16 * x + 4 * r + ((threadIdx.x & 63) >> 4);
}
__device__ __forceinline__ int bgj_col() { return 16 * ((threadIdx.x >> 6) & 3) + (threadIdx.x & 15); }

// a 64 x 64 tile from global memory (row stride ld) to LDS
template <int LD>
__device__ __forceinline__ void bgj_load(const double* __restrict__ src, int64_t ld, double* T) {
  double2 v[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int r = (threadIdx.x >> 5) + 16 * q, c = 2 * (threadIdx.x & 31);
    v[q] = *reinterpret_cast<const double2*>(src + (int64_t)r * ld + c);
  }
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int r = (threadIdx.x >> 5) + 16 * q, c = 2 * (threadIdx.x & 31);
    *reinterpret_cast<double2*>(T + r * LD + c) = v[q];
  }
}

// its transpose
template <int LD>
__device__ __forceinline__ void bgj_load_t(const double* __restrict__ src, int64_t ld, double* T) {
  double2 v[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int r = (threadIdx.x >> 5) + 16 * q, c = 2 * (threadIdx.x & 31);
    v[q] = *reinterpret_cast<const double2*>(src + (int64_t)r * ld + c);
  }
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int r = (threadIdx.x >> 5) + 16 * q, c = 2 * (threadIdx.x & 31);
    T[c * LD + r] = v[q].x;
    T[(c + 1) * LD + r] = v[q].y;
  }
}
// A_km (m != k) before step k, from the tiles held
template <int LD>
__device__ __forceinline__ void bgj_load_row(const double* __restrict__ M, int64_t np, int k, int m, double* T) {
  if (m < k)
    bgj_load<LD>(M + (int64_t)k * BG * np + m * BG, np, T);
  else
    bgj_load_t<LD>(M + (int64_t)m * BG * np + k * BG, np, T);
}
// |A_mk|: A_mk for m > k, -A_mk for m < k
template <int LD>
__device__ __forceinline__ void bgj_load_col(const double* __restrict__ M, int64_t np, int k, int m, double* T) {
  if (m > k)
    bgj_load<LD>(M + (int64_t)m * BG * np + k * BG, np, T);
  else
    bgj_load_t<LD>(M + (int64_t)k * BG * np + m * BG, np, T);
}
// tile b of the lower triangle, rows in turn
__device__ __forceinline__ void bgj_tile(int b, int& ti, int& tj) {
  ti = (int)((sqrtf(8.0f * b + 1.0f) - 1.0f) * 0.5f);
  while ((ti + 1) * (ti + 2) / 2 <= b) ++ti;
  while (ti * (ti + 1) / 2 > b) --ti;
  tj = b - ti * (ti + 1) / 2;
}

// 1 / x to rounding (two Newton steps from the hardware estimate; a zero gives
// inf or NaN, which the check finds)
__device__ __forceinline__ double bgj_reciprocal(double x) {
  double r = __builtin_amdgcn_rcp(x);
  r = __builtin_fma(r, __builtin_fma(-x, r, 1.0), r);
  return __builtin_fma(r, __builtin_fma(-x, r, 1.0), r);
}

// Inverse of the 64 x 64 block in T (stride BG_LDA) to out (row-major): in-place
// Gauss-Jordan in registers, lane = row, wavefront w holds columns 8 w .. 8 w
// + 7.  The pivot of a column is the largest of its remaining entries by the
// upper 30 bits of the magnitude (within 2^-19), ties to the lowest row; rows
// stay in place and the permutation is undone in the final store, which also
// takes the symmetric part (the tiles of the other triangle are never formed,
// so an asymmetry of D grows from step to step: on a random matrix of 1125
// unknowns, a tenth of its eigenvalues negative, the check's ratio is 2.7e-8
// without it and 7e-13 with it).  One barrier
// per column: the wavefront that holds the next column updates it first, finds
// its pivot and publishes column, pivot row and reciprocal before the rest of
// its update.  fb: 2 x 64 published columns, ipb: 2 reciprocals, pv: 128.
__device__ void bgj_invert(double* T, double* fb, double* ipb, int* pv, double* __restrict__ out, int* rejected) {
  const int l = threadIdx.x & 63, w = threadIdx.x >> 6;
  double a[8];
  __syncthreads();
#pragma unroll
  for (int j = 0; j < 8; ++j) a[j] = T[l * BG_LDA + 8 * w + j];
  bool act = true, bad = false;
  auto publish = [&](double v, int c) {  // column c, held by this wavefront
    const unsigned hi = (unsigned)(__builtin_bit_cast(unsigned long long, v) >> 32) & 0x7FFFFFFFu;
    const int key = act ? (int)(hi >> 1) + 1 : 0;
    int m = key;
    m = max(m, dpp_i<0xB1>(m));
    m = max(m, dpp_i<0x4E>(m));
    m = max(m, dpp_i<0x141>(m));
    m = max(m, dpp_i<0x140>(m));
    const int m0 = max(__builtin_amdgcn_readlane(m, 0), __builtin_amdgcn_readlane(m, 16));
    const int m1 = max(__builtin_amdgcn_readlane(m, 32), __builtin_amdgcn_readlane(m, 48));
    const int p = __ffsll((long long)__ballot(key == max(m0, m1))) - 1;
    const double piv = read_lane(v, p), ip = bgj_reciprocal(piv);
    bad = bad || !(fabs(piv) > 0.0);
    fb[64 * (c & 1) + l] = v;
    if (l == 0) {
      pv[c] = p;
      ipb[c & 1] = ip;
    }
  };
  if (w == 0) publish(a[0], 0);
#pragma unroll 1
  for (int wc = 0; wc < 8; ++wc) {
#pragma unroll
    for (int jc = 0; jc < 8; ++jc) {
      __syncthreads();
      const int c = 8 * wc + jc, jn = (jc + 1) & 7;
      const int p = __builtin_amdgcn_readfirstlane(pv[c]);
      const double fl = fb[64 * (jc & 1) + l], ip = ipb[jc & 1];
      const bool mine = l == p;
      act = act && !mine;
      // a - f ip a_p, and ip a_p in the pivot row: a keep - g a_p with the
      // broadcast entry as a scalar operand
      const double keep = mine ? 0.0 : 1.0, g = mine ? -ip : fl * ip;
      auto update = [&](int j) {
        const double s = read_lane(a[j], p);
        a[j] = __builtin_fma(-g, s, a[j] * keep);
      };
      update(jn);
      if (c + 1 < 64 && w == (jc == 7 ? wc + 1 : wc)) publish(a[jn], c + 1);
#pragma unroll
      for (int j = 0; j < 8; ++j)
        if (j != jn) update(j);
      if (w == wc) a[jc] = -g;
    }
  }
  if (bad && l == 0) atomicOr(rejected, 1);
  __syncthreads();  // pv complete
  // A^-1[c][p_m] sits in row p_c, column m
  int* pos = pv + 64;
  if (threadIdx.x < 64) pos[pv[threadIdx.x]] = threadIdx.x;
  __syncthreads();
  const int c = pos[l];
#pragma unroll
  for (int j = 0; j < 8; ++j) T[c * BG_LDA + pv[8 * w + j]] = a[j];
  __syncthreads();
  for (int idx = threadIdx.x; idx < BG * BG; idx += BGT) {
    const int r = idx >> 6, q = idx & 63;
    out[idx] = 0.5 * (T[r * BG_LDA + q] + T[q * BG_LDA + r]);
  }
}

// padded copy of the matrix's lower tiles (identity in the padding), the first block's inverse
template <class Jobs>
__global__ void __launch_bounds__(BGT) bgj_init_kernel(Jobs jobs) {
  __shared__ double T[BG * BG_LDA];
  __shared__ double fb[2 * BG], ipb[2];
  __shared__ int pv[2 * BG];
  const GJJob& jb = jobs.get();
  const int n = jb.n, nb = (n + BG - 1) / BG;
  int ti, tj;
  bgj_tile(blockIdx.x, ti, tj);
  if (ti >= nb) return;  // uniform
  const int64_t np = (int64_t)nb * BG;
  const bool first = ti == 0 && tj == 0;
  for (int idx = threadIdx.x; idx < BG * BG; idx += BGT) {
    const int r = idx >> 6, c = idx & 63, i = ti * BG + r, j = tj * BG + c;
    const double v = (i < n && j < n) ? jb.a[(int64_t)i * n + j] : (i == j ? 1.0 : 0.0);
    jb.b0[i * np + j] = v;
    if (first) T[r * BG_LDA + c] = v;
  }
  if (first) bgj_invert(T, fb, ipb, pv, jb.dinv, jb.rejected);
}

// panels of step k, tile m != k: rp_m = D A_km (64 x np), cp_m = |A_mk| (np x 64, in b1)
template <class Jobs>
__global__ void __launch_bounds__(BGT) bgj_panels_kernel(Jobs jobs, int k) {
  __shared__ double T1[BG * BG_LDA];
  __shared__ double T2[BG * BG_LDB];
  const GJJob& jb = jobs.get();
  const int nb = (jb.n + BG - 1) / BG, m = blockIdx.x;
  if (nb <= BG_FUSED_MAX || k >= nb || m >= nb || m == k) return;  // uniform
  const int64_t np = (int64_t)nb * BG;
  bgj_load<BG_LDA>(jb.dinv + (k & 1) * BG * BG, BG, T1);
  bgj_load_row<BG_LDB>(jb.b0, np, k, m, T2);
  __syncthreads();
  bg_vec4 acc[2] = {};
  bgj_product(T1, T2, acc);
#pragma unroll
  for (int x = 0; x < 2; ++x)
#pragma unroll
      for (int r = 0; r < 4; ++r) jb.rp[bgj_row(x, r) * np + m * BG + bgj_col()] = acc[x][r];
  // T2 holds A_km, of which |A_mk| is the transpose
  double* cp = jb.b1 + (int64_t)m * BG * BG;
  for (int idx = threadIdx.x; idx < BG * BG; idx += BGT) cp[idx] = T2[(idx & 63) * BG_LDB + (idx >> 6)];
}

template <bool FUSED, class Jobs>
__global__ void __launch_bounds__(BGT) bgj_step_kernel(Jobs jobs, int k) {
  __shared__ double T1[BG * BG_LDA];
  __shared__ double T2[BG * BG_LDB];
  __shared__ double fb[2 * BG], ipb[2];
  __shared__ int pv[2 * BG];
  const GJJob& jb = jobs.get();
  const int n = jb.n, nb = (n + BG - 1) / BG;
  if ((nb <= BG_FUSED_MAX) != FUSED || k >= nb) return;  // uniform
  int ti, tj;
  {  // the next diagonal tile's workgroup, which has most to do, comes first
    const int nx = (k + 1) * (k + 2) / 2 + k + 1, b = blockIdx.x;
    bgj_tile(k + 1 < nb && (b == 0 || b == nx) ? nx - b : b, ti, tj);
  }
  if (ti >= nb) return;  // uniform
  const int64_t np = (int64_t)nb * BG;
  const double* src = !FUSED || !(k & 1) ? jb.b0 : jb.b1;
  double* dst = !FUSED || (k & 1) ? jb.b0 : jb.b1;
  const double* __restrict__ D = jb.dinv + (k & 1) * BG * BG;
  const double* sij = src + (int64_t)ti * BG * np + tj * BG;
  bg_vec4 acc[2] = {}, old[2] = {};
  double sign = 1.0;  // result = sign * acc + old
  if (ti != k && tj != k) {  // the old tile, in flight during the products
#pragma unroll
    for (int x = 0; x < 2; ++x)
#pragma unroll
      for (int r = 0; r < 4; ++r) old[x][r] = sij[(int64_t)bgj_row(x, r) * np + bgj_col()];
  }
  if (ti == k && tj == k) {
#pragma unroll
    for (int x = 0; x < 2; ++x)
#pragma unroll
        for (int r = 0; r < 4; ++r) acc[x][r] = D[bgj_row(x, r) * BG + bgj_col()];
  } else if (tj == k) {
    bgj_load<BG_LDA>(sij, np, T1);
    bgj_load<BG_LDB>(D, BG, T2);
    __syncthreads();
    bgj_product(T1, T2, acc);
    sign = -1.0;
  } else if (!FUSED && ti == k) {
#pragma unroll
    for (int x = 0; x < 2; ++x)
#pragma unroll
        for (int r = 0; r < 4; ++r) acc[x][r] = jb.rp[bgj_row(x, r) * np + tj * BG + bgj_col()];
  } else {
    if (FUSED) {
      bgj_load<BG_LDA>(D, BG, T1);
      bgj_load_row<BG_LDB>(src, np, k, tj, T2);
      __syncthreads();
      bgj_product(T1, T2, acc);
    }
    if (ti != k) {
      if (FUSED) {
        __syncthreads();
#pragma unroll
        for (int x = 0; x < 2; ++x) {
#pragma unroll
          for (int r = 0; r < 4; ++r) T2[bgj_row(x, r) * BG_LDB + bgj_col()] = acc[x][r];
          acc[x] = bg_vec4{0.0, 0.0, 0.0, 0.0};
        }
        bgj_load_col<BG_LDA>(src, np, k, ti, T1);
      } else {
        bgj_load<BG_LDB>(jb.rp + tj * BG, np, T2);
        bgj_load<BG_LDA>(jb.b1 + (int64_t)ti * BG * BG, BG, T1);
      }
      __syncthreads();
      bgj_product(T1, T2, acc);
      sign = ti > k ? -1.0 : 1.0;
    }
  }
  const bool last = k == nb - 1, next = ti == k + 1 && tj == k + 1;
  if (next || last) __syncthreads();  // T1 is read no more
#pragma unroll
  for (int x = 0; x < 2; ++x)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int rr = bgj_row(x, r), cc = bgj_col();
        const double v = sign * acc[x][r] + old[x][r];
        if (!last) dst[((int64_t)ti * BG + rr) * np + tj * BG + cc] = v;
        if (next || last) T1[rr * BG_LDA + cc] = v;
      }
  if (next) bgj_invert(T1, fb, ipb, pv, jb.dinv + ((k + 1) & 1) * BG * BG, jb.rejected);
  if (!last) return;  // uniform
  __syncthreads();
  // the inverse, tile and transpose
  for (int idx = threadIdx.x; idx < BG * BG; idx += BGT) {
    const int r = idx >> 6, c = idx & 63;
    const int i = ti * BG + r, j = tj * BG + c, it = tj * BG + r, jt = ti * BG + c;
    if (i < n && j < n) jb.inv[(int64_t)i * n + j] = T1[r * BG_LDA + c];
    if (ti != tj && it < n && jt < n) jb.inv[(int64_t)it * n + jt] = T1[c * BG_LDA + r];
  }
}

// Check of the inverse X on one vector v of signs: x = X v, and in a second
// pass |A x - v| <= 1e-15 sqrt(n) (|A| |x| + 1) in every row.  Measured for the
// largest row of that ratio: 0.1 sqrt(n) 1e-15 on definite matrices of 1 to
// 3645 unknowns (0.2 with pivoting over all rows), below a quarter of the bound
// on two-level operators of up to 8100 unknowns and in 48 systems of running
// load sequences at 32^3; 2 to 27000 times sqrt(n) 1e-15 on random symmetric
// indefinite ones of 243 and more, where the block elimination loses digits,
// and 2 to 18 times on a slender column's operator of 1539 unknowns with 4 to 22
// negative eigenvalues.  Otherwise, or where anything is not
// finite, the matrix is marked for the elimination with pivoting over all rows.
__device__ __forceinline__ double bgj_sign(int j) { return (((unsigned)j * 2654435761u) >> 16) & 1 ? 1.0 : -1.0; }
template <class Jobs>
__global__ void __launch_bounds__(256) bgj_apply_kernel(Jobs jobs) {
  const GJJob& jb = jobs.get();
  const int row = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (row >= jb.n) return;
  const double* X = jb.inv + (int64_t)row * jb.n;
  double s = 0.0;
  for (int c = lane; c < jb.n; c += 64) s += X[c] * bgj_sign(c);
  for (int off = 32; off > 0; off >>= 1) s += __shfl_down(s, off, 64);
  if (lane == 0) jb.xv[row] = s;
}
template <class Jobs>
__global__ void __launch_bounds__(256) bgj_check_kernel(Jobs jobs) {
  const GJJob& jb = jobs.get();
  const int row = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (row >= jb.n) return;
  const double* A = jb.a + (int64_t)row * jb.n;
  double s = 0.0, m = 0.0;
  for (int c = lane; c < jb.n; c += 64) {
    const double t = A[c] * jb.xv[c];
    s += t;
    m += fabs(t);
  }
  for (int off = 32; off > 0; off >>= 1) {
    s += __shfl_down(s, off, 64);
    m += __shfl_down(m, off, 64);
  }
  if (lane == 0 && !(fabs(s - bgj_sign(row)) <= 1e-15 * sqrt((double)jb.n) * (m + 1.0))) atomicOr(jb.rejected, 1);
}

// Inversions of nj matrices (job table in device memory, or the one job by
// value), nmin to nmax unknowns: a job's `rejected` (zero before) is set where
// the result is to be replaced by the elimination with pivoting over all rows.
template <class Jobs>
static int bgj_run(const Jobs& jobs, int nj, int nmin, int nmax, hipStream_t s) {
  const int nb = (nmax + BG - 1) / BG;
  const bool some_fused = (nmin + BG - 1) / BG <= BG_FUSED_MAX;
  const auto tiles = [&](int b) { return dim3(b * (b + 1) / 2, 1, nj); };
  bgj_init_kernel<<<tiles(nb), BGT, 0, s>>>(jobs);
  for (int k = 0; k < nb; ++k) {  // a kernel leaves the other kind's jobs alone
    if (some_fused && k < BG_FUSED_MAX) bgj_step_kernel<true><<<tiles(std::min(nb, BG_FUSED_MAX)), BGT, 0, s>>>(jobs, k);
    if (nb > BG_FUSED_MAX) {
      bgj_panels_kernel<<<dim3(nb, 1, nj), BGT, 0, s>>>(jobs, k);
      bgj_step_kernel<false><<<tiles(nb), BGT, 0, s>>>(jobs, k);
    }
  }
  bgj_apply_kernel<<<dim3((nmax + 3) / 4, 1, nj), 256, 0, s>>>(jobs);
  bgj_check_kernel<<<dim3((nmax + 3) / 4, 1, nj), 256, 0, s>>>(jobs);
  return hipGetLastError() == hipSuccess ? 0 : -1;
}

int dense_invert(const GJJob& job, hipStream_t s) { return bgj_run(GJOne{job}, 1, job.n, job.n, s); }
// tab_dev: device table of the jobs of sizes ns
int dense_invert_batch(const GJJob* tab_dev, const std::vector<int>& ns, hipStream_t s) {
  if (ns.empty()) return 0;
  const auto [lo, hi] = std::minmax_element(ns.begin(), ns.end());
  return bgj_run(GJTab{tab_dev}, (int)ns.size(), *lo, *hi, s);
}

// x = Ainv b on the coarsest level; one wavefront per output unknown, FP64
// accumulation; b and x are level vectors (component-major, padded).  Bound by
// latency and reading Ainv once: CS_U entries in flight, the position in b
// carried along (a 64-bit division per entry, one entry at a time: 1944
// unknowns 20 -> 6.6 us, 3675 43 -> 27).
constexpr int CS_U = 8;
template <typename T>
__device__ __forceinline__ void coarse_solve_body(const Grid& g, const double* __restrict__ Ainv,
                                                  const T* __restrict__ b, T* __restrict__ x, int bid) {
  const int nd = NDOF * g.N;
  const int row = bid * 4 + (threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  if (row >= nd) return;
  double s = 0.0;
  const double* Ar = Ainv + (int64_t)row * nd;
  int node = lane, base = 0;  // entry c of b: b[base + node], base = component * Npad
  const auto wrap = [&] {
    while (node >= g.N) node -= g.N, base += g.Npad;
  };
  wrap();
  for (int c = lane; c < nd; c += 64 * CS_U) {
    double av[CS_U], bv[CS_U];
#pragma unroll
    for (int u = 0; u < CS_U; ++u) {
      const bool in = c + 64 * u < nd;
      av[u] = Ar[in ? c + 64 * u : c];
      bv[u] = in ? (double)b[in ? base + node : 0] : 0.0;
      node += 64;
      wrap();
    }
#pragma unroll
    for (int u = 0; u < CS_U; ++u) s += av[u] * bv[u];
  }
  for (int off = 32; off > 0; off >>= 1) s += __shfl_down(s, off, 64);
  if (lane == 0) {
    const int comp = row / g.N, node = row - comp * g.N;
    x[(int64_t)comp * g.Npad + node] = (T)s;
  }
}
template <typename T>
__global__ void __launch_bounds__(256) coarse_solve_kernel(Grid g, const double* __restrict__ Ainv,
                                                           const T* __restrict__ b, T* __restrict__ x) {
  coarse_solve_body<T>(g, Ainv, b, x, blockIdx.x);
}
template <typename T>
__global__ void __launch_bounds__(256) coarse_solve_batch(const BJob* __restrict__ jobs, int njobs) {
  int bid;
  const BJob& j = find_job(jobs, njobs, bid);
  coarse_solve_body<T>(j.g, (const double*)j.A, (const T*)j.b, (T*)j.y, bid);
}

template <typename T>
void launch_coarse_solve(const Grid& g, const double* Ainv, const T* b, T* x, hipStream_t s) {
  const int64_t nd = (int64_t)NDOF * g.N;
  coarse_solve_kernel<T><<<(int)((nd + 3) / 4), 256, 0, s>>>(g, Ainv, b, x);
}
template void launch_coarse_solve<float>(const Grid&, const double*, const float*, float*, hipStream_t);
template void launch_coarse_solve<double>(const Grid&, const double*, const double*, double*, hipStream_t);

template <typename T>
void launch_coarse_solve_batch(const BJob* jobs, int njobs, int blocks, hipStream_t s) {
  coarse_solve_batch<T><<<blocks, 256, 0, s>>>(jobs, njobs);
}
template void launch_coarse_solve_batch<float>(const BJob*, int, int, hipStream_t);
template void launch_coarse_solve_batch<double>(const BJob*, int, int, hipStream_t);

}  // namespace mvpf
