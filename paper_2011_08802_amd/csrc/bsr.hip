// 9x9-block operator kernels on the structured 27-point stencil.
//
// One thread per node row.  The operator is stored as symmetric half stencil,
// tiled structure-of-arrays (64 rows per tile, see common.h), so each operator
// load of a row is a fully coalesced 64-lane access (256 B in FP32, 512 B in
// FP64); vectors are component-major, so the 9 values of each neighbour are
// coalesced loads as well.  These kernels are HBM-bandwidth bound: per row
// they move 14*81*sizeof(TA) bytes of operator plus ~10 vector values, and
// 2*13*9 accumulation values for the transposed lower half.
#include "common.h"

namespace mvpf {

template <typename T>
struct Acc;
template <>
struct Acc<float> { using type = float; };
template <>
struct Acc<double> { using type = double; };

// Launch shape of the row kernels.  nb = ceil(Npad / 256) logical blocks of
// 256 rows.  With G = gridDim.x workgroups (a multiple of 8), workgroup b
// (which the hardware places on XCD b % 8) handles logical blocks
// L = r*G + (b % 8)*(G/8) + b/8 for rounds r = 0, 1, ...: within a round each
// XCD walks a contiguous range of rows, and only G*256 rows are in flight, so
// the transposed lower-half reads of neighbouring rows hit L2 / the infinity
// cache.  G >= nb is the plain one-block-per-256-rows launch.
__host__ __device__ inline int row_blocks(const Grid& g) { return (g.Npad + 255) / 256; }
inline int row_grid(const Grid& g, int G) {
  const int nb_pad = (row_blocks(g) + 7) / 8 * 8;
  if (G <= 0 || G >= nb_pad) return nb_pad;
  return std::max(8, G / 8 * 8);
}

// ROW_LOOP_B: the same for workgroup bid of nblk (a job of a batched launch)
#define ROW_LOOP_B(g, bid, nblk)                                                   \
  const int nb_ = row_blocks(g);                                                  \
  const int per_ = (nblk) >> 3;                                                    \
  for (int L_ = ((bid) & 7) * per_ + ((bid) >> 3); L_ < nb_; L_ += (nblk))         \
    for (int n = L_ * 256 + threadIdx.x, once_ = 1; once_; once_ = 0)
#define ROW_LOOP(g) ROW_LOOP_B(g, (int)blockIdx.x, (int)gridDim.x)

// Symmetric product in two passes, so that every stored block is read from
// memory exactly once whatever the cache does:
//  pass 1 (row n): acc_n (-)= sum_u A_u(n) x(n + off_u) over the 14 stored
//    blocks, and for the 13 off-diagonal ones the transposed contribution
//    A_u(n)^T x(n) to row m = n + off_u is written to C[u-1][.][m] (each
//    (u, m) has exactly one writer; lanes write consecutive m);
//  pass 2 (row m): acc_m (-)= sum_u C[u-1][.][m] over the in-grid lower
//    neighbours, then the kernel's epilogue (defect, Jacobi update, product).
// C holds 13 * NDOF * Npad values of the accumulation type.
// Stored blocks u0 .. u1 - 1 of row n (see upper_pass).
template <bool SUB, typename TA, typename TX, typename TC>
__device__ __forceinline__ void upper_range(const Grid& g, const TA* __restrict__ A, const TX* __restrict__ x, int n,
                                            int u0, int u1, TC acc[NDOF], TC* __restrict__ C) {
  const int t = n >> 6, l = n & 63;
  const int i = n % g.nnx, j = (n / g.nnx) % g.nny, k = n / (g.nnx * g.nny);
  TC xn[NDOF];
#pragma unroll
  for (int c = 0; c < NDOF; ++c) xn[c] = (TC)x[(int64_t)c * g.Npad + n];
#pragma unroll 1
  for (int u = u0; u < u1; ++u) {
    const int s = 13 + u;
    const int dx = s % 3 - 1, dy = (s / 3) % 3 - 1, dz = s / 9 - 1;
    if (!((i + dx >= 0) && (i + dx < g.nnx) && (j + dy >= 0) && (j + dy < g.nny) && (k + dz < g.nnz))) continue;
    const int m = n + dx + g.nnx * (dy + g.nny * dz);
    TC xv[NDOF];
#pragma unroll
    for (int c = 0; c < NDOF; ++c) xv[c] = (TC)x[(int64_t)c * g.Npad + m];
    using VT = typename Vec16<TA>::type;
    constexpr int V = Lay<TA>::V;
    const VT* Ab = reinterpret_cast<const VT*>(A + ((int64_t)t * NUP + u) * Lay<TA>::SLICE) + l;
    TC ct[NDOF] = {};
    TC sum[NDOF] = {};
#pragma unroll
    for (int q = 0; q < Lay<TA>::NQ; ++q) {
      const VT vq = Ab[q * TILE];
      TA av[V];
      __builtin_memcpy(av, &vq, sizeof(VT));
#pragma unroll
      for (int v = 0; v < V; ++v) {
        const int e = q * V + v;
        if (e < NBLK) {
          const int r = e / NDOF, c = e % NDOF;
          const TC a = (TC)av[v];
          sum[r] += a * xv[c];
          ct[c] += a * xn[r];
        }
      }
    }
#pragma unroll
    for (int r = 0; r < NDOF; ++r) {
      if (SUB) acc[r] -= sum[r]; else acc[r] += sum[r];
    }
    if (u > 0) {
      TC* Cu = C + (int64_t)(u - 1) * NDOF * g.Npad + m;
#pragma unroll
      for (int c = 0; c < NDOF; ++c) Cu[(int64_t)c * g.Npad] = ct[c];
    }
  }
}

// The 14 stored blocks are summed in two halves, u < USPLIT into acc and
// u >= USPLIT into a separate partial that is then added (or subtracted):
// the split kernels give each half its own wavefront, and every kernel
// family uses this same order, so results do not depend on the launch shape.
constexpr int USPLIT = 7;

template <bool SUB, typename TA, typename TX, typename TC>
__device__ __forceinline__ void upper_pass(const Grid& g, const TA* __restrict__ A, const TX* __restrict__ x, int n,
                                           TC acc[NDOF], TC* __restrict__ C) {
  upper_range<SUB>(g, A, x, n, 0, USPLIT, acc, C);
  TC p1[NDOF] = {};
  upper_range<false>(g, A, x, n, USPLIT, NUP, p1, C);
#pragma unroll
  for (int r = 0; r < NDOF; ++r) {
    if (SUB) acc[r] -= p1[r]; else acc[r] += p1[r];
  }
}

template <bool SUB, typename TC>
__device__ __forceinline__ void lower_pass(const Grid& g, int m, TC acc[NDOF], const TC* __restrict__ C) {
  const int i = m % g.nnx, j = (m / g.nnx) % g.nny, k = m / (g.nnx * g.nny);
#pragma unroll
  for (int u = 1; u < NUP; ++u) {
    const int s = 13 + u;
    const int dx = s % 3 - 1, dy = (s / 3) % 3 - 1, dz = s / 9 - 1;
    if (!((i - dx >= 0) && (i - dx < g.nnx) && (j - dy >= 0) && (j - dy < g.nny) && (k - dz >= 0))) continue;
    const TC* Cu = C + (int64_t)(u - 1) * NDOF * g.Npad + m;
#pragma unroll
    for (int c = 0; c < NDOF; ++c) {
      if (SUB) acc[c] -= Cu[(int64_t)c * g.Npad]; else acc[c] += Cu[(int64_t)c * g.Npad];
    }
  }
}

// y = A x: pass 1 writes the upper part into y, pass 2 adds the lower part.
template <typename TA, typename TX, typename TY>
__global__ void __launch_bounds__(256) spmv_upper_kernel(Grid g, const TA* __restrict__ A, const TX* __restrict__ x,
                                                         TY* __restrict__ y, TY* __restrict__ C) {
  ROW_LOOP(g) {
    if (n >= g.Npad) continue;
    TY acc[NDOF] = {};
    if (n < g.N) upper_pass<false>(g, A, x, n, acc, C);
#pragma unroll
    for (int r = 0; r < NDOF; ++r) y[(int64_t)r * g.Npad + n] = acc[r];
  }
}

template <typename TY>
__global__ void __launch_bounds__(256) spmv_lower_kernel(Grid g, TY* __restrict__ y, const TY* __restrict__ C) {
  ROW_LOOP(g) {
    if (n >= g.N) continue;
    TY acc[NDOF];
#pragma unroll
    for (int r = 0; r < NDOF; ++r) acc[r] = y[(int64_t)r * g.Npad + n];
    lower_pass<false>(g, n, acc, C);
#pragma unroll
    for (int r = 0; r < NDOF; ++r) y[(int64_t)r * g.Npad + n] = acc[r];
  }
}

// Pass 1 with the two halves of each tile's blocks on two wavefronts: a
// workgroup = 2 tiles x 2 halves; the second half's partial row sums go
// through LDS to the first, which finishes the row (same order as
// upper_pass).  Twice as many, shorter wavefronts as the one-wave kernels.
__device__ __forceinline__ int split_tile(int b, int nb_pad) {
  const int per = nb_pad >> 3;
  return ((b & 7) * per + (b >> 3)) * 2;  // first tile of logical block (XCD-contiguous)
}
inline int split_grid(const Grid& g) { return ((g.ntiles + 1) / 2 + 7) / 8 * 8; }

template <typename TA, typename TX, typename TY>
__global__ void __launch_bounds__(256) spmv_upper_split_kernel(Grid g, const TA* __restrict__ A,
                                                               const TX* __restrict__ x, TY* __restrict__ y,
                                                               TY* __restrict__ C) {
  __shared__ TY sh[2][NDOF][64];
  const int w = threadIdx.x >> 6, l = threadIdx.x & 63, tl = w >> 1, half = w & 1;
  const int t = split_tile(blockIdx.x, gridDim.x) + tl;
  const int n = t * TILE + l;
  const bool valid = t < g.ntiles;
  TY acc[NDOF] = {};
  if (valid && n < g.N) upper_range<false>(g, A, x, n, half ? USPLIT : 0, half ? NUP : USPLIT, acc, C);
  if (half) {
#pragma unroll
    for (int r = 0; r < NDOF; ++r) sh[tl][r][l] = acc[r];
  }
  __syncthreads();
  if (!half && valid) {
#pragma unroll
    for (int r = 0; r < NDOF; ++r) y[(int64_t)r * g.Npad + n] = acc[r] + sh[tl][r][l];
  }
}

// ---- small grids --------------------------------------------------------------
// On coarse levels the one-thread-per-row kernels are latency bound (27 rounds
// of dependent loads per thread).  Here 27 threads share a row, one per
// stencil block; each does one round of loads and the 27 partial products are
// summed through LDS in a fixed order.  SMALL_ROWS rows per workgroup, thread
// index = s * SMALL_ROWS + local row, so a load takes the 16-byte words of 8
// consecutive rows, a cache line; up to SMALL_CHUNK of them and the epilogue's
// operands are in flight together.  A row reads the 13 blocks below its
// diagonal from its neighbours' rows; consecutive workgroups share an XCD
// (ROW_LOOP's numbering), so these come from its L2.
// Per sweep, before (9 rows, scalar loads, workgroups dealt to all XCDs) and
// now: FP64 9261 nodes 41.6 -> 23.3 us (85 MB of operator: 3.6 TB/s), 1331
// nodes 9.8 -> 5.4, 125 nodes 6.0 -> 4.7; FP32 4913 nodes 16.2 -> 7.5 us.
constexpr int SMALL_ROWS = 8;
constexpr int SMALL_CHUNK = 21;  // 16-byte loads in flight per thread (an FP32 block of 9 x 9; half an FP64 one)
#define SMALL_OCC __attribute__((amdgpu_waves_per_eu(3, 3)))  // registers for them
constexpr int SMALL_THREADS = (SMALL_ROWS * NSTEN + 63) / 64 * 64;
// the padding included (a product leaves zeros there)
static int small_blocks(const Grid& g) { return (g.Npad / SMALL_ROWS + 7) / 8 * 8; }
static_assert(TILE % SMALL_ROWS == 0);

enum RowMode { ROW_PRODUCT, ROW_DEFECT, ROW_PBJ };  // out = A x, b - A x, x + omega Dinv (b - A x)
template <typename TA, typename TX, typename T, RowMode MODE>
__device__ __forceinline__ void row_small_body(const Grid& g, const TA* __restrict__ A, const T* __restrict__ Dinv,
                                               const TX* __restrict__ x, const T* __restrict__ b,
                                               T* __restrict__ out, T omega, int bid, int nblk) {
  constexpr bool PBJ = MODE == ROW_PBJ;
  __shared__ T part[SMALL_ROWS][NSTEN][NDOF];
  __shared__ T res[SMALL_ROWS][NDOF];
  using VT = typename Vec16<TA>::type;
  constexpr int V = Lay<TA>::V;
  const int tid = threadIdx.x;
  const int s = tid / SMALL_ROWS, ln = tid % SMALL_ROWS;
  const int n0 = ((bid & 7) * (nblk >> 3) + (bid >> 3)) * SMALL_ROWS;
  const int n = n0 + ln;
  // the epilogue's operands (thread = local row x component), in flight from the start
  const int ln2 = tid / NDOF, r2 = tid % NDOF;
  const int n2 = n0 + ln2;
  const bool own = tid < SMALL_ROWS * NDOF && n2 < g.N;
  T b2 = 0, x2 = 0, d2[NDOF];
  if (own) {
    if (MODE != ROW_PRODUCT) b2 = b[(int64_t)r2 * g.Npad + n2];
    if (PBJ) {
      x2 = (T)x[(int64_t)r2 * g.Npad + n2];
      const T* Db = Dinv + (int64_t)(n2 >> 6) * Lay<T>::SLICE;
#pragma unroll
      for (int c = 0; c < NDOF; ++c) d2[c] = Db[Lay<T>::off(r2 * NDOF + c, n2 & 63)];
    }
  }
  T pr[NDOF] = {};
  if (s < NSTEN && n < g.N) {
    const int i = n % g.nnx, j = (n / g.nnx) % g.nny, k = n / (g.nnx * g.nny);
    const int dx = s % 3 - 1, dy = (s / 3) % 3 - 1, dz = s / 9 - 1;
    if (i + dx >= 0 && i + dx < g.nnx && j + dy >= 0 && j + dy < g.nny && k + dz >= 0 && k + dz < g.nnz) {
      const int m = n + dx + g.nnx * (dy + g.nny * dz);
      T xv[NDOF];
#pragma unroll
      for (int c = 0; c < NDOF; ++c) xv[c] = (T)x[(int64_t)c * g.Npad + m];
      const bool upper = s >= 13;
      const int o = upper ? n : m;  // the row that stores the block
      const VT* Ab =
          reinterpret_cast<const VT*>(A + ((int64_t)(o >> 6) * NUP + (upper ? s - 13 : 13 - s)) * Lay<TA>::SLICE) +
          (o & 63);
#pragma unroll
      for (int q0 = 0; q0 < Lay<TA>::NQ; q0 += SMALL_CHUNK) {
        VT vq[SMALL_CHUNK];
#pragma unroll
        for (int q = 0; q < SMALL_CHUNK; ++q)
          if (q0 + q < Lay<TA>::NQ) vq[q] = Ab[(q0 + q) * TILE];
        // one branch per chunk: the stored block, or its transpose
        auto add = [&](auto up) {
#pragma unroll
          for (int q = 0; q < SMALL_CHUNK; ++q) {
            TA av[V];
            __builtin_memcpy(av, &vq[q], sizeof(VT));
#pragma unroll
            for (int v = 0; v < V; ++v) {
              const int e = (q0 + q) * V + v;
              if (e < NBLK) {
                const int r = e / NDOF, c = e % NDOF;
                pr[up.value ? r : c] += (T)av[v] * xv[up.value ? c : r];
              }
            }
          }
        };
        if (upper) add(std::true_type{}); else add(std::false_type{});
      }
    }
  }
  if (s < NSTEN)
#pragma unroll
    for (int r = 0; r < NDOF; ++r) part[ln][s][r] = pr[r];
  __syncthreads();
  if (own) {
    T acc = b2;
#pragma unroll
    for (int ss = 0; ss < NSTEN; ++ss) acc += MODE == ROW_PRODUCT ? part[ln2][ss][r2] : -part[ln2][ss][r2];
    if (PBJ)
      res[ln2][r2] = acc;
    else
      out[(int64_t)r2 * g.Npad + n2] = acc;
  }
  if (MODE == ROW_PRODUCT && tid < SMALL_ROWS * NDOF && n2 >= g.N && n2 < g.Npad) out[(int64_t)r2 * g.Npad + n2] = 0;
  if (!PBJ) return;
  __syncthreads();
  if (own) {
    T acc = 0;
#pragma unroll
    for (int c = 0; c < NDOF; ++c) acc += d2[c] * res[ln2][c];
    out[(int64_t)r2 * g.Npad + n2] = x2 + omega * acc;
  }
}
template <typename TA, typename TX, typename T, RowMode MODE>
__global__ void __launch_bounds__(SMALL_THREADS) SMALL_OCC
    row_small_kernel(Grid g, const TA* __restrict__ A, const T* __restrict__ Dinv, const TX* __restrict__ x,
                     const T* __restrict__ b, T* __restrict__ out, T omega) {
  row_small_body<TA, TX, T, MODE>(g, A, Dinv, x, b, out, omega, blockIdx.x, gridDim.x);
}

template <typename T>
void launch_row_small(const Grid& g, const T* A, const T* Dinv, const T* x, const T* b, T* out, T omega, bool pbj,
                      hipStream_t s) {
  const int nb = small_blocks(g);
  if (pbj)
    row_small_kernel<T, T, T, ROW_PBJ><<<nb, SMALL_THREADS, 0, s>>>(g, A, Dinv, x, b, out, omega);
  else
    row_small_kernel<T, T, T, ROW_DEFECT><<<nb, SMALL_THREADS, 0, s>>>(g, A, Dinv, x, b, out, omega);
}
template void launch_row_small<float>(const Grid&, const float*, const float*, const float*, const float*, float*,
                                      float, bool, hipStream_t);
template void launch_row_small<double>(const Grid&, const double*, const double*, const double*, const double*,
                                       double*, double, bool, hipStream_t);

// ---- products -------------------------------------------------------------------
template <typename TA, typename TX, typename TY>
void launch_spmv(const Grid& g, const TA* A, const TX* x, TY* y, void* C, hipStream_t s, int small_nodes, int G) {
  // FP64, 15 unknowns per node, 10648 nodes: 508 us in two passes (one thread per
  // row, 42 workgroups), 95 here (270 MB of operator)
  if (g.N <= small_nodes) {
    row_small_kernel<TA, TX, TY, ROW_PRODUCT><<<small_blocks(g), SMALL_THREADS, 0, s>>>(g, A, nullptr, x, nullptr, y,
                                                                                       (TY)0);
    return;
  }
  const int nb = row_grid(g, G);
  // FP64 operators keep one wavefront per tile (2 waves per SIMD fit either
  // way and the split measured slower); FP32 ones split
  if (G <= 0 && sizeof(TA) == 4)
    spmv_upper_split_kernel<TA, TX, TY><<<split_grid(g), 256, 0, s>>>(g, A, x, y, (TY*)C);
  else
    spmv_upper_kernel<TA, TX, TY><<<nb, 256, 0, s>>>(g, A, x, y, (TY*)C);
  spmv_lower_kernel<TY><<<nb, 256, 0, s>>>(g, y, (const TY*)C);
}
template void launch_spmv<double, double, double>(const Grid&, const double*, const double*, double*, void*,
                                                  hipStream_t, int, int);
template void launch_spmv<double, float, double>(const Grid&, const double*, const float*, double*, void*,
                                                 hipStream_t, int, int);
template void launch_spmv<float, float, float>(const Grid&, const float*, const float*, float*, void*, hipStream_t,
                                               int, int);

// r = b - A x
template <typename T>
__global__ void __launch_bounds__(256) defect_upper_kernel(Grid g, const T* __restrict__ A, const T* __restrict__ x,
                                                           const T* __restrict__ b, T* __restrict__ r,
                                                           T* __restrict__ C) {
  ROW_LOOP(g) {
    if (n >= g.Npad) continue;
    T acc[NDOF];
#pragma unroll
    for (int c = 0; c < NDOF; ++c) acc[c] = b[(int64_t)c * g.Npad + n];
    if (n < g.N) upper_pass<true>(g, A, x, n, acc, C);
#pragma unroll
    for (int c = 0; c < NDOF; ++c) r[(int64_t)c * g.Npad + n] = (n < g.N) ? acc[c] : (T)0;
  }
}

template <typename T>
__device__ __forceinline__ void defect_lower_body(const Grid& g, T* __restrict__ r, const T* __restrict__ C, int bid,
                                                  int nblk) {
  ROW_LOOP_B(g, bid, nblk) {
    if (n >= g.N) continue;
    T acc[NDOF];
#pragma unroll
    for (int c = 0; c < NDOF; ++c) acc[c] = r[(int64_t)c * g.Npad + n];
    lower_pass<true>(g, n, acc, C);
#pragma unroll
    for (int c = 0; c < NDOF; ++c) r[(int64_t)c * g.Npad + n] = acc[c];
  }
}
template <typename T>
__global__ void __launch_bounds__(256) defect_lower_kernel(Grid g, T* __restrict__ r, const T* __restrict__ C) {
  defect_lower_body<T>(g, r, C, blockIdx.x, gridDim.x);
}

template <typename T>
__device__ __forceinline__ void defect_upper_split_body(const Grid& g, const T* __restrict__ A,
                                                        const T* __restrict__ x, const T* __restrict__ b,
                                                        T* __restrict__ r, T* __restrict__ C, int bid, int nblk) {
  __shared__ T sh[2][NDOF][64];
  const int w = threadIdx.x >> 6, l = threadIdx.x & 63, tl = w >> 1, half = w & 1;
  const int t = split_tile(bid, nblk) + tl;
  const int n = t * TILE + l;
  const bool valid = t < g.ntiles;
  T acc[NDOF] = {};
  if (valid && !half) {
#pragma unroll
    for (int c = 0; c < NDOF; ++c) acc[c] = b[(int64_t)c * g.Npad + n];
  }
  if (valid && n < g.N) {
    if (half)
      upper_range<false>(g, A, x, n, USPLIT, NUP, acc, C);
    else
      upper_range<true>(g, A, x, n, 0, USPLIT, acc, C);
  }
  if (half) {
#pragma unroll
    for (int c = 0; c < NDOF; ++c) sh[tl][c][l] = acc[c];
  }
  __syncthreads();
  if (!half && valid) {
#pragma unroll
    for (int c = 0; c < NDOF; ++c) r[(int64_t)c * g.Npad + n] = (n < g.N) ? acc[c] - sh[tl][c][l] : (T)0;
  }
}
template <typename T>
__global__ void __launch_bounds__(256) defect_upper_split_kernel(Grid g, const T* __restrict__ A,
                                                                 const T* __restrict__ x, const T* __restrict__ b,
                                                                 T* __restrict__ r, T* __restrict__ C) {
  defect_upper_split_body<T>(g, A, x, b, r, C, blockIdx.x, gridDim.x);
}

template <typename T>
void launch_defect(const Grid& g, const T* A, const T* x, const T* b, T* r, void* C, hipStream_t s, int G) {
  const int nb = row_grid(g, G);
  if (G <= 0)
    defect_upper_split_kernel<T><<<split_grid(g), 256, 0, s>>>(g, A, x, b, r, (T*)C);
  else
    defect_upper_kernel<T><<<nb, 256, 0, s>>>(g, A, x, b, r, (T*)C);
  defect_lower_kernel<T><<<nb, 256, 0, s>>>(g, r, (const T*)C);
}
template void launch_defect<float>(const Grid&, const float*, const float*, const float*, float*, void*, hipStream_t,
                                   int);
template void launch_defect<double>(const Grid&, const double*, const double*, const double*, double*, void*,
                                    hipStream_t, int);

// Damped point-block Jacobi sweep (Sec. 3.4): xo = x + omega D^-1 (b - A x).
// Pass 1 leaves the partial residual in xo; pass 2 completes it and updates.
// With a zero initial guess the product with A vanishes: xo = omega D^-1 b
// (packed: D holds the upper triangles of the matrix-free level's inverses,
// 45 instead of 81 values per row of the stream that bounds this kernel).
template <typename T, bool PACKED>
__device__ __forceinline__ void pbj_zero_row(const Grid& g, const T* __restrict__ Dinv, const T* __restrict__ b,
                                             T* __restrict__ xo, T omega, int n) {
  const int t = n >> 6, l = n & 63;
  const T* Db = Dinv + (int64_t)t * (PACKED ? LaySym<T>::SLICE : Lay<T>::SLICE);
  T bv[NDOF];
#pragma unroll
  for (int c = 0; c < NDOF; ++c) bv[c] = b[(int64_t)c * g.Npad + n];
#pragma unroll
  for (int r = 0; r < NDOF; ++r) {
    T s = 0;
#pragma unroll
    for (int c = 0; c < NDOF; ++c)
      s += Db[PACKED ? LaySym<T>::off(sym_index(r, c), l) : Lay<T>::off(r * NDOF + c, l)] * bv[c];
    xo[(int64_t)r * g.Npad + n] = (n < g.N) ? omega * s : (T)0;
  }
}
template <typename T>
__device__ __forceinline__ void pbj_zero_body(const Grid& g, const T* __restrict__ Dinv, bool packed,
                                              const T* __restrict__ b, T* __restrict__ xo, T omega, int bid,
                                              int nblk) {
  ROW_LOOP_B(g, bid, nblk) {
    if (n >= g.Npad) continue;
    if (packed)
      pbj_zero_row<T, true>(g, Dinv, b, xo, omega, n);
    else
      pbj_zero_row<T, false>(g, Dinv, b, xo, omega, n);
  }
}
template <typename T>
__global__ void __launch_bounds__(256) pbj_zero_kernel(Grid g, const T* __restrict__ Dinv, bool packed,
                                                       const T* __restrict__ b, T* __restrict__ xo, T omega) {
  pbj_zero_body<T>(g, Dinv, packed, b, xo, omega, blockIdx.x, gridDim.x);
}

template <typename T>
void launch_pbj_zero(const Grid& g, const T* Dinv, bool packed, const T* b, T* xo, T omega, hipStream_t s, int G) {
  pbj_zero_kernel<T><<<row_grid(g, G), 256, 0, s>>>(g, Dinv, packed, b, xo, omega);
}
template void launch_pbj_zero<float>(const Grid&, const float*, bool, const float*, float*, float, hipStream_t, int);
template void launch_pbj_zero<double>(const Grid&, const double*, bool, const double*, double*, double, hipStream_t,
                                      int);

template <typename T>
__device__ __forceinline__ void pbj_lower_body(const Grid& g, const T* __restrict__ Dinv, const T* __restrict__ x,
                                               T* __restrict__ xo, const T* __restrict__ C, T omega, int bid,
                                               int nblk) {
  ROW_LOOP_B(g, bid, nblk) {
    if (n >= g.N) continue;
    T res[NDOF];
#pragma unroll
    for (int c = 0; c < NDOF; ++c) res[c] = xo[(int64_t)c * g.Npad + n];
    lower_pass<true>(g, n, res, C);
    const int t = n >> 6, l = n & 63;
    const T* Db = Dinv + (int64_t)t * Lay<T>::SLICE;
#pragma unroll
    for (int r = 0; r < NDOF; ++r) {
      T s = 0;
#pragma unroll
      for (int c = 0; c < NDOF; ++c) s += Db[Lay<T>::off(r * NDOF + c, l)] * res[c];
      xo[(int64_t)r * g.Npad + n] = x[(int64_t)r * g.Npad + n] + omega * s;
    }
  }
}
template <typename T>
__global__ void __launch_bounds__(256) pbj_lower_kernel(Grid g, const T* __restrict__ Dinv, const T* __restrict__ x,
                                                        T* __restrict__ xo, const T* __restrict__ C, T omega) {
  pbj_lower_body<T>(g, Dinv, x, xo, C, omega, blockIdx.x, gridDim.x);
}

template <typename T>
void launch_pbj(const Grid& g, const T* A, const T* Dinv, const T* x, const T* b, T* xo, T omega, void* C,
                hipStream_t s, int G) {
  const int nb = row_grid(g, G);
  if (G <= 0)
    defect_upper_split_kernel<T><<<split_grid(g), 256, 0, s>>>(g, A, x, b, xo, (T*)C);
  else
    defect_upper_kernel<T><<<nb, 256, 0, s>>>(g, A, x, b, xo, (T*)C);
  pbj_lower_kernel<T><<<nb, 256, 0, s>>>(g, Dinv, x, xo, (const T*)C, omega);
}
template void launch_pbj<float>(const Grid&, const float*, const float*, const float*, const float*, float*, float,
                                void*, hipStream_t, int);
template void launch_pbj<double>(const Grid&, const double*, const double*, const double*, const double*, double*,
                                 double, void*, hipStream_t, int);

// ---- batched launches (one launch for the jobs of many problems) ------------
template <typename T>
__global__ void __launch_bounds__(256) pbj_zero_batch(const BJob* __restrict__ jobs, int njobs) {
  int bid;
  const BJob& j = find_job(jobs, njobs, bid);
  pbj_zero_body<T>(j.g, (const T*)j.D, j.packed, (const T*)j.b, (T*)j.y, (T)j.omega, bid, j.nblk);
}
template <typename T>
__global__ void __launch_bounds__(256) defect_upper_split_batch(const BJob* __restrict__ jobs, int njobs) {
  int bid;
  const BJob& j = find_job(jobs, njobs, bid);
  defect_upper_split_body<T>(j.g, (const T*)j.A, (const T*)j.x, (const T*)j.b, (T*)j.y, (T*)j.C, bid, j.nblk);
}
template <typename T>
__global__ void __launch_bounds__(256) pbj_lower_batch(const BJob* __restrict__ jobs, int njobs) {
  int bid;
  const BJob& j = find_job(jobs, njobs, bid);
  pbj_lower_body<T>(j.g, (const T*)j.D, (const T*)j.x, (T*)j.y, (const T*)j.C, (T)j.omega, bid, j.nblk);
}
template <typename T>
__global__ void __launch_bounds__(256) defect_lower_batch(const BJob* __restrict__ jobs, int njobs) {
  int bid;
  const BJob& j = find_job(jobs, njobs, bid);
  defect_lower_body<T>(j.g, (T*)j.y, (const T*)j.C, bid, j.nblk);
}
template <typename T, RowMode MODE>
__global__ void __launch_bounds__(SMALL_THREADS) SMALL_OCC row_small_batch(const BJob* __restrict__ jobs, int njobs) {
  int bid;
  const BJob& j = find_job(jobs, njobs, bid);
  row_small_body<T, T, T, MODE>(j.g, (const T*)j.A, (const T*)j.D, (const T*)j.x, (const T*)j.b, (T*)j.y, (T)j.omega, bid,
                         j.nblk);
}

template <typename T>
void launch_bsr_batch(int op, const BJob* jobs, int njobs, int blocks, hipStream_t s) {
  switch (op) {
    case BOP_PBJ_ZERO: pbj_zero_batch<T><<<blocks, 256, 0, s>>>(jobs, njobs); break;
    case BOP_DEFECT_SPLIT: defect_upper_split_batch<T><<<blocks, 256, 0, s>>>(jobs, njobs); break;
    case BOP_PBJ_LOWER: pbj_lower_batch<T><<<blocks, 256, 0, s>>>(jobs, njobs); break;
    case BOP_DEFECT_LOWER: defect_lower_batch<T><<<blocks, 256, 0, s>>>(jobs, njobs); break;
    case BOP_ROW_SMALL_PBJ: row_small_batch<T, ROW_PBJ><<<blocks, SMALL_THREADS, 0, s>>>(jobs, njobs); break;
    case BOP_ROW_SMALL_DEFECT: row_small_batch<T, ROW_DEFECT><<<blocks, SMALL_THREADS, 0, s>>>(jobs, njobs); break;
    default: break;
  }
}
template void launch_bsr_batch<float>(int, const BJob*, int, int, hipStream_t);
template void launch_bsr_batch<double>(int, const BJob*, int, int, hipStream_t);

// workgroups of one job (plain shapes: one logical block of 256 rows per
// workgroup, rounded up to whole rounds over the 8 XCDs)
int bsr_job_blocks(int op, const Grid& g) {
  switch (op) {
    case BOP_PBJ_ZERO:
    case BOP_PBJ_LOWER:
    case BOP_DEFECT_LOWER: return row_grid(g, 0);
    case BOP_DEFECT_SPLIT: return split_grid(g);
    case BOP_ROW_SMALL_PBJ:
    case BOP_ROW_SMALL_DEFECT: return small_blocks(g);
    default: return 0;
  }
}

}  // namespace mvpf
