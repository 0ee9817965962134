// Grid transfers between nested structured levels (Sec. 3.4: prolongation and
// restriction between the rediscretised levels; state for reassembly).
//  * prolongation P: trilinear interpolation; fine node i takes weight 1 from
//    the coincident coarse node, 1/2 from each of the two coarse neighbours of
//    an edge midpoint, and so on (product of 1D weights);
//  * restriction R = P^T;
//  * state injection: coarse node value = fine value at the coincident node.
// Restricted residuals are zeroed on constrained coarse dofs and prolongated
// corrections are not added on constrained fine dofs.
#include "common.h"

namespace mvpf {

// Latency bounds the transfers: most of a V-cycle's levels hold fewer nodes
// than the chip has lanes, and a thread that takes a whole node walks
// 27 x NDOF loads one neighbour at a time.  So one thread takes one component
// of one node, with its 27 (restriction) or 8 (prolongation) loads in flight
// together, in the order of the sums.  FP64, 41^3 -> 21^3 nodes: restriction
// 13.6 -> 6.4 us with the coarse level's first sweep in it, prolongation
// 9.3 -> 5.6; 5^3 -> 3^3: 7.2 -> 3.5 and 7.3 -> 3.2.
//
// The restriction's workgroup takes RN coarse nodes (few, to spread a small
// level's loads over the chip); with block inverses it exchanges the
// restricted components through LDS and writes the level's first sweep from a
// zero guess as well, x = omega D^-1 b, in the order of pbj_zero_kernel.
constexpr int RN = 16;
constexpr int RT = (NDOF * RN + 63) / 64 * 64;
template <typename T>
__device__ __forceinline__ void restrict_body(const Grid& f, const Grid& c, const T* __restrict__ rf,
                                              const uint16_t* __restrict__ cmask, T* __restrict__ bc,
                                              const T* __restrict__ Dinv, T* __restrict__ xc, T omega, int bid) {
  __shared__ T sh[NDOF][RN];
  const int l = threadIdx.x % RN, q = threadIdx.x / RN;
  const int I = bid * RN + l;
  const bool own = q < NDOF;
  T acc = 0, dv[NDOF];
  if (own && Dinv) {
    const T* Db = Dinv + (int64_t)(I / TILE) * Lay<T>::SLICE;
#pragma unroll
    for (int d = 0; d < NDOF; ++d) dv[d] = Db[Lay<T>::off(q * NDOF + d, I % TILE)];
  }
  if (own && I < c.N) {
    const unsigned msk = cmask[I];
    const int ci = I % c.nnx, cj = (I / c.nnx) % c.nny, ck = I / (c.nnx * c.nny);
    const int fi = 2 * ci, fj = 2 * cj, fk = 2 * ck;
    const T* r = rf + (int64_t)q * f.Npad + fi + f.nnx * (fj + f.nny * fk);
    T v[NSTEN];
    bool in[NSTEN];
#pragma unroll
    for (int s = 0; s < NSTEN; ++s) {
      const int dx = s % 3 - 1, dy = (s / 3) % 3 - 1, dz = s / 9 - 1;
      in[s] = (unsigned)(fi + dx) < (unsigned)f.nnx && (unsigned)(fj + dy) < (unsigned)f.nny &&
              (unsigned)(fk + dz) < (unsigned)f.nnz;
      v[s] = r[in[s] ? dx + f.nnx * (dy + f.nny * dz) : 0];
    }
#pragma unroll
    for (int s = 0; s < NSTEN; ++s) {
      const int dx = s % 3 - 1, dy = (s / 3) % 3 - 1, dz = s / 9 - 1;
      acc += (T)((dx ? 0.5 : 1.0) * (dy ? 0.5 : 1.0) * (dz ? 0.5 : 1.0)) * (in[s] ? v[s] : (T)0);
    }
    if ((msk >> q) & 1) acc = 0;
  }
  if (own) bc[(int64_t)q * c.Npad + I] = acc;
  if (!Dinv) return;  // uniform
  if (own) sh[q][l] = acc;
  __syncthreads();
  if (!own) return;
  T s = 0;
#pragma unroll
  for (int d = 0; d < NDOF; ++d) s += dv[d] * sh[d][l];
  xc[(int64_t)q * c.Npad + I] = I < c.N ? omega * s : (T)0;
}
template <typename T>
__global__ void __launch_bounds__(RT) restrict_kernel(Grid f, Grid c, const T* __restrict__ rf,
                                                      const uint16_t* __restrict__ cmask, T* __restrict__ bc,
                                                      const T* __restrict__ Dinv, T* __restrict__ xc, T omega) {
  restrict_body<T>(f, c, rf, cmask, bc, Dinv, xc, omega, blockIdx.x);
}
static_assert(TILE % RN == 0, "a workgroup's nodes lie in one tile, whole workgroups cover the padding");
static int restrict_blocks(const Grid& coarse) { return coarse.Npad / RN; }

template <typename T>
void launch_restrict(const Grid& fine, const Grid& coarse, const T* rf, const uint16_t* cmask, T* bc, const T* Dinv,
                     T* xc, T omega, hipStream_t s) {
  restrict_kernel<T><<<restrict_blocks(coarse), RT, 0, s>>>(fine, coarse, rf, cmask, bc, Dinv, xc, omega);
}
template void launch_restrict<float>(const Grid&, const Grid&, const float*, const uint16_t*, float*, const float*,
                                     float*, float, hipStream_t);
template void launch_restrict<double>(const Grid&, const Grid&, const double*, const uint16_t*, double*,
                                      const double*, double*, double, hipStream_t);

// workgroup bid = node block * NDOF + component: the components of a node
// block run together and share its masks
template <typename T>
__device__ __forceinline__ void prolong_add_body(const Grid& f, const Grid& c, const T* __restrict__ ec,
                                                 const uint16_t* __restrict__ fmask, T* __restrict__ xf, int bid) {
  const int n = bid / NDOF * 256 + threadIdx.x, q = bid % NDOF;
  if (n >= f.N) return;
  if ((fmask[n] >> q) & 1) return;
  const int i = n % f.nnx, j = (n / f.nnx) % f.nny, k = n / (f.nnx * f.nny);
  const T* e = ec + (int64_t)q * c.Npad + (i >> 1) + c.nnx * ((j >> 1) + c.nny * (k >> 1));
  T v[8];
#pragma unroll
  for (int s = 0; s < 8; ++s) {
    const bool in = (!(s & 1) || (i & 1)) && (!(s & 2) || (j & 1)) && (!(s & 4) || (k & 1));
    v[s] = in ? e[(s & 1) + c.nnx * ((s >> 1 & 1) + c.nny * (s >> 2))] : (T)0;
  }
  T acc = 0;
#pragma unroll
  for (int s = 0; s < 8; ++s) acc += v[s];
  const T w = (T)((i & 1 ? 0.5 : 1.0) * (j & 1 ? 0.5 : 1.0) * (k & 1 ? 0.5 : 1.0));
  xf[(int64_t)q * f.Npad + n] += w * acc;
}
template <typename T>
__global__ void __launch_bounds__(256) prolong_add_kernel(Grid f, Grid c, const T* __restrict__ ec,
                                                          const uint16_t* __restrict__ fmask, T* __restrict__ xf) {
  prolong_add_body<T>(f, c, ec, fmask, xf, blockIdx.x);
}
static int prolong_blocks(const Grid& fine) { return (fine.Npad + 255) / 256 * NDOF; }

template <typename T>
void launch_prolong_add(const Grid& fine, const Grid& coarse, const T* ec, const uint16_t* fmask, T* xf,
                        hipStream_t s) {
  prolong_add_kernel<T><<<prolong_blocks(fine), 256, 0, s>>>(fine, coarse, ec, fmask, xf);
}
template void launch_prolong_add<float>(const Grid&, const Grid&, const float*, const uint16_t*, float*, hipStream_t);
template void launch_prolong_add<double>(const Grid&, const Grid&, const double*, const uint16_t*, double*,
                                         hipStream_t);

__global__ void __launch_bounds__(256) inject_kernel(Grid f, Grid c, const double* __restrict__ sf,
                                                     double* __restrict__ sc) {
  const int I = blockIdx.x * blockDim.x + threadIdx.x;
  if (I >= c.Npad) return;
  if (I >= c.N) {
    for (int q = 0; q < NSTATE; ++q) sc[(int64_t)q * c.Npad + I] = 0.0;
    return;
  }
  const int ci = I % c.nnx, cj = (I / c.nnx) % c.nny, ck = I / (c.nnx * c.nny);
  const int m = 2 * ci + f.nnx * (2 * cj + f.nny * 2 * ck);
#pragma unroll
  for (int q = 0; q < NSTATE; ++q) sc[(int64_t)q * c.Npad + I] = sf[(int64_t)q * f.Npad + m];
}

void launch_inject(const Grid& fine, const Grid& coarse, const double* sf, double* sc, hipStream_t s) {
  inject_kernel<<<(coarse.Npad + 255) / 256, 256, 0, s>>>(fine, coarse, sf, sc);
}

__global__ void __launch_bounds__(256) inject_mask_kernel(Grid f, Grid c, const uint16_t* __restrict__ mf,
                                                          uint16_t* __restrict__ mc) {
  const int I = blockIdx.x * blockDim.x + threadIdx.x;
  if (I >= c.Npad) return;
  if (I >= c.N) { mc[I] = 0; return; }
  const int ci = I % c.nnx, cj = (I / c.nnx) % c.nny, ck = I / (c.nnx * c.nny);
  mc[I] = mf[2 * ci + f.nnx * (2 * cj + f.nny * 2 * ck)];
}

void launch_inject_mask(const Grid& fine, const Grid& coarse, const uint16_t* mf, uint16_t* mc, hipStream_t s) {
  inject_mask_kernel<<<(coarse.Npad + 255) / 256, 256, 0, s>>>(fine, coarse, mf, mc);
}

// ---- batched launches: g = fine grid, g2 = coarse grid of every job ---------
template <typename T>
__global__ void __launch_bounds__(RT) restrict_batch(const BJob* __restrict__ jobs, int njobs) {
  int bid;
  const BJob& j = find_job(jobs, njobs, bid);
  restrict_body<T>(j.g, j.g2, (const T*)j.x, j.mask, (T*)j.y, (const T*)j.D, (T*)j.C, (T)j.omega, bid);
}
template <typename T>
__global__ void __launch_bounds__(256) prolong_add_batch(const BJob* __restrict__ jobs, int njobs) {
  int bid;
  const BJob& j = find_job(jobs, njobs, bid);
  prolong_add_body<T>(j.g, j.g2, (const T*)j.x, j.mask, (T*)j.y, bid);
}
template <typename T>
void launch_transfer_batch(int op, const BJob* jobs, int njobs, int blocks, hipStream_t s) {
  if (op == BOP_RESTRICT)
    restrict_batch<T><<<blocks, RT, 0, s>>>(jobs, njobs);
  else if (op == BOP_PROLONG)
    prolong_add_batch<T><<<blocks, 256, 0, s>>>(jobs, njobs);
}
template void launch_transfer_batch<float>(int, const BJob*, int, int, hipStream_t);
template void launch_transfer_batch<double>(int, const BJob*, int, int, hipStream_t);

// workgroups of one job
int transfer_job_blocks(int op, const BJob& j) { return op == BOP_RESTRICT ? restrict_blocks(j.g2) : prolong_blocks(j.g); }

}  // namespace mvpf
