// Sum factorisation over lane pairs, for kernels in which eight lanes hold an
// element: lane j owns corner j and Gauss point j of the 2x2x2 rule (bit d of
// j: the side along direction d for both).
#pragma once
#include "common.h"

namespace mvpf {

constexpr double MGQ0 = 0.21132486540518711775;  // (1 - 1/sqrt 3) / 2
constexpr double MGQ1 = 0.78867513459481288225;

// Lane exchanges inside groups of 8 lanes by DPP (no LDS traffic): xor 1 and
// xor 2 are quad permutations; xor 4 is the half-row mirror (lane i <- 7 - i)
// followed by the quad reversal (i <- i ^ 3), since (7 - i) ^ 3 = i ^ 4.
template <int X, typename T>
__device__ __forceinline__ T lane_xor(T v) {
  if constexpr (X == 1) return dpp_t<0xB1>(v);       // quad_perm [1,0,3,2]
  else if constexpr (X == 2) return dpp_t<0x4E>(v);  // quad_perm [2,3,0,1]
  else return dpp_t<0x1B>(dpp_t<0x141>(v));          // row_half_mirror, then quad_perm [3,2,1,0]
}

// One direction of the trilinear interpolation at the Gauss points, by lane
// pairs (sum factorisation).  Each lane holds n values belonging to its node
// index bit b along this direction; with t = (partner's value) - (own value)
// it gets, at its Gauss coordinate q (the same bit selects q), the
// interpolated value s = own + qq t (qq = MGQ0, the other node's weight, for
// either b) and, for the first nd values, the difference across the pair, d =
// sg t (sg = +1 for b = 0, -1 for b = 1): the derivative along this direction
// on the unit reference cube.  The partner's value enters only through the
// subtraction, so the lane exchange folds into it (a DPP operand), and no lane
// selects are needed.
template <int X, typename T, int n, int nd>
__device__ __forceinline__ void interp_pair(const T (&in)[n], T qq, T sg, T (&s)[n], T (&d)[nd]) {
#pragma unroll
  for (int k = 0; k < n; ++k) {
    const T t = lane_xor<X>(in[k]) - in[k];
    s[k] = in[k] + qq * t;
    if (k < nd) d[k] = sg * t;
  }
}

// Transpose of interp_pair: a lane at Gauss coordinate q along this
// direction holds coefficients a (of the values) and bs = sb * b (of the
// derivatives, sb = -1 for node bit 0, +1 for bit 1: the sign is applied by
// the caller where b is formed); afterwards it holds, for its node bit, the
// sum over both Gauss points of a * phi(q) + b * phi', phi = 1 - q or q,
// phi' = -1 or +1.  Own part a mq + bs, partner's part a tq - bs (mq = MGQ1,
// tq = MGQ0); the exchange folds into the final addition.
template <int X, typename T, int n>
__device__ __forceinline__ void interp_pair_t(const T (&a)[n], const T (&bs)[n], T mq, T tq, T (&out)[n]) {
#pragma unroll
  for (int k = 0; k < n; ++k) {
    const T mine = a[k] * mq + bs[k];
    const T theirs = a[k] * tq - bs[k];
    out[k] = mine + lane_xor<X>(theirs);
  }
}

// Element outputs through LDS: a lane holds NC values of corner gp of element jw
// of its workgroup (lane = 8 * element + corner).  Staged per stream (corner, c),
// the workgroup merges each element's left corners with the right corners of its
// predecessor in the same row and stores one contiguous, aligned run of each
// merged stream (whole 128-byte lines at 32 elements in FP32), plus the right
// corners that no element of the workgroup takes (its last element's, row ends):
//   E[(NC q + c) se + e], then W[(NC q + c) nw + bid], Rr[(NC q + c) nr + row]
// (q = by + 2 bz; W and Rr follow E's 4 NC streams).  Every lane of the
// workgroup reaches the barrier.  eo: 8 NC (epw + 1) values; the workgroup's
// elements are e = bid epw ..., ne of them exist, a row holds nx and e = 0 starts one.
template <typename T, int NC>
__device__ __forceinline__ void store_corners(T* eo, const T (&out)[NC], int gp, int jw, int epw, int bid, int nx,
                                              int64_t ne, T* __restrict__ E, int64_t se, int64_t nw, int64_t nr) {
#pragma unroll
  for (int c = 0; c < NC; ++c) eo[(gp * NC + c) * (epw + 1) + jw] = out[c];
  __syncthreads();
  const int64_t ew = (int64_t)bid * epw;  // the workgroup's first element
  const int ex0 = (int)(ew % nx);
  T* __restrict__ W = E + 4 * NC * se;
  T* __restrict__ Rr = W + 4 * NC * nw;
  for (int idx = threadIdx.x; idx < 4 * NC * epw; idx += blockDim.x) {
    const int s = idx / epw, jj = idx - s * epw;  // merged stream s = NC q + c
    const int64_t e = ew + jj;
    if (e >= ne) continue;
    const int q = s / NC, c = s - NC * q;
    int ex = ex0 + jj;
    while (ex >= nx) ex -= nx;
    const T* left = eo + (2 * NC * q + c) * (epw + 1);      // corner 2q
    const T* right = eo + (2 * NC * q + NC + c) * (epw + 1);  // corner 2q + 1
    T v = left[jj];
    if (jj > 0 && ex > 0) v = v + right[jj - 1];
    E[(int64_t)s * se + e] = v;
    if (ex == nx - 1) Rr[(int64_t)s * nr + e / nx] = right[jj];
    else if (jj == epw - 1) W[(int64_t)s * nw + bid] = right[jj];
  }
}

// Merged element outputs of one assembly slab (whole element layers, chunk-local
// elements, SLAB_EPW per workgroup), NC values per corner: values in all, and the
// node sum of value c at node (i, j) and node layer k counted from the slab's
// first element layer.
constexpr int SLAB_EPW = 32;
__host__ __device__ inline int64_t slab_nw(const Chunk& ck) { return ck.NEcpad / SLAB_EPW; }
__host__ __device__ inline int64_t slab_values(const Chunk& ck, int nx, int nc) {
  return 4 * (int64_t)nc * (ck.NEcpad + slab_nw(ck) + ck.NEc / nx);
}
__device__ __forceinline__ double slab_node_sum(const Grid& g, const Chunk& ck, const double* __restrict__ E, int nc,
                                                int c, int i, int j, int k) {
  const int nz = ck.NEc / (g.nx * g.ny);
  const int64_t nw = slab_nw(ck), nr = ck.NEc / g.nx;
  const double* __restrict__ W = E + 4 * (int64_t)nc * ck.NEcpad;
  const double* __restrict__ Rr = W + 4 * (int64_t)nc * nw;
  double s = 0.0;
#pragma unroll
  for (int q = 3; q >= 0; --q) {  // element row (j - by, k - bz) holds the node at (by, bz)
    const int ey = j - (q & 1), ez = k - (q >> 1);
    if (ey < 0 || ey >= g.ny || ez < 0 || ez >= nz) continue;
    const int64_t r = ey + (int64_t)g.ny * ez, st = nc * q + c;
    if (i < g.nx) {
      const int64_t e = i + g.nx * r;
      double t = E[st * ck.NEcpad + e];
      if (i > 0 && (e & (SLAB_EPW - 1)) == 0) t = t + W[st * nw + e / SLAB_EPW - 1];
      s += t;
    } else {
      s += Rr[st * nr + r];
    }
  }
  return s;
}

}  // namespace mvpf
