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

}  // namespace mvpf
