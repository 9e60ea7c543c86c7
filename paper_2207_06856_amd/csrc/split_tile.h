// Squared distances to float32 accuracy on the binary16 matrix cores.
//
// With a = (x - c) / l (c the centre of the points' bounding box, float64) and
// a unit u with R / 2000 <= u < R sqrt(2) / 2000 for the box's scaled half
// diagonal R, every coordinate is cut into an integer and a remainder,
// a / u = q + f with |q| <= 2000 and |f| <= 1/2.  Then
//   |a_i - a_j|^2 / u^2 = |q_i - q_j|^2 + [2 (q_i - q_j).(f_i - f_j) + |f_i - f_j|^2].
// The first term is a sum of products of integers that binary16 holds exactly
// (q, -2q up to 4000 and even, |q|^2 <= 2004^2 as 2048 N1 + N0), and every
// partial sum is an integer below 2^24: the first 32-wide MFMA forms it with no
// rounding at all, so nothing is lost to the cancellation in
// |a_i|^2 + |a_j|^2 - 2 a_i.a_j, which is what keeps a plain float32 (or
// split) expansion from the accuracy of coordinate differences.  The bracket is
// smaller by |f| / |q| ~ 2^-11, and the following MFMAs add it from f in two
// binary16 parts and g = 2 q.f + |f|^2 in three, from zero, and the two sums are
// added once.  (On top of the first sum every MFMA would round at its size: 1.1 to 3
// times the error of sums of far entries.)  The remainder rounds at q.f's size, up to
// 2^12 before it cancels: an entry's r^2 carries 2^-25 of itself and 1.2e-10 R^2.
// Coordinate differences of the float32 x / l carry 2 r |x / l| 2^-25, and their
// float32 sum d / 2 roundings: more on ordinary points, less for close ones on wide
// boxes, hence the radius limits of the callers; a caller with one point set takes
// the diagonal's distance as 0.  u is chosen so that the scale from r^2 / u^2 to the
// exponent's argument is a power of two: the argument takes no further rounding, and
// no constant's.
// Not for Matern-1/2, whose value falls linearly in r at r = 0, where an
// absolute error of r^2 would be magnified.
//
// Operand rows of KC 32-wide chunks (side 0: output rows, side 1: columns):
//   slot        side 0              side 1
//   0 .. d-1    q                   -2 q
//   d .. d+3    1, 2048, N0, N1     N0, N1, 1, 2048
//   32 + ..     q, q, f1, f2, f1    -2 f1, -2 f2, -2 q, -2 q, -2 f1     (d each)
//   then        1, 1, 1, g1..g3     g1..g3, 1, 1, 1
//
// The fine form, for the true residual, whose distances are float64 otherwise:
// a / u = q + f + e, f a multiple of 2^-10 and e = E / 2048, E in binary16 (a to 2^-24 u,
// 2^-35 R), with the expanded sums
//   I = -2 q_i.q_j + N_i + N_j,      N = |q|^2 + rint(2 q.f),
//   F = -2 q_i.f_j - 2 f_i.q_j,
//   T = -2 q_i.e_j - 2 e_i.q_j - 2 f_i.f_j - 2 f_i.e_j - 2 e_i.f_j + h_i + h_j,
//       h = 2 q.f - rint(2 q.f) + 2 q.e + |f|^2 + 2 f.e
// (|e_i - e_j|^2 < d 2^-20 is left out).  F's terms are multiples of 2^-9 whose
// partial sums stay below 2^15, so that its MFMAs are exact like I's, and I + F is
// exact for close points.  T is some 2^4 at most before it cancels, with h in three
// binary16 parts: its roundings are about 2^-19 u^2, R^2 2^-40 in r^2; I + F and
// (I + F) + T are rounded once each, as the float64 distance is when it becomes a
// float32 and is scaled to the exponent's argument.  One more MFMA and two additions:
//   slot        side 0                           side 1
//   first chunk as above, with this N
//   F           q, f                             -2 f, -2 q                      (d each)
//   T           q / 2^11, E, f, f / 2^5, E / 2^6 -2 E, -q / 2^10, -2 f, -E / 2^5, -f / 2^4
//   then        1, 1, 1, h1..h3                  h1..h3, 1, 1, 1
#pragma once

#include "fused_tile.h"
#include "internal.h"

namespace gpmi {
namespace split {

using f16::f4;
using f16::h4;
using f16::h8;

// r^2 / u^2 of 16 columns (operand fragments a) and 16 rows (b): element v of
// a lane is column 4 g + v, row l16.
template <int KC>
__device__ __forceinline__ f4 sqdist(const h8 (&a)[KC], const h8 (&b)[KC]) {
  const f4 z = f4{0.f, 0.f, 0.f, 0.f};
  f4 s = f16::mfma32<_Float16>(a[0], b[0], z), t = z;
#pragma unroll
  for (int kc = 1; kc < KC; ++kc) t = f16::mfma32<_Float16>(a[kc], b[kc], t);
#pragma unroll
  for (int v = 0; v < 4; ++v) s[v] += t[v];
  return s;
}

// The same from fine operands.
template <int KC>
__device__ __forceinline__ f4 sqdist_fine(const h8 (&a)[KC], const h8 (&b)[KC]) {
  constexpr int F = 1 + f_chunks_of(KC);         // the first chunk of T
  const f4 z = f4{0.f, 0.f, 0.f, 0.f};
  f4 s = f16::mfma32<_Float16>(a[0], b[0], z), f = z, t = z;
#pragma unroll
  for (int kc = 1; kc < F; ++kc) f = f16::mfma32<_Float16>(a[kc], b[kc], f);
#pragma unroll
  for (int kc = F; kc < KC; ++kc) t = f16::mfma32<_Float16>(a[kc], b[kc], t);
#pragma unroll
  for (int v = 0; v < 4; ++v) s[v] = (s[v] + f[v]) + t[v];
  return s;
}

// float32 kernel value from D = r^2 / u^2 (cs: Info::cs).
template <int KIND>
__device__ __forceinline__ float kval(float D, float cs) {
  constexpr float kLn2f = 0.6931471805599453f;
  if constexpr (KIND == GP_KERNEL_RBF) {
    return __builtin_amdgcn_exp2f(D * cs);
  } else {
    const float sp = __builtin_amdgcn_sqrtf(fabsf(D * cs));   // distance times log2 e
    const float e = __builtin_amdgcn_exp2f(-sp);
    if constexpr (KIND == GP_KERNEL_MATERN32)
      return fmaf(sp, kLn2f, 1.0f) * e;
    else
      return fmaf(sp, fmaf(sp, kLn2f * kLn2f / 3.0f, kLn2f), 1.0f) * e;
  }
}

}  // namespace split
}  // namespace gpmi
