// The spline interpolation systems (k = 3, 4, 5) inside the zero-padded
// transforms.
//
// Along one axis the coefficients C of a line d of n values solve T C = d on
// [0, n), C = 0 outside, T the symmetric stencil ((1, 6, 1) / 8, (1, 4, 1) / 6,
// (1, 76, 230, 76, 1) / 384).  On the zero-padded period 2n the line that C
// itself is mapped to by the circulant T is d plus a few values outside it,
//   (T C)_-1 = t1 C_0 + t2 C_1,  (T C)_-2 = t2 C_0,  and the same past the end,
// so the transform of C is that of d with these values in the padding slots
// -1, -2, n, n + 1, divided by the symbol t0 + 2 t1 cos(th) + 2 t2 cos(2 th) (at
// least 1/5; the division is part of the stored spectra, FP64 at plan time).
// No system is solved per step.  The values are sums over the line,
//   (T C)_-1 = sum_i c0_i d_i,  (T C)_-2 = sum_i c1_i d_i,
// whose coefficients (combinations of the first two rows of the inverse of the
// n x n matrix, symmetric under reversal of the line) fall below 1e-18 of the
// first after kBndReach entries.  They are summed in FP64.
//
// Adjoint: the line's gradient is that of the cropped transform plus c0_i, c1_i
// times the gradients found in the padding slots.
#pragma once
#include <hip/hip_runtime.h>

#include "fft.hpp"

namespace sg {

constexpr int kBndLen = 48;  // entries of c0, then of c1, in a coefficient table (zero past the reach)
__host__ __device__ constexpr int bnd_reach(int order) { return order == 3 ? 24 : (order == 4 ? 32 : 42); }

// The inverse symbol of order's system at bin p of a period of 2n.
__device__ __forceinline__ double bnd_symbol(int order, int p, int n) {
  double s1, c1;  // sin, cos of th
  sincospi((double)p / n, &s1, &c1);
  if (order == 3) return 8.0 / (6.0 + 2.0 * c1);
  if (order == 4) return 6.0 / (4.0 + 2.0 * c1);
  return 384.0 / (230.0 + 152.0 * c1 + 2.0 * (2.0 * c1 * c1 - 1.0));
}

// Adjoint: value v of element i plus c0_i, c1_i times the gradients u0, u1 of
// the two padding slots beyond its end of the line.
template <typename R>
__device__ __forceinline__ R bnd_add(R v, R u0, R u1, const double* __restrict__ bc, int i) {
  return (R)((double)v + bc[i] * (double)u0 + bc[kBndLen + i] * (double)u1);
}
template <typename R>
__device__ __forceinline__ cx<R> bnd_add(cx<R> v, cx<R> u0, cx<R> u1, const double* __restrict__ bc, int i) {
  return {bnd_add(v.x, u0.x, u1.x, bc, i), bnd_add(v.y, u0.y, u1.y, bc, i)};
}

// The padding values of columns of more than one wave come from pass A in parts (the
// shorter columns' threads sum their own), one per group of rows of
// a size that depends on the row length and the precision only, so that the result
// does not depend on the rows per workgroup (bnd_parts of them, in groups of gp
// rows): part w of the value of slot N, N + 1, -1, -2 (i = 0 .. 3) of column c < M at
// xb[4 (w M + c) + i], so that the rows of one group leave their parts of
// neighbouring columns next to each other.
__host__ __device__ constexpr int bnd_parts(int order, int n, int gp) {
  const int len = bnd_reach(order) < n ? bnd_reach(order) : n;
  return (len + gp - 1) / gp;
}
template <typename R>
__device__ __forceinline__ cx<R> bnd_total(const cx<R>* __restrict__ p, int pg, int M) {
  double x = 0.0, y = 0.0;
  constexpr int B = sizeof(R) == 8 ? 14 : 8;
  for (int w0 = 0; w0 < pg; w0 += B) {
    // B loads together, those past pg masked (FP64 rows of 8192 leave up to 42: eight
    // together, step of 8192 x 2048, k = 5 1132 us against 1108)
    cx<R> z[B];
#pragma unroll
    for (int i = 0; i < B; ++i) z[i] = p[(int64_t)4 * M * (w0 + i < pg ? w0 + i : pg - 1)];
#pragma unroll
    for (int i = 0; i < B; ++i) {
      x += w0 + i < pg ? (double)z[i].x : 0.0;
      y += w0 + i < pg ? (double)z[i].y : 0.0;
    }
  }
  return cx<R>{(R)x, (R)y};
}
// The value that thread t of the column's T >= 4 threads folds in: that of slot
// N + t for t < 2, of slot t - T for the last two; zero elsewhere.
template <int T, typename R>
__device__ __forceinline__ cx<R> bnd_value(const cx<R>* __restrict__ xb, int pg, int M, int c, int t) {
  if (!xb || (t >= 2 && t < T - 2)) return cx<R>{(R)0, (R)0};
  return bnd_total(xb + 4 * c + (t < 2 ? t : 2 + T - 1 - t), pg, M);
}

}  // namespace sg
