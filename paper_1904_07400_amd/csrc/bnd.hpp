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

// Value of the lane whose index differs by the mask m, within w lanes.  A host
// build that emulates the kernels and takes this path defines it itself.
#ifndef SG_SHFL_XOR
#ifdef __HIPCC__
#define SG_SHFL_XOR(v, m, w) __shfl_xor(v, m, w)
#else
#include <stdlib.h>
#define SG_SHFL_XOR(v, m, w) (abort(), (v))
#endif
#endif

// Sum over the G consecutive threads of a group (a power of two, at most 64).
template <int G>
__device__ __forceinline__ double group_sum(double v) {
#pragma unroll
  for (int m = G / 2; m > 0; m /= 2) v += SG_SHFL_XOR(v, m, G);
  return v;
}

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

// The two sums of the line x(0), x(1), ... of N values, by the G threads q of
// a group, for NC independent lines (the components of x).  Loads past the
// line's end or the table's are clamped and masked, not branched around, so
// that all of a thread's loads issue together.
template <int N, int G, int NC, typename F>
__device__ __forceinline__ void bnd_sums(F x, int order, const double* __restrict__ bc, int q, double (&s)[2][NC]) {
  constexpr int LEN = N < kBndLen ? N : kBndLen, IT = (LEN + G - 1) / G;
  double v[IT][NC], c[2][IT];
#pragma unroll
  for (int k = 0; k < IT; ++k) {
    const int i = q + k * G < LEN ? q + k * G : LEN - 1;
    x(i, v[k]);
    c[0][k] = bc[i];
    c[1][k] = bc[kBndLen + i];
  }
#pragma unroll
  for (int a = 0; a < NC; ++a) s[0][a] = s[1][a] = 0.0;
#pragma unroll
  for (int k = 0; k < IT; ++k) {
    const bool in = (k + 1) * G <= LEN || q + k * G < LEN;
#pragma unroll
    for (int a = 0; a < NC; ++a) {
      s[0][a] += in ? c[0][k] * v[k][a] : 0.0;
      s[1][a] += in ? c[1][k] * v[k][a] : 0.0;
    }
  }
#pragma unroll
  for (int a = 0; a < NC; ++a) {
    s[0][a] = group_sum<G>(s[0][a]);
    if (order == 5) s[1][a] = group_sum<G>(s[1][a]);  // else zero: c1 is
  }
}

// The values of a complex line (N values) past its ends, by the T threads of
// its slice of the workgroup (t: this thread): end holds those of slots N, N + 1
// in the slice's first group of threads, start those of slots -1, -2 in its
// last; both are zero elsewhere.
template <int N, int T, typename R>
__device__ __forceinline__ void bnd_line(const cx<R>* __restrict__ col, int order, const double* __restrict__ bc,
                                         int t, cx<R> (&end)[2], cx<R> (&start)[2]) {
  constexpr int G = T < 64 ? T : 64;
  auto sums = [&](bool rev, cx<R>(&o)[2]) {
    double s[2][2];
    bnd_sums<N, G, 2>(
        [&](int i, double(&v)[2]) {
          const cx<R> z = col[(unsigned)(rev ? N - 1 - i : i)];
          v[0] = (double)z.x;
          v[1] = (double)z.y;
        },
        order, bc, t % G, s);
    o[0] = cx<R>{(R)s[0][0], (R)s[0][1]};
    o[1] = cx<R>{(R)s[1][0], (R)s[1][1]};
  };
  end[0] = end[1] = start[0] = start[1] = cx<R>{(R)0, (R)0};
  if (t / G == 0) sums(true, end);
  if (t / G == (T - 1) / G) sums(false, start);
}

// The value that thread t of a column c's T threads folds in: that of slot N + t
// for t < 2, of slot t - T for the last two, from the parts that pass A left (xb,
// pg parts per value); zero elsewhere.
template <int T, typename R>
__device__ __forceinline__ cx<R> bnd_value(const cx<R>* __restrict__ xb, int pg, int c, int t) {
  if (!xb || (t >= 2 && t < T - 2)) return cx<R>{(R)0, (R)0};
  const cx<R>* p = xb + (int64_t)(4 * c + (t < 2 ? t : 2 + T - 1 - t)) * pg;
  double x = 0.0, y = 0.0;
  for (int w0 = 0; w0 < pg; w0 += 8) {
    // eight loads together, those past pg masked
    cx<R> z[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) z[i] = p[w0 + i < pg ? w0 + i : pg - 1];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      x += w0 + i < pg ? (double)z[i].x : 0.0;
      y += w0 + i < pg ? (double)z[i].y : 0.0;
    }
  }
  return cx<R>{(R)x, (R)y};
}

}  // namespace sg
