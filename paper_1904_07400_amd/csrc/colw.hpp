// Column pass on 16-element threads (FP32, N = 2^a): one column of the row
// spectra on T = N / 16 threads, its transforms in three steps of radix 16,
// 16 and R3 = N / 256, with one workgroup exchange each.
//
// A length-N transform, input index n = t + T e, output index
// k = k1 + 16 k2 + 256 k3, with t = t0 + R3 t1 (t1 < 16, t0 < R3):
//   step 1: thread t holds x[t + T e] and runs a 16-point DFT over e -> k1,
//           then the twiddle w_N^(t k1);
//   exchange 1 (workgroup): thread u = t0 + R3 k1 then holds t1 = 0 .. 15;
//   step 2: 16-point DFT over t1 -> k2, then the twiddle w_T^(t0 k2);
//   exchange 2 (inside a wave): thread u = k2lo + R3 k1 then holds
//           register b R3 + t0, for k2 = k2lo + R3 b;
//   step 3: R3-point DFTs over t0 -> k3.
// Exchange 2 moves elements between the R3 threads of one k1 only, in the
// LDS rows that these threads read in exchange 1, so it needs no workgroup
// barrier.  The inverse runs the steps backwards and takes the forward's
// output order.  Against the four-step form of fft4.hpp (8 elements per
// thread, three exchanges per transform): two exchanges, half the threads,
// and so two independent workgroups per compute unit at N = 4096, the length that
// the library launches (N = 256 .. 2048, P columns per wave, in the CPU emulation).
// Its registers do not hold all of it: 76 bytes of scratch per lane forward (hi + lo
// tables 100, even k 112), none in the adjoint with single-float tables.
//
// LDS slot: element (k1, t1 or k2, t0) at k1 ROW + STR (t1 or k2) + t0, STR =
// R3 + 1; ROW is chosen so that the 32 lanes of one access of 8-byte words
// fall in distinct banks (writes of exchange 1 excepted, whose skew by one
// element per R3 lanes meets at most two lanes per bank).
#pragma once
#include "colfs.hpp"

namespace sg {

template <int N>
struct cw_shape {
  static constexpr int E = 16;
  static constexpr int T = N / E;
  static constexpr int R3 = N / 256;
  static constexpr int STR = R3 > 1 ? R3 + 1 : 1;
  static constexpr int ROW = R3 == 16 ? 272 : (R3 == 8 ? 152 : (R3 == 4 ? 84 : (R3 == 2 ? 50 : 17)));
  static constexpr int SLOT = 16 * ROW;
  static constexpr int P = T >= 64 ? 1 : 64 / T;  // columns per workgroup
  static_assert(N >= 256 && N <= 4096 && (N & (N - 1)) == 0, "16 x 16 x R3, R3 <= 16");
  static_assert(ROW >= 16 * STR && N + N / 16 <= SLOT, "LDS slot");
  // twiddle table: w_N^(t k1) at k1 T + t, then w_T^(t0 k2) at N + k2 R3 + t0, then
  // (even k) w_2N^q' of the bins q' = d3_base(u) at N + T + u and d3_base(u) +
  // 15 D3_SPAN at N + 2 T + u
  static constexpr int TW_SIZE = N + 3 * T;
  // output order of the forward transform: thread u, register r holds bin
  // d3_base(u) + d3_off(r)
  static constexpr int D3_SPAN = 16 * R3;
  __host__ __device__ static constexpr int d3_base(int u) { return u / R3 + 16 * (u % R3); }
  __host__ __device__ static constexpr int d3_off(int r) { return 16 * R3 * (r / R3) + 256 * (r % R3); }
  // the same offset as D3_SPAN * H, H = 0 .. 15: register of H
  __host__ __device__ static constexpr int d3_reg(int H) { return H % (16 / R3) * R3 + H / (16 / R3); }

  // ---- spectrum tables of this pass: one row of TAB entries per column bin,
  // in the order the threads hold the bins, so that a thread reads its
  // entries as whole 8-entry pieces.  Stored are the bins q' < N / 2 of each
  // half (q = 2q' + 1 in [0, N/2), q = 2q' in [N/2, N)), bin d3_base(u) +
  // D3_SPAN H of thread u at 8 u + H (H < 8).  The mirrored bins (H >= 8) of
  // thread u are the stored ones of another thread in reverse order:
  // q' -> N - 1 - q' (odd q) maps (u, H) to (T - 1 - u, 15 - H); q' -> N - q'
  // (even q) maps it to (T + R3 - 1 - u, 15 - H) for u >= R3, to (R3 - u, 15 -
  // H) for 0 < u < R3, and (0, H) to (0, 16 - H), for which entries 1 .. 8 of
  // u = 0 (the last is bin N / 2) are stored again in [N, N + 8).
  static constexpr int TAB = N + 8;
  __host__ __device__ static constexpr int tab_index(int qq, int half) {  // qq < N / 2
    return (half ? 0 : N / 2) + 8 * ((qq / 16) % R3 + R3 * (qq % 16)) + qq / D3_SPAN;
  }
  // the second place of bin q' = qq of half 0 (qq <= N / 2), or -1
  __host__ __device__ static constexpr int tab_again(int qq) {
    return qq > 0 && qq % D3_SPAN == 0 ? N - 1 + qq / D3_SPAN : -1;
  }
  __host__ __device__ static constexpr int tab_own(int u, int half) { return (half ? 0 : N / 2) + 8 * u; }
  // first of the 8 entries of thread u's mirrored bins, H = 15 down to 8
  __host__ __device__ static constexpr int tab_mirror(int u, int half) {
    return half ? 8 * (T - 1 - u) : (u == 0 ? N : N / 2 + 8 * (u < R3 ? R3 - u : T + R3 - 1 - u));
  }
};

// 16 bytes of table entries, loaded together
struct alignas(16) cw_tab16 {
  float v[4];
};

// A thread's 16 entries of one half of one table row, by register.
template <int N, typename TO>
__device__ __forceinline__ void cw_load_tab(const TO* row, int u, int half, TO* e) {
  using S = cw_shape<N>;
  constexpr int W = (int)sizeof(TO) / 2;  // 16-byte pieces of 8 entries
  constexpr int PER = 8 / W;              // entries per piece
  const cw_tab16* own = reinterpret_cast<const cw_tab16*>(row + S::tab_own(u, half));
  const cw_tab16* mir = reinterpret_cast<const cw_tab16*>(row + S::tab_mirror(u, half));
#pragma unroll
  for (int i = 0; i < W; ++i) {
    const cw_tab16 a = own[i], b = mir[i];
#pragma unroll
    for (int j = 0; j < PER; ++j) {
      TO x, y;
      __builtin_memcpy(&x, &a.v[j * (4 / PER)], sizeof(TO));
      __builtin_memcpy(&y, &b.v[j * (4 / PER)], sizeof(TO));
      e[S::d3_reg(i * PER + j)] = x;
      e[S::d3_reg(15 - (i * PER + j))] = y;
    }
  }
}
// Whether the bin of register r of thread u is below the reflection (sign
// +1; bin N / 2 of half 0, thread 0's H = 8, is its own mirror).
template <int N>
__host__ __device__ constexpr bool cw_direct(int u, int r, int half) {
  constexpr int D = N / 2;
  return cw_shape<N>::d3_off(r) < D || (half == 0 && cw_shape<N>::d3_off(r) == D && u == 0);
}

// Orders LDS accesses of the T threads of a column: inside one wave, or
// across the workgroup.
template <int T>
__device__ __forceinline__ void cw_sync() {
  if constexpr (T <= 64) wave_sync();
  else __syncthreads();
}

// Keeps the instruction scheduler from moving work across a phase boundary
// (loads hoisted from later phases would not fit the registers).
#ifndef SG_CW_FENCE
#define SG_CW_FENCE() __builtin_amdgcn_sched_barrier(0)
#endif

// This thread's twiddles: w_N^(t k1) and w_T^(t0 k2), in registers (KEEP) or
// read from the table where they are used.
template <int N, typename R, bool KEEP1, bool KEEP2>
struct cw_tw {
  using S = cw_shape<N>;
  cx<R> a[KEEP1 ? 16 : 1], b[KEEP2 ? 16 : 1];
  const cx<R>* tab;
  int o1, o2;
  __device__ __forceinline__ void init(const cx<R>* __restrict__ table, int t) {
    tab = table;
    o1 = t;
    o2 = N + t % S::R3;
    if constexpr (KEEP1)
#pragma unroll
      for (int q = 1; q < 16; ++q) a[q] = tab[(unsigned)(o1 + q * S::T)];
    if constexpr (KEEP2 && S::R3 > 1)
#pragma unroll
      for (int q = 1; q < 16; ++q) b[q] = tab[(unsigned)(o2 + q * S::R3)];
  }
  __device__ __forceinline__ void get1(cx<R>* w) const {
    const int o = KEEP1 ? 0 : opaque(o1);
#pragma unroll
    for (int q = 1; q < 16; ++q) {
      if constexpr (KEEP1) w[q] = a[q];
      else w[q] = tab[(unsigned)(o + q * S::T)];
    }
  }
  __device__ __forceinline__ void get2(cx<R>* w) const {
    const int o = KEEP2 ? 0 : opaque(o2);
#pragma unroll
    for (int q = 1; q < 16; ++q) {
      if constexpr (KEEP2) w[q] = b[q];
      else w[q] = tab[(unsigned)(o + q * S::R3)];
    }
  }
};

// Forward transform of NA arrays (slot i of array i at lds + i SLOT).
// sync_before: some thread may still be reading the slots.
template <int N, int NA, typename R, typename TW>
__device__ __forceinline__ void cw_fwd(cx<R> (&v)[NA][16], cx<R>* lds, const TW& tw, bool sync_before, int t) {
  using S = cw_shape<N>;
  {
    cx<R> w[16];
    tw.get1(w);
#pragma unroll
    for (int i = 0; i < NA; ++i) {
      dft16<false>(v[i]);
#pragma unroll
      for (int q = 1; q < 16; ++q) v[i][q] = cmul(v[i][q], w[q]);
    }
  }
  cx<R>* own = lds + (t / S::R3) * S::ROW + t % S::R3;  // (k1, ., t0)
  cx<R>* all = lds + (t / S::R3) * S::STR + t % S::R3;  // (., t1, t0)
  SG_CW_FENCE();
  if (sync_before) cw_sync<S::T>();
#pragma unroll
  for (int i = 0; i < NA; ++i)
#pragma unroll
    for (int q = 0; q < 16; ++q) all[i * S::SLOT + q * S::ROW] = v[i][q];
  cw_sync<S::T>();
  SG_CW_FENCE();
#pragma unroll
  for (int i = 0; i < NA; ++i)
#pragma unroll
    for (int q = 0; q < 16; ++q) v[i][q] = own[i * S::SLOT + q * S::STR];
#pragma unroll
  for (int i = 0; i < NA; ++i) dft16<false>(v[i]);
  SG_CW_FENCE();
  if constexpr (S::R3 > 1) {
    cx<R> w[16];
    tw.get2(w);
    cx<R>* row = lds + (t / S::R3) * S::ROW + (t % S::R3) * S::STR;  // (k1, k2lo, .)
#pragma unroll
    for (int i = 0; i < NA; ++i)
#pragma unroll
      for (int q = 0; q < 16; ++q) own[i * S::SLOT + q * S::STR] = q ? cmul(v[i][q], w[q]) : v[i][q];
    wave_sync();
    SG_CW_FENCE();
#pragma unroll
    for (int i = 0; i < NA; ++i)
#pragma unroll
      for (int r = 0; r < 16; ++r)
        v[i][r] = row[i * S::SLOT + (r / S::R3) * S::R3 * S::STR + r % S::R3];
#pragma unroll
    for (int i = 0; i < NA; ++i)
#pragma unroll
      for (int b = 0; b < 16 / S::R3; ++b) dft<S::R3, false>(&v[i][b * S::R3]);
    wave_sync();
  }
}

// Inverse transform (unnormalised) of NA arrays, input in cw_fwd's output
// order.  sync_before: as above.
template <int N, int NA, typename R, typename TW>
__device__ __forceinline__ void cw_inv(cx<R> (&v)[NA][16], cx<R>* lds, const TW& tw, bool sync_before, int t) {
  using S = cw_shape<N>;
  cx<R>* own = lds + (t / S::R3) * S::ROW + t % S::R3;
  cx<R>* all = lds + (t / S::R3) * S::STR + t % S::R3;
  if constexpr (S::R3 > 1) {
    cx<R>* row = lds + (t / S::R3) * S::ROW + (t % S::R3) * S::STR;
#pragma unroll
    for (int i = 0; i < NA; ++i)
#pragma unroll
      for (int b = 0; b < 16 / S::R3; ++b) dft<S::R3, true>(&v[i][b * S::R3]);
    if (sync_before) cw_sync<S::T>();
#pragma unroll
    for (int i = 0; i < NA; ++i)
#pragma unroll
      for (int r = 0; r < 16; ++r)
        row[i * S::SLOT + (r / S::R3) * S::R3 * S::STR + r % S::R3] = v[i][r];
    wave_sync();
    SG_CW_FENCE();
    cx<R> w[16];
    tw.get2(w);
#pragma unroll
    for (int i = 0; i < NA; ++i)
#pragma unroll
      for (int q = 0; q < 16; ++q) {
        const cx<R> x = own[i * S::SLOT + q * S::STR];
        v[i][q] = q ? cmulc(x, w[q]) : x;
      }
  }
#pragma unroll
  for (int i = 0; i < NA; ++i) dft16<true>(v[i]);
  SG_CW_FENCE();
  if (S::R3 == 1 && sync_before) cw_sync<S::T>();
#pragma unroll
  for (int i = 0; i < NA; ++i)
#pragma unroll
    for (int q = 0; q < 16; ++q) own[i * S::SLOT + q * S::STR] = v[i][q];
  cw_sync<S::T>();
  SG_CW_FENCE();
  {
    cx<R> w[16];
    tw.get1(w);
#pragma unroll
    for (int i = 0; i < NA; ++i) {
#pragma unroll
      for (int q = 0; q < 16; ++q) {
        const cx<R> x = all[i * S::SLOT + q * S::ROW];
        v[i][q] = q ? cmulc(x, w[q]) : x;
      }
      dft16<true>(v[i]);
    }
  }
}

// Single-float entries of both halves and both twiddle sets fit the registers;
// hi + lo pairs are read where they are used, the first set as well.
template <typename TO>
struct cw_keep {
  static constexpr bool on = sizeof(TO) == 4;
};

// exp(-2 pi i e / 32), e < 16
template <typename R>
__host__ __device__ constexpr cx<R> cw_w32(int e) {
  constexpr double c[9] = {1.0, 0.98078528040323044913, 0.92387953251128675613, 0.83146961230254523708,
                           0.70710678118654752440, 0.55557023301960222474, 0.38268343236508977173,
                           0.19509032201612826785, 0.0};
  return e <= 8 ? cx<R>{(R)c[e], (R)-c[8 - e]} : cx<R>{(R)-c[16 - e], (R)-c[e - 8]};
}

// Even k: the bin phases exp(-i pi (c/2M + q/2N)) (CJ: their conjugates) onto
// one half's bins d3_base(u) + D3_SPAN H.  D3_SPAN / 2N = 1 / 32, so each is a constant
// times the phase w0 of H = 0 (H < 8) or w15 of H = 15, whichever is nearer in
// frequency: the bins next to zero on either side, which hold most of a smooth
// density, get the product of the column's and the bin's phase and no more (all
// from w0: 9 % more error at 4096^2, k = 2).
template <int N, bool CJ, typename R>
__device__ __forceinline__ void cw_phase(cx<R> (&a)[16], cx<R> w0, cx<R> w15) {
  using S = cw_shape<N>;
#pragma unroll
  for (int H = 0; H < 16; ++H) {
    const cx<R> p = H < 8 ? cmul(w0, cw_w32<R>(H)) : cmulc(w15, cw_w32<R>(15 - H));
    cx<R>& z = a[S::d3_reg(H)];
    z = CJ ? cmulc(z, p) : cmul(z, p);
  }
}
// exp(-i pi c / 2M), c < M, of the column: the Taylor sums of sine and cosine on
// [0, pi/2) in FP64 to 1e-10, rounded once (the library's sincospi, once per column,
// takes 28 us of the forward and 41 of the adjoint pass at 4096^2).
template <typename R>
__device__ __forceinline__ cx<R> cw_phase_col(int c, int M) {
  const double a = (double)c * (1.57079632679489661923 / M), z = -a * a;
  double cs = 1.0, sn = 1.0;
#pragma unroll
  for (int n = 16; n >= 2; n -= 2) {  // sum of z^(n/2) / n!, of z^(n/2) / (n + 1)!
    cs = 1.0 + z * (1.0 / (n * (n - 1))) * cs;
    sn = 1.0 + z * (1.0 / (n * (n + 1))) * sn;
  }
  return {(R)cs, (R)(-a * sn)};
}

// One column (or, T < 64, the P columns of one wave).  exch: this workgroup
// holds the packed column 0.  t: this thread within its column c, lds: the
// column's two slots.
template <typename R, typename TO, int N, int kind, typename TW>
__device__ __forceinline__ void cw_column(const cx<R>* __restrict__ X, cx<R>* __restrict__ V, int M, int tj,
                                          const TO* __restrict__ tox, const TO* __restrict__ toy,
                                          const cx<R>* __restrict__ r2n, const TW& tw, cx<R>* lds, int c,
                                          int t, bool exch, const cx<R>* __restrict__ xb, int pg) {
  using S = cw_shape<N>;
  constexpr int T = S::T, SL = S::SLOT;
  constexpr bool PRE = cw_keep<TO>::on;
  const bool packed = c == 0;
  const cx<R>* col = X + (int64_t)c * N;
  cx<R> f[2][16];
#pragma unroll
  for (int e = 0; e < 16; ++e) f[0][e] = col[(unsigned)(t + T * e)];
  // the column's padding values (bnd.hpp), in the threads that fold them in
  const cx<R> xv = bnd_value<T>(xb, pg, M, c, t);
  // the spectrum entries (x, y) of one half at this thread's output bins
  const int db = S::d3_base(t);
  auto load_tab = [&](int64_t p, int h, TO (&e)[2][16]) {
    cw_load_tab<N>(tox + p * S::TAB, t, h, e[0]);
    cw_load_tab<N>(toy + p * S::TAB, t, h, e[1]);
  };
  TO tv[2][16];
  if constexpr (PRE) load_tab(c, 0, tv);

  SG_CW_FENCE();
  // ---- forward: even and odd bins of the zero-padded column
  {
    // w_2N^(t + T e), loaded per column (opaque(): not held from one to the next)
    const int tw2 = opaque(t);
    auto w2n_at = [&](int e) -> cx<R> { return r2n[(unsigned)(tw2 + T * e)]; };
#pragma unroll
    for (int e = 0; e < 16; ++e) f[1][e] = cmul(f[0][e], w2n_at(e));
    if (xb) {
      // onto elements 0, 1 (threads 0, 1) and N - 1, N - 2 (the last two)
      if (t < 2) {
        f[0][0] = f[0][0] + xv;
        f[1][0] = f[1][0] - cmul(xv, w2n_at(0));
      } else {  // zero but in the last two
        f[0][15] = f[0][15] + xv;
        f[1][15] = f[1][15] - cmul(xv, w2n_at(15));
      }
    }
  }
  cw_fwd<N, 2>(f, lds, tw, false, t);
  SG_CW_FENCE();
  if constexpr (kind == 1) {
    // this thread's roots of the bin phases
    const int tp = opaque(N + T + t);
    const cx<R> wc = cw_phase_col<R>(c, M);
    const cx<R> ph0 = tw.tab[(unsigned)tp], ph15 = tw.tab[(unsigned)(tp + T)];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const cx<R> w = h ? cmul(wc, fs_half_phase<R>(1.0 / (2.0 * N))) : wc;
      cw_phase<N, false>(f[h], cmul(ph0, w), cmul(ph15, w));
    }
  }

  // ---- one half at a time: the products of both components and their
  // inverses; Y = IFFT(G_e) + w_2N^-j IFFT(G_o)
  constexpr R ex = kind == 1 ? (R)-1 : (R)1;  // reflection sign of the x table (y: -ex)
  cx<R> acc[2][16];
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    cx<R> gg[2][16];
    if (!PRE) load_tab(c, h, tv);
#pragma unroll
    for (int comp = 0; comp < 2; ++comp)
#pragma unroll
      for (int r = 0; r < 16; ++r)
        gg[comp][r] = fs_iA(f[h][r], tv[comp][r], cw_direct<N>(t, r, h) ? (R)1 : (comp ? -ex : ex));
    if (exch) {
      // Packed column: U(q) = C_0 + i C_M, so with U~(q) = conj U(-q)
      //   C_0 = (U + U~) / 2,  C_M = (U - U~) / 2i,
      // and G_0 + i G_M = i (A_0 (U + U~) + A_M (U - U~)) / 2 (odd k).  Even
      // k: u holds U with its phase, whose partner is -conj u(-q) (conj u(0)
      // at q = 0), and the phase of bin M is -i times that of bin 0:
      // i A_0 (u + u~) / 2 + A_M (u - u~) / 2.  Partners through slot h.
      cw_sync<T>();
      cx<R>* sl = lds + h * SL;
#pragma unroll
      for (int r = 0; r < 16; ++r) sl[db + db / 16 + S::d3_off(r) / 16 * 17] = f[h][r];
      cw_sync<T>();
      if (packed) {
        const int own = S::tab_own(t, h), mir = S::tab_mirror(t, h);
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          if (r % 4 == 0) SG_CW_FENCE();  // few entries in flight
          const int H = S::d3_off(r) / S::D3_SPAN;
          const int qq = db + S::d3_off(r);
          const int qm = h == 0 ? (qq == 0 ? 0 : N - qq) : N - 1 - qq;
          cx<R> um = conj(sl[qm + qm / 16]);
          if (kind == 1 && !(h == 0 && qq == 0)) um = cx<R>{-um.x, -um.y};
          const cx<R> u = f[h][r], d = kind == 1 ? cx<R>{u.y - um.y, um.x - u.x} : u - um;  // even k: -i (u - u~)
#pragma unroll
          for (int comp = 0; comp < 2; ++comp) {
            const TO* row0 = (comp ? toy : tox) + (H < 8 ? own + H : mir + 15 - H);
            const R sgn = cw_direct<N>(t, r, h) ? (R)1 : (comp ? -ex : ex);
            const cx<R> z = gg[comp][r] + fs_iA(um, row0[0], sgn) + fs_iA(d, row0[(int64_t)M * S::TAB], sgn);
            gg[comp][r] = cx<R>{(R)0.5 * z.x, (R)0.5 * z.y};
          }
        }
      }
    }
    SG_CW_FENCE();
    if (h == 0 && PRE) load_tab(c, 1, tv);  // in flight during the inverses of half 0
    // h = 0: the slots' last readers of another wave read them before
    // exchange 1's barrier, except for the packed column's partners
    cw_inv<N, 2>(gg, lds, tw, h == 1 || exch, t);
    SG_CW_FENCE();
    if (h == 0) {
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        acc[0][e] = gg[0][e];
        acc[1][e] = gg[1][e];
      }
    } else {
      // w_2N^(t + T e): loaded for even k; for odd k (T / 2N = 1 / 32) w_2N^t times a
      // constant
      const int tw2 = opaque(t);
      const cx<R> wb = r2n[(unsigned)tw2];
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const cx<R> w = kind == 1 ? r2n[(unsigned)(tw2 + T * e)] : cmul(wb, cw_w32<R>(e));
#pragma unroll
        for (int comp = 0; comp < 2; ++comp) {  // as multiply-adds onto the even half
          const cx<R> z = gg[comp][e];
          acc[comp][e] = cx<R>{(acc[comp][e].x + z.x * w.x) + z.y * w.y, (acc[comp][e].y + z.y * w.x) - z.x * w.y};
        }
      }
    }
  }
  // ---- V(c) = Yx + i Yy, V(2M - c) = conj(Yx) + i conj(Yy); packed: V(0) =
  // Re Yx + i Re Yy, V(M) = Im Yx + i Im Yy.  V(p, j) at
  // ((j/tj*2 + p%2)*M + p/2)*tj + j%tj; tj divides T.
  {
    const int ts = opaque(t);
    const int pa = c, pb = packed ? M : 2 * M - c;
    const int64_t o0 = (int64_t)(ts / tj) * 2 * M * tj + ts % tj;
    cx<R>* va = V + ((int64_t)(pa & 1) * M + (pa >> 1)) * tj + o0;
    cx<R>* vb = V + ((int64_t)(pb & 1) * M + (pb >> 1)) * tj + o0;
    const int64_t step = (int64_t)2 * M * T;
    if (!packed) {
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const cx<R> x = acc[0][e], y = acc[1][e];
        va[step * e] = cx<R>{x.x - y.y, x.y + y.x};
        vb[step * e] = cx<R>{x.x + y.y, y.x - x.y};
      }
    } else {
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const cx<R> x = acc[0][e], y = acc[1][e];
        va[step * e] = cx<R>{x.x, y.x};
        vb[step * e] = cx<R>{x.y, y.y};
      }
    }
  }
}

// kind, xb and pg as in k_colfs (kind: its MODE 0 or 1), the tables in the
// order of cw_shape.  A workgroup loops over tiles of P columns
// blockIdx.x, blockIdx.x + gridDim.x, ..., so that its twiddles are read once.
template <typename R, typename TO, int N, int kind>
__global__ void __launch_bounds__(cw_shape<N>::T* cw_shape<N>::P) SG_WAVES_PER_EU(2)
    k_colw(const cx<R>* __restrict__ X, cx<R>* __restrict__ V, int M, int tj, const TO* __restrict__ tox,
           const TO* __restrict__ toy, const cx<R>* __restrict__ r2n, const cx<R>* __restrict__ twc,
           const sg_bgrid* __restrict__ bg, const cx<R>* __restrict__ xb, int pg) {
  using S = cw_shape<N>;
  constexpr int T = S::T;
  if (bg) {
    const sg_bgrid d = grid_desc(bg);
    X = reinterpret_cast<const cx<R>*>(d.X);
    V = reinterpret_cast<cx<R>*>(d.V);
    tox = reinterpret_cast<const TO*>(d.tabx);
    toy = reinterpret_cast<const TO*>(d.taby);
    xb = reinterpret_cast<const cx<R>*>(d.xb);
  }
  __shared__ cx<R> smem[S::P * 2 * S::SLOT];
  const int t0 = S::P == 1 ? threadIdx.x : threadIdx.x % T, g = S::P == 1 ? 0 : threadIdx.x / T;
  cx<R>* lds = smem + g * 2 * S::SLOT;
  cw_tw<N, R, cw_keep<TO>::on, true> tw;
  tw.init(twc, t0);
  const int nt = M / S::P;  // tiles of P columns
  for (int it = blockIdx.x;;) {
    // opaque(): the index arithmetic of a column stays in the loop body
    const int t = opaque(t0);
    const int tile = xcd_tile(it, nt);
    cw_column<R, TO, N, kind>(X, V, M, tj, tox, toy, r2n, tw, lds, tile * S::P + g, t, tile == 0, xb, pg);
    it += gridDim.x;
    if (it >= nt) break;
    cw_sync<T>();  // this column's last LDS reads come before the next one's writes
  }
}

// Adjoint column pass (the arguments and results of k_colfs_adj; kind: its MODE 0
// or 1): per half the transforms of both gradients' spectra, the products with
// the conjugate spectra (conj(i A) = -i A) summed over the components; the
// inverses of both halves; the padding values' share (bnd.hpp; bord, bc).
template <typename R, typename TO, int N, int kind>
__global__ void __launch_bounds__(cw_shape<N>::T) SG_WAVES_PER_EU(2)
    k_colw_adj(const cx<R>* __restrict__ Xx, const cx<R>* __restrict__ Xy, cx<R>* __restrict__ Y, int M, int tj,
               const TO* __restrict__ tox, const TO* __restrict__ toy, const cx<R>* __restrict__ r2n,
               const cx<R>* __restrict__ twc, const sg_bgrid* __restrict__ bg, int bord,
               const double* __restrict__ bc) {
  using S = cw_shape<N>;
  constexpr int T = S::T, SL = S::SLOT;
  static_assert(S::P == 1 && T >= kBndLen, "one column per workgroup, its ends in one element of a thread");
  if (bg) {  // batched: gx spectra in X, gy spectra in the first half of V, output in its second half
    const sg_bgrid d = grid_desc(bg);
    Xx = reinterpret_cast<const cx<R>*>(d.X);
    Xy = reinterpret_cast<const cx<R>*>(d.V);
    Y = reinterpret_cast<cx<R>*>(d.V) + (int64_t)M * N;
    tox = reinterpret_cast<const TO*>(d.tabx);
    toy = reinterpret_cast<const TO*>(d.taby);
  }
  __shared__ cx<R> smem[2 * SL];
  const int t0 = threadIdx.x;
  cw_tw<N, R, cw_keep<TO>::on, true> tw;
  tw.init(twc, t0);
  constexpr R ex = kind == 1 ? (R)-1 : (R)1;  // reflection sign of the x table (y: -ex)
  for (int it = blockIdx.x;;) {
    const int t = opaque(t0);
    const int c = xcd_tile(it, M);
    const bool packed = (c == 0);
    const int db = S::d3_base(t);
    cx<R> hs[2][16];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      cx<R> f[2][16];
      {
        const int tl = opaque(t);
#pragma unroll
        for (int e = 0; e < 16; ++e) {
          f[0][e] = Xx[(int64_t)c * N + (unsigned)(tl + T * e)];
          f[1][e] = Xy[(int64_t)c * N + (unsigned)(tl + T * e)];
        }
      }
      TO tv[2][16];
      if constexpr (cw_keep<TO>::on) {
        cw_load_tab<N>(tox + (int64_t)c * S::TAB, t, h, tv[0]);
        cw_load_tab<N>(toy + (int64_t)c * S::TAB, t, h, tv[1]);
      }
      if (h) {
        const int tw2 = opaque(t);
#pragma unroll
        for (int e = 0; e < 16; ++e) {
          const cx<R> w = r2n[(unsigned)(tw2 + T * e)];  // w_2N^(t + T e)
          f[0][e] = cmul(f[0][e], w);
          f[1][e] = cmul(f[1][e], w);
        }
      }
      SG_CW_FENCE();
      cw_fwd<N, 2>(f, smem, tw, h == 1, t);
      SG_CW_FENCE();
      if constexpr (!cw_keep<TO>::on) {
        cw_load_tab<N>(tox + (int64_t)c * S::TAB, t, h, tv[0]);
        cw_load_tab<N>(toy + (int64_t)c * S::TAB, t, h, tv[1]);
      }
      if constexpr (kind == 1) {
        const int tp = opaque(N + T + t);
        const cx<R> wc = cw_phase_col<R>(c, M), w = h ? cmul(wc, fs_half_phase<R>(1.0 / (2.0 * N))) : wc;
        const cx<R> w0 = cmul(tw.tab[(unsigned)tp], w), w15 = cmul(tw.tab[(unsigned)(tp + T)], w);
        cw_phase<N, true>(f[0], w0, w15);
        cw_phase<N, true>(f[1], w0, w15);
      }
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const bool dir = cw_direct<N>(t, r, h);
        hs[h][r] = fs_iA(f[0][r], tv[0][r], dir ? (R)-1 : -ex) + fs_iA(f[1][r], tv[1][r], dir ? (R)-1 : ex);
      }
      if (packed) {
        // as in cw_column: with u = U (odd k) or U with its conjugate phase (even
        // k), H_0 + i H_M = -i (A_0 (u + u~) + A_M (u - u~)) / 2, and for even k
        // A_M (u - u~) without the -i; x through slot 0, y through slot 1
        cw_sync<T>();
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int at = db + db / 16 + S::d3_off(r) / 16 * 17;
          smem[at] = f[0][r];
          smem[SL + at] = f[1][r];
        }
        cw_sync<T>();
        const int own = S::tab_own(t, h), mir = S::tab_mirror(t, h);
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          if (r % 4 == 0) SG_CW_FENCE();  // few entries in flight
          const int H = S::d3_off(r) / S::D3_SPAN;
          const int qq = db + S::d3_off(r);
          const int qm = h == 0 ? (qq == 0 ? 0 : N - qq) : N - 1 - qq;
          cx<R> z = hs[h][r];
#pragma unroll
          for (int comp = 0; comp < 2; ++comp) {
            cx<R> um = conj(smem[comp * SL + qm + qm / 16]);
            if (kind == 1 && !(h == 0 && qq == 0)) um = cx<R>{-um.x, -um.y};
            const cx<R> u = f[comp][r], d = kind == 1 ? cx<R>{um.y - u.y, u.x - um.x} : u - um;  // even k: i (u - u~)
            const TO* row0 = (comp ? toy : tox) + (H < 8 ? own + H : mir + 15 - H);
            const R sgn = cw_direct<N>(t, r, h) ? (R)-1 : (comp ? ex : -ex);
            z = z + fs_iA(um, row0[0], sgn) + fs_iA(d, row0[(int64_t)M * S::TAB], sgn);
          }
          hs[h][r] = cx<R>{(R)0.5 * z.x, (R)0.5 * z.y};
        }
      }
      SG_CW_FENCE();
    }
    if (packed) cw_sync<T>();
    cw_inv<N, 2>(hs, smem, tw, false, t);
    SG_CW_FENCE();
    cx<R> past{(R)0, (R)0}, before{(R)0, (R)0};  // slots N, N + 1 (threads 0, 1), -1, -2 (the last two)
    const int tw2 = opaque(t);
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      if (e % 4 == 0) SG_CW_FENCE();  // few roots in flight
      const cx<R> o = cmulc(hs[1][e], r2n[(unsigned)(tw2 + T * e)]);
      if (e == 0) past = hs[0][e] - o;
      if (e == 15) before = hs[0][e] - o;
      hs[0][e] = hs[0][e] + o;
    }
    const int ts = opaque(t);
    if (bord) {
      // the gradients found in the padding slots, to the threads of the ends
      cw_sync<T>();
      if (ts < 2) smem[ts] = past;
      if (ts >= T - 2) smem[2 + T - 1 - ts] = before;
      cw_sync<T>();
      const int len = bnd_reach(bord), j1 = T - 1 - ts;
      if (ts < len) hs[0][0] = bnd_add(hs[0][0], smem[2], smem[3], bc, ts);
      if (j1 < len) hs[0][15] = bnd_add(hs[0][15], smem[0], smem[1], bc, j1);
    }
    cx<R>* out = Y + ((int64_t)(c & 1) * (M / 2) + (c >> 1)) * tj + (int64_t)(ts / tj) * M * tj + ts % tj;
    const int64_t step = (int64_t)M * T;
#pragma unroll
    for (int e = 0; e < 16; ++e) out[step * e] = hs[0][e];
    it += gridDim.x;
    if (it >= M) break;
    cw_sync<T>();  // this column's last LDS reads come before the next one's writes
  }
}

// Host side: the twiddle table of cw_shape<N> from root(m, L, re, im) =
// exp(-2 pi i m / L).
template <int N, typename F>
void cw_fill_twiddles(F root, double* re, double* im) {
  using S = cw_shape<N>;
  for (int k1 = 0; k1 < 16; ++k1)
    for (int t = 0; t < S::T; ++t) root(k1 * t, N, re + k1 * S::T + t, im + k1 * S::T + t);
  for (int k2 = 0; k2 < 16; ++k2)
    for (int t0 = 0; t0 < S::R3; ++t0) root(k2 * t0, S::T, re + N + k2 * S::R3 + t0, im + N + k2 * S::R3 + t0);
  for (int u = 0; u < S::T; ++u) {
    double *x = re + N + S::T + u, *y = im + N + S::T + u;
    root(S::d3_base(u), 2 * N, x, y);
    root(S::d3_base(u) + 15 * S::D3_SPAN, 2 * N, x + S::T, y + S::T);
  }
}

}  // namespace sg
