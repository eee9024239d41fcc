// Host driver of the CPU emulation of the column kernels as the library launches
// them for every order: no system solved inside, the interpolation system in the
// tables and its padding values as parts (forward) or as the share of the ends
// (adjoint).  Reads the kernel's inputs from a file written by the test, runs it
// over every column, writes its output.  Configuration at compile time:
// EMU_KERNEL (0 k_colfs, 1 k_colfs_xy, 2 k_colfs3, 3 k_colw, 4 k_colfs_adj, 5
// k_specfs), EMU_R (float|double), EMU_TO (table element type), EMU_N, EMU_E,
// EMU_SLOTS, EMU_SPLIT (k_colfs: 1 one launch per component), EMU_KIND (0 odd order,
// 1 even), EMU_ORD (its interpolation system, or 0), EMU_XT (tiled row spectra),
// EMU_PG (parts per padding value).
#include <hip/hip_runtime.h>

#include <stdio.h>
#include <stdlib.h>

#include <cmath>
#include <type_traits>
#include <vector>

#define SG_CW_FENCE() ((void)0)
#include "colfs3.hpp"
#include "colw.hpp"

using namespace sg;
using R = EMU_R;
using TO = EMU_TO;
constexpr int N = EMU_N, E = EMU_E, SLOTS = EMU_SLOTS, KIND = EMU_KIND, ORD = EMU_ORD, XT = EMU_XT, PG = EMU_PG;

template <typename T>
static void rd(FILE* f, std::vector<T>& v, size_t n) {
  v.resize(n);
  if (fread(v.data(), sizeof(T), n, f) != n) {
    fprintf(stderr, "short input\n");
    exit(2);
  }
}

static void root(int m, int L, double* cr, double* ci) {
  const long double a = 6.283185307179586476925286766559005768L * m / L;
  *cr = (double)cosl(a);
  *ci = (double)-sinl(a);
}

// the tables in k_colw's order from the natural one (rows of N + 1: half 0 at [0,
// N / 2], half 1 at N / 2 + 1 + [0, N / 2))
template <typename S>
static std::vector<TO> reorder(const std::vector<TO>& nat, int M) {
  std::vector<TO> out((size_t)(M + 1) * S::TAB);
  for (int p = 0; p <= M; ++p)
    for (int h = 0; h < 2; ++h)
      for (int qq = 0; qq <= N / 2 - h; ++qq) {
        const TO v = nat[(size_t)p * (N + 1) + (h ? N / 2 + 1 : 0) + qq];
        if (qq < N / 2) out[(size_t)p * S::TAB + S::tab_index(qq, h)] = v;
        if (h == 0 && S::tab_again(qq) >= 0) out[(size_t)p * S::TAB + S::tab_again(qq)] = v;
      }
  return out;
}

template <int K>
static void run(FILE* f, FILE* o, int M) {
  const int tj = K == 3 ? 8 : pow2_div(N, sizeof(R) == 4 ? 8 : 2);
  fwrite(&tj, sizeof(int), 1, o);
  std::vector<double> re, im;
  if constexpr (K == 3) {
    using S = cw_shape<K == 3 ? N : 4096>;
    re.resize(S::TW_SIZE), im.resize(S::TW_SIZE);
    cw_fill_twiddles<K == 3 ? N : 4096>(root, re.data(), im.data());
  } else {
    constexpr int TN = K == 2 ? 512 : (K == 3 ? 2048 : N), TE = K == 2 ? 8 : E;  // k_colfs3: its 512-point part
    using S = fs_shape<TN, TE>;
    re.resize(S::TW_SIZE), im.resize(S::TW_SIZE);
    fs_fill_twiddles<TN, TE>(root, re.data(), im.data());
  }
  std::vector<cx<R>> tw(re.size());
  for (size_t i = 0; i < re.size(); ++i) tw[i] = cx<R>{(R)re[i], (R)im[i]};
  if constexpr (K == 5) {
    std::vector<cx<double>> Sg, r2n, twd(re.size());
    for (size_t i = 0; i < re.size(); ++i) twd[i] = cx<double>{re[i], im[i]};
    rd(f, Sg, (size_t)M * 2 * N);
    rd(f, r2n, (size_t)2 * N);
    const int fp32 = std::is_same<TO, double>::value ? 0 : (std::is_same<TO, float>::value ? 2 : 1);
    std::vector<TO> tab((size_t)(M + 1) * (N + 1));
    emu::launch(dim3(M), dim3(N / E), [&] {
      k_specfs<N, E>(Sg.data(), M, tab.data(), KIND, fp32, 0.25, r2n.data(), twd.data(), ORD);
    });
    fwrite(tab.data(), sizeof(TO), tab.size(), o);
  } else {
    std::vector<cx<R>> X, Xy, r2n, xb;
    std::vector<TO> tx, ty;
    std::vector<double> bc;
    rd(f, X, (size_t)M * N);
    if (K == 4) rd(f, Xy, (size_t)M * N);
    rd(f, tx, (size_t)(M + 1) * (N + 1));
    rd(f, ty, (size_t)(M + 1) * (N + 1));
    rd(f, r2n, (size_t)2 * N);
    if (K == 4) rd(f, bc, 2 * kBndLen);
    else rd(f, xb, (size_t)4 * M * PG);
    const cx<R>* pad = ORD ? xb.data() : nullptr;
    std::vector<cx<R>> V((size_t)(K == 4 ? 1 : 2) * M * N, cx<R>{(R)0, (R)0});
    if constexpr (K == 0) {
      auto go = [&](auto comp) {
        emu::launch(dim3(M), dim3(N / E), [&] {
          k_colfs<R, TO, N, KIND, E, SLOTS, decltype(comp)::value>(X.data(), V.data(), M, tj, tx.data(), ty.data(),
                                                                   r2n.data(), tw.data(), nullptr, pad, PG, XT);
        });
      };
      if constexpr (EMU_SPLIT) {
        go(std::integral_constant<int, 1>{});
        go(std::integral_constant<int, 2>{});
      } else {
        go(std::integral_constant<int, 0>{});
      }
    } else if constexpr (K == 1) {
      emu::launch(dim3(M), dim3(N / E), [&] {
        k_colfs_xy<R, TO, N, KIND, E, SLOTS>(X.data(), V.data(), M, tj, tx.data(), ty.data(), r2n.data(), tw.data(),
                                             nullptr, pad, PG, XT);
      });
    } else if constexpr (K == 2) {
      emu::launch(dim3(M), dim3(kC3T), [&] {
        k_colfs3<R, TO, KIND, N / 3>(X.data(), V.data(), M, tj, tx.data(), ty.data(), r2n.data(), tw.data(), nullptr, pad,
                                     PG);
      });
    } else if constexpr (K == 3) {
      using S = cw_shape<K == 3 ? N : 4096>;
      tx = reorder<S>(tx, M);
      ty = reorder<S>(ty, M);
      emu::launch(dim3(2), dim3(S::T * S::P), [&] {  // two workgroups over the columns
        k_colw<R, TO, N, KIND>(X.data(), V.data(), M, tj, tx.data(), ty.data(), r2n.data(), tw.data(), nullptr, pad, PG);
      });
    } else {
      emu::launch(dim3(M), dim3(N / E), [&] {
        k_colfs_adj<R, TO, N, KIND, E, SLOTS, (bool)XT>(X.data(), Xy.data(), V.data(), M, tj, tx.data(), ty.data(),
                                                        r2n.data(), tw.data(), nullptr, ORD, bc.data(), XT);
      });
    }
    fwrite(V.data(), sizeof(cx<R>), V.size(), o);
  }
}

int main(int argc, char** argv) {
  if (argc != 4) {
    fprintf(stderr, "usage: %s M in.bin out.bin\n", argv[0]);
    return 2;
  }
  FILE* f = fopen(argv[2], "rb");
  FILE* o = fopen(argv[3], "wb");
  if (!f || !o) return 2;
  run<EMU_KERNEL>(f, o, atoi(argv[1]));
  fclose(f);
  fclose(o);
  return 0;
}
