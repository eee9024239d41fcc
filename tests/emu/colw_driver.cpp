// Host driver of the CPU emulation of the 16-element column kernels
// (colw.hpp): reads the kernel's inputs from a file written by the test, runs
// it over every column, writes its output.  Configuration at compile time:
// EMU_N, EMU_KIND (0 odd order, 1
// even), EMU_ORD (its interpolation system, or 0), EMU_ADJ (1: the adjoint pass), EMU_TO (table
// element type).
#include <hip/hip_runtime.h>

#include <stdio.h>
#include <stdlib.h>

#include <cmath>
#include <vector>

#define SG_CW_FENCE() ((void)0)
#include "colw.hpp"

using namespace sg;
using R = float;
using TO = EMU_TO;
constexpr int N = EMU_N, KIND = EMU_KIND, ORD = EMU_ORD;

template <typename T>
static void rd(FILE* f, std::vector<T>& v, size_t n) {
  v.resize(n);
  if (fread(v.data(), sizeof(T), n, f) != n) {
    fprintf(stderr, "short input\n");
    exit(2);
  }
}

// a table in the kernel's order from one in the natural order (rows of N + 1:
// half 0 at [0, N/2], half 1 at N/2 + 1 + [0, N/2))
static std::vector<TO> reorder(const std::vector<TO>& nat, int M) {
  using S = cw_shape<N>;
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

int main(int argc, char** argv) {
  if (argc != 4) {
    fprintf(stderr, "usage: %s M in.bin out.bin\n", argv[0]);
    return 2;
  }
  const int M = atoi(argv[1]);
  FILE* f = fopen(argv[2], "rb");
  if (!f) return 2;
  using S = cw_shape<N>;
  std::vector<double> re(S::TW_SIZE), im(S::TW_SIZE);
  cw_fill_twiddles<N>(
      [](int m, int L, double* cr, double* ci) {
        const long double a = 6.283185307179586476925286766559005768L * m / L;
        *cr = (double)cosl(a);
        *ci = (double)-sinl(a);
      },
      re.data(), im.data());
  std::vector<cx<R>> tw(S::TW_SIZE), X, r2n, xb;
  for (int i = 0; i < S::TW_SIZE; ++i) tw[i] = cx<R>{(R)re[i], (R)im[i]};
  std::vector<TO> tx, ty;
  std::vector<cx<R>> Xy;
  std::vector<double> bc;
  rd(f, X, (size_t)M * N);
  if (EMU_ADJ) rd(f, Xy, (size_t)M * N);
  rd(f, tx, (size_t)(M + 1) * (N + 1));
  rd(f, ty, (size_t)(M + 1) * (N + 1));
  rd(f, r2n, (size_t)2 * N);
  if (EMU_ADJ) rd(f, bc, 2 * kBndLen);
  else rd(f, xb, (size_t)4 * M);
  tx = reorder(tx, M);
  ty = reorder(ty, M);
  const int tj = 8;
  FILE* o = fopen(argv[3], "wb");
  fwrite(&tj, sizeof(int), 1, o);
  std::vector<cx<R>> V((size_t)(EMU_ADJ ? 1 : 2) * M * N, cx<R>{(R)0, (R)0});
  // two workgroups over the tiles of columns
#if EMU_ADJ
  emu::launch(dim3(2), dim3(S::T), [&] {
    k_colw_adj<R, TO, N, KIND>(X.data(), Xy.data(), V.data(), M, tj, tx.data(), ty.data(), r2n.data(), tw.data(),
                               nullptr, ORD, bc.data());
  });
#else
  emu::launch(dim3(M / S::P < 2 ? 1 : 2), dim3(S::T * S::P), [&] {
    k_colw<R, TO, N, KIND>(X.data(), V.data(), M, tj, tx.data(), ty.data(), r2n.data(), tw.data(), nullptr,
                           ORD ? xb.data() : nullptr, 1);
  });
#endif
  fwrite(V.data(), sizeof(cx<R>), V.size(), o);
  fclose(f);
  fclose(o);
  return 0;
}
