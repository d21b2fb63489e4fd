// Host build of what the kernels run around one interface (interface_fluxes of
// hweno_math.h, side_vjp of hweno_adjoint.h), driven from tests/test_host_fluxes.py:
//   flux_host g0 g1 g2 eps gamma
// then each input line is <op> <prec> <an> <alpha> <values...>, prec 'd' or 'f'; a
// stencil is four points of U, h Dn, h Dt each:
//   a  4 x 3 values            linear advection: fh hh xx
//   p  4 x 12 values           2D Euler, characteristic fields: fh hh xx (4 each)
//   c  4 x 12 values           2D Euler, component by component: the same
//   P  4 x 12 values, gfh[4]   adjoint of fh: gU, g(h Dn) of the four points (characteristic)
//   C  4 x 12 values, gfh[4]   the same, component by component
// and prints its results on one line, 17 significant digits each.
#include <cstdio>
#include <cstdlib>

#include "../../paper_2207_05258_amd/csrc/hweno_adjoint.h"

using namespace hweno;

static double g[3], eps, gam;

template <typename T>
static Consts<T> consts() {
  Consts<T> k{};
  k.rw.g0 = T(g[0]), k.rw.g1 = T(g[1]), k.rw.g2 = T(g[2]), k.rw.eps = T(eps);
  k.rb = recon_blend(T(g[1]), T(g[2]), T(eps));
  k.gm1 = T(gam - 1.0);
  k.gam = T(gam);
  return k;
}

template <typename T, int PHYS, int M, bool PROJ>
static void flux(T an, T alpha, const T* v) {
  auto ld = [&](int s, T* U, T* Dn, T* Dt) {
    for (int c = 0; c < M; ++c)
      U[c] = v[3 * M * s + c], Dn[c] = v[3 * M * s + M + c], Dt[c] = v[3 * M * s + 2 * M + c];
  };
  T o[3][M];
  interface_fluxes<T, PHYS, M, true, PROJ>(ld, alpha, an, consts<T>(), o[0], o[1], o[2]);
  for (auto& r : o)
    for (T x : r) std::printf("%.17g ", double(x));
  std::printf("\n");
}

// as the adjoint kernel puts the pieces together: both sides, the reconstructed
// fields' way back through the Roe average, the point fluxes last
template <typename T, bool PROJ>
static void adjoint(T alpha, const T* v, const T* gf) {
  constexpr int M = 4;
  const Consts<T> k = consts<T>();
  auto ld = [&](int s, T* U, T* Dn) {
    for (int c = 0; c < M; ++c) U[c] = v[12 * s + c], Dn[c] = v[12 * s + M + c];
  };
  Eigen<T, M> eg{};
  EigenAdj<T> ge;
  T gw[M], w[M] = {}, gU[4][M] = {}, gN[4][M] = {};
  if (PROJ) {
    eg.roe(v + 12, v + 24, k.gm1);
    back_T(eg, gf, gw);
  } else {
    for (int c = 0; c < M; ++c) gw[c] = gf[c];
  }
  for (int c = 0; c < M; ++c) gw[c] *= T(1.0 / 6.0);
  for (int side = 0; side < 2; ++side) {
    const bool plus = side == 0;
    const T al = plus ? alpha : -alpha;
    T gx[3][M], gy[3][M];
    side_vjp<T, PH_EULER, M, PROJ>(ld, plus, alpha, T(0), k, eg, gw, gf, w, ge, gx[0], gy[0], gx[1],
                                   gy[1], gx[2], gy[2]);
    for (int r = 0; r < 3; ++r) {
      const int s = plus ? r : 3 - r;
      const T* p = v + 12 * s;
      for (int c = 0; c < M; ++c) gU[s][c] += al * gx[r][c], gN[s][c] += al * gy[r][c];
      point_fluxes_vjp<T, PH_EULER, M, false>(p, p + M, p + M, k, T(0), gx[r], gy[r], nullptr, gU[s],
                                              gN[s], nullptr);
    }
  }
  if (PROJ) {
    for (T& x : w) x *= T(1.0 / 6.0);
    back_eigen_adj(eg, w, gf, ge);
    roe_vjp<T, M>(v + 12, v + 24, k.gm1, ge, gU[1], gU[2]);
  }
  for (int s = 0; s < 4; ++s) {
    for (T x : gU[s]) std::printf("%.17g ", double(x));
    for (T x : gN[s]) std::printf("%.17g ", double(x));
  }
  std::printf("\n");
}

template <typename T>
static void run(char op, const double* in) {
  T v[52];
  for (int i = 0; i < 52; ++i) v[i] = T(in[2 + i]);
  const T an = T(in[0]), alpha = T(in[1]);
  switch (op) {
    case 'a': flux<T, PH_LINADV, 1, false>(an, alpha, v); break;
    case 'p': flux<T, PH_EULER, 4, true>(an, alpha, v); break;
    case 'c': flux<T, PH_EULER, 4, false>(an, alpha, v); break;
    case 'P': adjoint<T, true>(alpha, v, v + 48); break;
    default: adjoint<T, false>(alpha, v, v + 48); break;
  }
}

int main(int argc, char** argv) {
  if (argc != 6) {
    std::fprintf(stderr, "usage: flux_host g0 g1 g2 eps gamma\n");
    return 2;
  }
  for (int i = 0; i < 3; ++i) g[i] = std::atof(argv[1 + i]);
  eps = std::atof(argv[4]);
  gam = std::atof(argv[5]);
  char op, prec;
  while (std::scanf(" %c %c", &op, &prec) == 2) {
    const int n = 2 + (op == 'a' ? 12 : op == 'p' || op == 'c' ? 48 : 52);
    double v[54] = {};
    for (int i = 0; i < n; ++i)
      if (std::scanf("%lf", &v[i]) != 1) return 3;
    if (prec == 'd')
      run<double>(op, v);
    else
      run<float>(op, v);
  }
  return 0;
}
