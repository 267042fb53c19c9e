// The double arithmetic of csrc/device.h, adjoint.h and nu_table.h
// compiled for the CPU, with the fused
// multiply-adds of the device build, behind plain arrays: tests/test_arith_cpu.py.
#include "../../paper_2503_07953_amd/csrc/adjoint.h"
#include "../../paper_2503_07953_amd/csrc/device.h"
#include "../../paper_2503_07953_amd/csrc/nu_table.h"

#include <type_traits>

using namespace mfc;

extern "C" {

// Both biased values of m reconstruction centres: f is five rows of m values.
// variant: 0 WENO5-JS, 1 WENO5-Z, 3 WENO5-M.
void arith_weno(int variant, double eps, int m, const double* f, double* fl, double* fr) {
  const WenoK<double> K = weno_consts(eps);
  for (int i = 0; i < m; ++i) {
    const double a = f[i], b = f[m + i], c = f[2 * m + i], d = f[3 * m + i], e = f[4 * m + i];
    if (variant == 1)
      weno5_z(a, b, c, d, e, K, fl[i], fr[i]);
    else if (variant == 3)
      weno5_m(a, b, c, d, e, K, fl[i], fr[i]);
    else
      weno5_js(a, b, c, d, e, K, fl[i], fr[i]);
  }
}

// WENO5-JS adjoint of m centres: cotangents gL, gR of both values to those of the
// four differences (gD: four rows of m).
void arith_weno_js_vjp(double eps, int m, const double* f, const double* gL, const double* gR, double* gD) {
  const WenoK<double> K = weno_consts(eps);
  for (int i = 0; i < m; ++i) {
    double g[4];
    weno_js_centre_vjp(f[i], f[m + i], f[2 * m + i], f[3 * m + i], f[4 * m + i], K, gL[i], gR[i], g);
    for (int k = 0; k < 4; ++k) gD[k * m + i] = g[k];
  }
}

// WENO5-JS at the centre 2 of five cells of an axis with the given six faces, m
// stencils f; base: the 24 rows of its table entry that the folded ones come from.
int arith_weno_nu(double eps, const double* faces, int m, const double* f, double* fl, double* fr, double* base) {
  Params pm = {};
  pm.n[0] = 5;
  pm.bc_lo[0] = pm.bc_hi[0] = BC_EXTRAP;
  std::vector<double> tab;
  if (!build_axis_table(pm, 0, std::vector<double>(faces, faces + 6), 0.0, tab)) return 1;
  pm.nu[0] = tab.data();
  for (int r = 0; r < 24; ++r) base[r] = tab[r * 11 + 2 + 3];
  const NuK<double> K = nu_entry<double>(pm, 0, 2);
  for (int i = 0; i < m; ++i)
    weno5_nu(f[i], f[m + i], f[2 * m + i], f[3 * m + i], f[4 * m + i], eps, K, fl[i], fr[i]);
  return 0;
}

// Fluxes and face velocity of m faces of a 2D grid along x with the option bits of
// `options` (RS_*): rows of m values.  vjp_uf: the face velocity as the adjoint forms it.
void arith_face(int options, int nf, const double* gamma, const double* pi_inf, int m, const double* wl, const double* wr,
                double* flux, double* uf, double* vjp_uf) {
  Params pm = {};
  for (int i = 0; i < 2; ++i) {
    const int k = i < nf ? i : 0;
    pm.G[i] = 1.0 / (gamma[k] - 1.0);
    pm.P[i] = gamma[k] * pi_inf[k] / (gamma[k] - 1.0);
  }
  auto face = [&](auto options_, auto nf_) {
    constexpr int RS = decltype(options_)::value, NF = decltype(nf_)::value, NEQ = Rows<NF, 2>::NEQ;
    for (int i = 0; i < m; ++i) {
      double L[NEQ], R[NEQ], F[NEQ], Fb[NEQ], Lb[NEQ], Rb[NEQ];
      for (int v = 0; v < NEQ; ++v) {
        L[v] = wl[v * m + i];
        R[v] = wr[v * m + i];
        Fb[v] = 1.0;
        Lb[v] = Rb[v] = 0.0;
      }
      if constexpr ((RS & RS_THORNBER) != 0) thornber<NF, 2, 0, double>(pm, L, R);
      riemann<RS, NF, 2, 0, double>(pm, L, R, F, uf[i]);
      riemann_vjp<RS, NF, 2, 0>(pm, L, R, Fb, 1.0, Lb, Rb, &vjp_uf[i]);
      for (int v = 0; v < NEQ; ++v) flux[v * m + i] = F[v];
    }
  };
  auto fluids = [&](auto options_) {
    if (nf == 1)
      face(options_, std::integral_constant<int, 1>());
    else
      face(options_, std::integral_constant<int, 2>());
  };
  switch (options) {
    case RS_HLL: fluids(std::integral_constant<int, RS_HLL>()); break;
    case RS_THORNBER: fluids(std::integral_constant<int, RS_THORNBER>()); break;
    case RS_APC: fluids(std::integral_constant<int, RS_APC>()); break;
    default: fluids(std::integral_constant<int, 0>()); break;
  }
}

}  // extern "C"
