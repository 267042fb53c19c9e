// The double arithmetic of csrc/device.h, adjoint.h and nu_table.h
// compiled for the CPU, with the fused
// multiply-adds of the device build, behind plain arrays: tests/test_arith_cpu.py.
#include "../../paper_2503_07953_amd/csrc/adjoint.h"
#include "../../paper_2503_07953_amd/csrc/device.h"
#include "../../paper_2503_07953_amd/csrc/nu_table.h"

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

}  // extern "C"
