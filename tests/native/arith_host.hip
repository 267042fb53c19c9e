// The double arithmetic of csrc/device.h compiled for the CPU, with the fused
// multiply-adds of the device build, behind plain arrays: tests/test_arith_cpu.py.
#include "../../paper_2503_07953_amd/csrc/device.h"

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

}  // extern "C"
