// vjp.hip -- dispatch of the RHS adjoint over the reconstruction variants
// (vjp_wv*.hip), and the adjoints of the field conversions.
#include "vjp_impl.h"

namespace mfc {

MFC_EXTERN_VJP(0)
MFC_EXTERN_VJP(1)
MFC_EXTERN_VJP(2)
MFC_EXTERN_VJP(3)
MFC_EXTERN_VJP(4)

hipError_t launch_rhs_vjp(int nf, int ndim, const Params& pm, const double* q, const double* rbar, double* qbar,
                          double* wsum, bool accumulate, hipStream_t s, PassTimer* tm, const StageEpi* epi) {
  const StageEpi ep = epi ? *epi : StageEpi{0, 0.0, nullptr, nullptr, nullptr};
  if (pm.nu[0] || pm.nu[1] || pm.nu[2])
    return launch_rhs_vjp_wv<kWvNonUniform>(nf, ndim, pm, q, rbar, qbar, wsum, accumulate, s, tm, ep);
  switch (pm.weno_variant) {
    case 1: return launch_rhs_vjp_wv<1>(nf, ndim, pm, q, rbar, qbar, wsum, accumulate, s, tm, ep);
    case 2: return launch_rhs_vjp_wv<2>(nf, ndim, pm, q, rbar, qbar, wsum, accumulate, s, tm, ep);
    case 3: return launch_rhs_vjp_wv<3>(nf, ndim, pm, q, rbar, qbar, wsum, accumulate, s, tm, ep);
    default: return launch_rhs_vjp_wv<0>(nf, ndim, pm, q, rbar, qbar, wsum, accumulate, s, tm, ep);
  }
}

// ---------------------------------------------------------------------------
// per-cell conversions' adjoints
// ---------------------------------------------------------------------------
template <int NF, int D, bool TO_CONS>
__global__ __launch_bounds__(256) void convert_vjp_kernel(Params pm, const double* __restrict__ x,
                                                          const double* __restrict__ ybar, double* __restrict__ xbar,
                                                          int accumulate) {
  using R = Rows<NF, D>;
  constexpr int NEQ = R::NEQ;
  const long long nc = pm.ncell;
  for (long long c = (long long)blockIdx.x * blockDim.x + threadIdx.x; c < nc; c += (long long)gridDim.x * blockDim.x) {
    double X[NEQ], Yb[NEQ], Xb[NEQ];
#pragma unroll
    for (int v = 0; v < NEQ; ++v) {
      X[v] = x[v * nc + c];
      Yb[v] = ybar[v * nc + c];
      Xb[v] = 0.0;
    }
    if constexpr (TO_CONS)
      prim_to_cons_vjp<NF, D>(pm, X, Yb, Xb);
    else
      cons_to_prim_vjp<NF, D>(pm, X, Yb, Xb);
#pragma unroll
    for (int v = 0; v < NEQ; ++v) {
      const long long e = v * nc + c;
      xbar[e] = accumulate ? xbar[e] + Xb[v] : Xb[v];
    }
  }
}

hipError_t launch_convert_vjp(int nf, int ndim, bool to_cons, const Params& pm, const double* x, const double* ybar,
                              double* xbar, bool accumulate, hipStream_t s) {
  long long nb = (pm.ncell + 255) / 256;
  if (nb > 65536) nb = 65536;
  dim3 grid((unsigned)nb), block(256);
  const int acc = accumulate ? 1 : 0;
#define MFC_CASE(NF, D)                                                                                       \
  if (nf == NF && ndim == D) {                                                                                \
    if (to_cons)                                                                                              \
      hipLaunchKernelGGL((convert_vjp_kernel<NF, D, true>), grid, block, 0, s, pm, x, ybar, xbar, acc);       \
    else                                                                                                      \
      hipLaunchKernelGGL((convert_vjp_kernel<NF, D, false>), grid, block, 0, s, pm, x, ybar, xbar, acc);      \
    return hipGetLastError();                                                                                 \
  }
  MFC_CASE(1, 1)
  MFC_CASE(1, 2)
  MFC_CASE(1, 3)
  MFC_CASE(2, 1)
  MFC_CASE(2, 2)
  MFC_CASE(2, 3)
#undef MFC_CASE
  return hipErrorInvalidValue;
}

}  // namespace mfc
