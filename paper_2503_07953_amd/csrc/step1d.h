// step1d.h -- a whole SSP-RK3 step of a short 1D grid in one block.
//
// A 200-cell shock tube is five dependent launches (signal maxima, dt, three
// stages) of 4.4 us each around less than 1 us of work a stage: 22 us a step.
// One block that keeps the cells in registers and LDS takes 8.5 us at 200 cells
// (1 fluid, FP64; 2 fluids 19.4 -> 9.6) and 8.9 and 13.0 at 510 instead of 17.8
// and 20.1 back to back; what is left is three stages of latency on one CU.
// The grid has to fit a block, one thread per reconstruction centre -1 .. n.  A
// block of 512 leaves the two-fluid kernels their registers (1024 threads spill
// 20 to 96 of them); longer grids take the passes of their own.
//
// Thread t is centre and cell t - 1.  Arithmetic and rounding are those of the
// x pass (same device functions, same order).
#pragma once

#include "device.h"
#include "internal.h"

namespace mfc {

constexpr int kStep1dThreads = 512;

template <int NF, typename Real, int WV, int RS>
__global__ __launch_bounds__(kStep1dThreads) void step1d_kernel(Params pm, Real* __restrict__ q, double cfl,
                                                                double dt_fixed, double t_remaining,
                                                                double* __restrict__ smax_out,
                                                                double* __restrict__ dt_out,
                                                                double* __restrict__ dt_user, int* __restrict__ flag) {
  constexpr int D = 1;
  using R = Rows<NF, D>;
  constexpr int NEQ = R::NEQ;
  // primitives at slots t + 2 (cells -3 .. n + 2); in their place, later in the
  // stage, the biased values and the fluxes
  __shared__ Real sh[(NEQ + 1) * (kStep1dThreads + 4)];
  __shared__ double red[kStep1dThreads / 64];
  __shared__ double dt_s;
  constexpr int LS = kStep1dThreads + 4;
  const int t = threadIdx.x;
  const int n = pm.n[0];
  const int c = t - 1;
  const bool cell = c >= 0 && c < n;
  const bool centre = c <= n;
  const long long nc = pm.ncell;
  Real qn[NEQ], qk[NEQ];
  double W[NEQ];
  bool bad_any = false;
  if (cell) {
#pragma unroll
    for (int v = 0; v < NEQ; ++v) qk[v] = qn[v] = q[v * nc + c];
  }
  const double ihd = (WV == kWvNonUniform) ? (cell ? inv_width(pm, 0, c) : 0.0) : pm.inv_dx[0];

  double dt = dt_fixed;
#pragma unroll 1
  for (int stage = 1; stage <= 3; ++stage) {
    // ---- primitives of the cells, ghosts from their source cells --------------
    double sg = 0.0;
    if (cell) {
      double U[NEQ];
#pragma unroll
      for (int v = 0; v < NEQ; ++v) U[v] = double(qk[v]);
      cons_to_prim<NF, D, Real>(pm, U, W);
#pragma unroll
      for (int v = 0; v < NEQ; ++v) sh[v * LS + t + 2] = Real(W[v]);
      if (stage == 1 && cfl > 0.0) {
        bool b;
        const double x = cell_signal<NF, D>(pm, U, W, b, &ihd);
        bad_any |= b;
        sg = (x > sg) ? x : sg;  // NaN never wins; it is flagged instead
      }
    }
    if (stage == 1 && cfl > 0.0) {
      sg = wave_max(sg);
      if ((t & 63) == 0) red[t >> 6] = sg;
    }
    __syncthreads();
    if (t < 6) {
      // slot of ghost position g is g + 3
      const int g = t < 3 ? t - 3 : n + t - 3;
      bool flip;
      const int src = ghost_index(g, n, pm.bc_lo[0], pm.bc_hi[0], flip);
#pragma unroll
      for (int v = 0; v < NEQ; ++v) {
        const Real x = sh[v * LS + src + 3];
        sh[v * LS + g + 3] = (flip && v == R::MOM) ? -x : x;
      }
    }
    if (stage == 1 && cfl > 0.0 && t == 0) {
      double m = red[0];
      for (int w = 1; w < (int)blockDim.x / 64; ++w) m = fmax(m, red[w]);
      double d = cfl / m;
      if (t_remaining > 0.0 && d > t_remaining) d = t_remaining;
      dt_s = d;
      *smax_out = m;
      *dt_out = d;
    }
    __syncthreads();
    if (stage == 1) {
      if (cfl > 0.0) dt = dt_s;
      if (t == 0 && dt_user) *dt_user = dt;
    }

    // ---- WENO at centre c, HLLC at the face c - 1/2 ----------------------------
    Real WLc[NEQ], WR[NEQ];
    Real al[2] = {Real(0), Real(0)};
    if (centre) {
      const WenoK<Real> K = weno_consts(Real(pm.eps));
      NuK<Real> KN;
      if constexpr (WV == kWvNonUniform) KN = nu_entry<Real>(pm, 0, c);
#pragma unroll
      for (int v = 0; v < NEQ; ++v) {
        const Real* f = sh + v * LS + t;
        if constexpr (WV == kWvNonUniform)
          weno5_nu(f[0], f[1], f[2], f[3], f[4], K.eps, KN, WLc[v], WR[v]);
        else
          weno5<WV>(f[0], f[1], f[2], f[3], f[4], K, WLc[v], WR[v]);
      }
      if constexpr (NF == 2) {
        al[0] = sh[R::ALPHA * LS + t + 2];
        al[1] = sh[(R::ALPHA + 1) * LS + t + 2];
        if constexpr ((RS & RS_KAPILA) != 0) {
          const double Kc = kapila_K(pm, double(sh[R::E * LS + t + 2]), double(al[0]), double(al[1]));
          al[0] = Real(double(al[0]) + Kc);
          al[1] = Real(double(al[1]) - Kc);
        }
      }
    }
    __syncthreads();
    if (centre) {
#pragma unroll
      for (int v = 0; v < NEQ; ++v) sh[v * LS + t] = WLc[v];
    }
    __syncthreads();
    Real F[NEQ];
    Real uf = Real(0);
    const bool face = centre && c >= 0;
    if (face) {
      Real WL[NEQ];
#pragma unroll
      for (int v = 0; v < NEQ; ++v) WL[v] = sh[v * LS + t - 1];
      if constexpr ((RS & RS_THORNBER) != 0) thornber<NF, D, 0, Real>(pm, WL, WR);
      bad_any |= riemann<RS, NF, D, 0, Real>(pm, WL, WR, F, uf);
    }
    __syncthreads();
    if (face) {
#pragma unroll
      for (int v = 0; v < NEQ; ++v) sh[v * LS + t] = F[v];
      sh[NEQ * LS + t] = uf;
    }
    __syncthreads();

    // ---- stage update of cell c ---------------------------------------------------
    if (cell) {
      const Real ih = Real(ihd);
      const Real div = ih * (sh[NEQ * LS + t + 1] - uf);
      double Uc[NEQ];
      if constexpr (sizeof(Real) == 8) prim_to_cons<NF, D, Real>(pm, W, Uc);
#pragma unroll
      for (int v = 0; v < NEQ; ++v) {
        Real r = ih * (F[v] - sh[v * LS + t + 1]);
        if constexpr (NF == 2) {
          if (v == R::ALPHA) r = r + al[0] * div;
          if (v == R::ALPHA + 1) r = r + al[1] * div;
        }
        const double uk = sizeof(Real) == 8 ? Uc[v] : double(qk[v]);
        qk[v] = Real(rk3_stage(stage, double(qn[v]), uk, dt, double(r)));
      }
    }
    __syncthreads();
  }
  if (cell) {
#pragma unroll
    for (int v = 0; v < NEQ; ++v) q[v * nc + c] = qk[v];
  }
  if (bad_any) atomicOr(flag, 1);
}

// Whether a grid's step is taken in one block.
inline bool step1d_fits(int ndim, const Params& pm) { return ndim == 1 && pm.n[0] + 2 <= kStep1dThreads; }

template <int NF, typename Real, int WV, int RS>
static hipError_t launch_step1d_t(const Params& pm, Real* q, double cfl, double dt_fixed, double t_remaining,
                                  double* smax_out, double* dt_out, double* dt_user, int* flag, hipStream_t s,
                                  PassTimer* tm) {
  const int threads = (pm.n[0] + 2 + 63) / 64 * 64;
  if (tm) tm->begin(KIND_PASS_X, s);
  hipLaunchKernelGGL((step1d_kernel<NF, Real, WV, RS>), dim3(1), dim3((unsigned)threads), 0, s, pm, q, cfl, dt_fixed,
                     t_remaining, smax_out, dt_out, dt_user, flag);
  if (tm) tm->end(KIND_PASS_X, s);
  return hipGetLastError();
}

}  // namespace mfc
