// plane_impl.h -- both axes of a 2D RHS evaluation in one pass over LDS tiles.
//
// A block holds the primitives of 30 x 14 output cells and their halo (three
// cells on every side) and takes the x axis, then the y axis from them; the sum
// of both is the RHS, so no accumulator goes through memory and q is read and
// converted once.  A thread is a centre of the 32 x 16 inner tile.  The x axis
// moves biased values and fluxes between lanes (a row is half a wave) and
// leaves its contribution in registers; the y axis then takes the tile's LDS.
//
// What it replaces: a y pass and an x pass with the accumulator between them and
// a reduction launch for dt.  At these sizes half of a step was the latency of
// seven dependent launches; now there are four.  Two-fluid CFL steps, us, passes
// against this: FP32 64^2 44 / 42, 256^2 42 / 34, 512^2 70 / 65, 701 x 293 63 / 51,
// 1200^2 228 / 212, 2048^2 612 / 563; FP64 512^2 80 / 66, 1200^2 290 / 242; an RHS
// alone at 256^2 in FP32 12.1 / 8.6.  Every size gains, so 2D has no
// other path.  A block's own chain (load, two axes, 8 us at two waves per SIMD)
// bounds the small grids, the issue rate the large ones.  Six waves per SIMD
// instead of five (80 registers, 4 to 10 spilled) measured the same at 512^2 and
// 7 % slower at 2048^2.
#pragma once

#include "device.h"
#include "internal.h"
#include "lanes.h"

namespace mfc {

struct PlaneTile {
  static constexpr int CX = 32, CY = 16;  // centres
  static constexpr int OX = CX - 2, OY = CY - 2;
  static constexpr int SX = CX + 4, SY = CY + 4;  // LDS slots
  static constexpr int NT = CX * CY;
};

// MODE_SIGNAL (with MODE_STEP): the stage takes its dt from the kReduceBlocks
// signal maxima of `sig`.  Every block reduces them for itself, two loads a
// thread behind the tile's own, and block 0 writes dt out: a launch less than a
// reduction of its own (4.4 us).
// The cells of an axis shared out evenly over its tiles.  (A last tile of two or
// four columns takes up to twice a full one's time, as in the axis passes: 92 x 53
// FP64 15.1 us an RHS with full tiles first, 8.7 evenly.)
struct PlaneAxis {
  int width, more;  // cells a tile; the first `more` tiles have one more
  __host__ __device__ int start(int t) const { return t * width + (t < more ? t : more); }
};
struct PlaneSplit {
  unsigned ntx;
  PlaneAxis x, y;
};

template <int NF, typename Real, int MODE, int WV, int RS>
__global__ __launch_bounds__(PlaneTile::NT) void plane_kernel(Params pm, const Real* __restrict__ qk,
                                                              Real* __restrict__ acc, const Real* __restrict__ qn,
                                                              Real* __restrict__ qout, StageArgs st, SignalFuse sig,
                                                              int* __restrict__ flag, PlaneSplit split, unsigned base,
                                                              unsigned tiles) {
  constexpr int D = 2;
  using R = Rows<NF, D>;
  using TL = PlaneTile;
  constexpr int NEQ = R::NEQ;
  constexpr int LS = TL::SX * TL::SY;  // one row of primitives
  constexpr bool kStep = (MODE & MODE_STEP) != 0;
  constexpr bool kSignal = (MODE & MODE_SIGNAL) != 0;
  constexpr bool kNU = WV == kWvNonUniform;
  static_assert((NEQ + 1) * TL::NT <= NEQ * LS, "the y exchange fits the tile's LDS");
  __shared__ Real sh[NEQ * LS];
  __shared__ double smax[kSignal ? TL::NT / 64 : 1];

  // Blocks are dispatched to the eight XCDs in turn: each takes a band of
  // consecutive tiles, which share halo and cache lines.
  const unsigned tile = base + (blockIdx.x & 7u) * (gridDim.x >> 3) + (blockIdx.x >> 3);
  if (tile >= tiles) return;
  const int nx = pm.n[0], ny = pm.n[1];
  const long long nc = pm.ncell;
  const int ix = (int)(tile % split.ntx), iy = (int)(tile / split.ntx);
  const int ox = split.x.start(ix), oy = split.y.start(iy);
  const int wx = split.x.start(ix + 1) - ox, wy = split.y.start(iy + 1) - oy;  // this tile's outputs

  // this thread's centre: the last wave takes the two rows outside the output
  // rows, which the x axis has no work for
  const int tid = threadIdx.x;
  const int a = tid & (TL::CX - 1), k = tid / TL::CX;
  const int r = (k < TL::OY) ? k + 1 : (k == TL::OY ? 0 : TL::CY - 1);
  const int cx = ox - 1 + a, cy = oy - 1 + r;
  const int own = (r + 2) * TL::SX + a + 2;

  // ---- load and convert the tile and its halo ---------------------------------
  // every thread its own centre, the first 176 a cell of the halo too: two
  // columns on both sides of the output rows, two rows above and below the
  // output columns
  constexpr int kHaloX = 4 * TL::OY, kHaloY = 4 * TL::OX;
  int slot[2], px[2], py[2];
  bool live[2];
  px[0] = cx;
  py[0] = cy;
  slot[0] = own;
  live[0] = a <= wx + 3 && r <= wy + 3;
  {
    int sx, sy;
    if (tid < kHaloX) {
      const int h = tid & 3;
      sx = h < 2 ? h : h + TL::CX;
      sy = (tid >> 2) + 3;
    } else {
      const int h = tid - kHaloX, row = h / TL::OX;
      sx = h - row * TL::OX + 3;
      sy = row < 2 ? row : row + TL::CY;
    }
    px[1] = ox - 3 + sx;
    py[1] = oy - 3 + sy;
    slot[1] = sy * TL::SX + sx;
    live[1] = tid < kHaloX + kHaloY && sx <= wx + 5 && sy <= wy + 5;
  }
  Real raw[2][NEQ];
  bool fx[2], fy[2];
#pragma unroll
  for (int it = 0; it < 2; ++it) {
    if (!live[it]) continue;
    const int gx = ghost_index(px[it], nx, pm.bc_lo[0], pm.bc_hi[0], fx[it]);
    const int gy = ghost_index(py[it], ny, pm.bc_lo[1], pm.bc_hi[1], fy[it]);
    const long long cell = (long long)gy * nx + gx;
#pragma unroll
    for (int v = 0; v < NEQ; ++v) raw[it][v] = qk[v * nc + cell];
  }
  if constexpr (kSignal) {
    static_assert(kReduceBlocks == 2 * TL::NT, "two maxima a thread");
    const double m = wave_max(fmax(sig.partial[tid], sig.partial[tid + TL::NT]));
    if ((tid & 63) == 0) smax[tid >> 6] = m;
  }
#pragma unroll
  for (int it = 0; it < 2; ++it) {
    if (!live[it]) continue;
    double U[NEQ], W[NEQ];
#pragma unroll
    for (int v = 0; v < NEQ; ++v) U[v] = double(raw[it][v]);
    if (fx[it]) U[R::MOM] = -U[R::MOM];
    if (fy[it]) U[R::MOM + 1] = -U[R::MOM + 1];
    cons_to_prim<NF, D, Real>(pm, U, W);
#pragma unroll
    for (int v = 0; v < NEQ; ++v) sh[v * LS + slot[it]] = Real(W[v]);
  }
  __syncthreads();

  const WenoK<Real> K = weno_consts(Real(pm.eps));
  const bool out_ok = a >= 1 && a <= wx && r >= 1 && r <= wy;
  // volume fractions of the centre for the alpha source; with RS_KAPILA they
  // carry Kapila's K of the cell
  Real al[2] = {Real(0), Real(0)};
  if constexpr (NF == 2) {
    if (out_ok) {
      al[0] = sh[R::ALPHA * LS + own];
      al[1] = sh[(R::ALPHA + 1) * LS + own];
      if constexpr ((RS & RS_KAPILA) != 0) {
        const double Kc = kapila_K(pm, double(sh[R::E * LS + own]), double(al[0]), double(al[1]));
        al[0] = Real(double(al[0]) + Kc);
        al[1] = Real(double(al[1]) - Kc);
      }
    }
  }
  bool bad = false;

  // ---- x axis: whole waves of output rows ------------------------------------
  const Real ihx = Real(kNU ? (out_ok ? inv_width(pm, 0, cx) : 0.0) : pm.inv_dx[0]);
  Real dx[NEQ];
  if (k < TL::OY) {
    Real WLc[NEQ], WL[NEQ], WR[NEQ], F[NEQ], uf = Real(0);
    const bool centre = r <= wy && a <= wx + 1;
    if (centre) {
      NuK<Real> KN;
      if constexpr (kNU) KN = nu_entry<Real>(pm, 0, cx);
#pragma unroll
      for (int v = 0; v < NEQ; ++v) {
        const Real* f = sh + v * LS + own;
        if constexpr (kNU)
          weno5_nu(f[-2], f[-1], f[0], f[1], f[2], K.eps, KN, WLc[v], WR[v]);
        else
          weno5<WV>(f[-2], f[-1], f[0], f[1], f[2], K, WLc[v], WR[v]);
      }
    }
#pragma unroll
    for (int v = 0; v < NEQ; ++v) WL[v] = lane_shift<kFromPrev>(WLc[v]);
    if (centre && a >= 1) {
      if constexpr ((RS & RS_THORNBER) != 0) thornber<NF, D, 0, Real>(pm, WL, WR);
      bad = riemann<RS, NF, D, 0, Real>(pm, WL, WR, F, uf);
    }
    const Real div = ihx * (lane_shift<kFromNext>(uf) - uf);
#pragma unroll
    for (int v = 0; v < NEQ; ++v) {
      const Real fhi = lane_shift<kFromNext>(F[v]);
      dx[v] = F[v] - fhi;
      if constexpr (NF == 2) {
        if (v == R::ALPHA) dx[v] = ihx * (F[v] - fhi) + al[0] * div;
        if (v == R::ALPHA + 1) dx[v] = ihx * (F[v] - fhi) + al[1] * div;
      }
    }
  }

  // ---- y axis -----------------------------------------------------------------
  const bool centre = a >= 1 && a <= wx && r <= wy + 1;
  Real WL[NEQ], WR[NEQ], F[NEQ], uf = Real(0);
  if (centre) {
    NuK<Real> KN;
    if constexpr (kNU) KN = nu_entry<Real>(pm, 1, cy);
#pragma unroll
    for (int v = 0; v < NEQ; ++v) {
      const Real* f = sh + v * LS + own;
      constexpr int S = TL::SX;
      if constexpr (kNU)
        weno5_nu(f[-2 * S], f[-S], f[0], f[S], f[2 * S], K.eps, KN, WL[v], WR[v]);
      else
        weno5<WV>(f[-2 * S], f[-S], f[0], f[S], f[2 * S], K, WL[v], WR[v]);
    }
  }
  __syncthreads();
  const int e = r * TL::CX + a;
  if (centre) {
#pragma unroll
    for (int v = 0; v < NEQ; ++v) sh[v * TL::NT + e] = WL[v];
  }
  __syncthreads();
  const bool face = centre && r >= 1;
  if (face) {
#pragma unroll
    for (int v = 0; v < NEQ; ++v) WL[v] = sh[v * TL::NT + e - TL::CX];
    if constexpr ((RS & RS_THORNBER) != 0) thornber<NF, D, 1, Real>(pm, WL, WR);
    bad |= riemann<RS, NF, D, 1, Real>(pm, WL, WR, F, uf);
  }
  if (bad) atomicOr(flag, 1);
  // the output cell's q_k and q^n arrive behind the exchange of the fluxes
  const long long cell = (long long)cy * nx + cx;
  Real qkv[kStep ? NEQ : 1], qnv[kStep ? NEQ : 1];
  if constexpr (kStep) {
    if (out_ok) {
#pragma unroll
      for (int v = 0; v < NEQ; ++v) qkv[v] = qk[v * nc + cell];
#pragma unroll
      for (int v = 0; v < NEQ; ++v) qnv[v] = (st.stage != 1) ? qn[v * nc + cell] : Real(0);
    }
  }
  __syncthreads();
  if (face) {
#pragma unroll
    for (int v = 0; v < NEQ; ++v) sh[v * TL::NT + e] = F[v];
    sh[NEQ * TL::NT + e] = uf;
  }
  __syncthreads();
  double dt_block = 0.0;
  if constexpr (kSignal) {
    double m = smax[0];
#pragma unroll
    for (int w = 1; w < TL::NT / 64; ++w) m = fmax(m, smax[w]);
    dt_block = sig.cfl / m;
    if (sig.t_remaining > 0.0 && dt_block > sig.t_remaining) dt_block = sig.t_remaining;
    if (tile == 0 && tid == 0) {
      *sig.smax_out = m;
      *sig.dt_out = dt_block;
      if (sig.dt_user) *sig.dt_user = dt_block;
    }
  }
  if (!out_ok) return;
  const Real ihy = Real(kNU ? inv_width(pm, 1, cy) : pm.inv_dx[1]);
  const Real div = ihy * (sh[NEQ * TL::NT + e + TL::CX] - uf);
  double dt = 0.0;
  if constexpr (kSignal) {
    dt = dt_block;
  } else if constexpr (kStep) {
    dt = st.dt_ptr ? *st.dt_ptr : st.dt;
  }
#pragma unroll
  for (int v = 0; v < NEQ; ++v) {
    Real Dv = ihy * (F[v] - sh[v * TL::NT + e + TL::CX]);
    if constexpr (NF == 2) {
      if (v == R::ALPHA) Dv = Dv + al[0] * div;
      if (v == R::ALPHA + 1) Dv = Dv + al[1] * div;
    }
    // the fused operation of the separate x pass
    const Real rv = (NF == 2 && v >= R::ALPHA) ? Dv + dx[v] : fma(ihx, dx[v], Dv);
    if constexpr (kStep)
      qout[v * nc + cell] = Real(rk3_stage(st.stage, double(qnv[v]), double(qkv[v]), dt, double(rv)));
    else
      acc[v * nc + cell] = rv;
  }
}

// ---------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------
template <int NF, typename Real, int MODE, int WV, int RS>
static hipError_t launch_plane(const Params& pm, const Real* qk, Real* acc, const Real* qn, Real* qout, StageArgs st,
                               int* flag, hipStream_t s, PassTimer* tm, const SignalFuse* sig) {
  using TL = PlaneTile;
  const int ntx = (pm.n[0] + TL::OX - 1) / TL::OX, nty = (pm.n[1] + TL::OY - 1) / TL::OY;
  const unsigned tiles = (unsigned)ntx * (unsigned)nty;
  const PlaneSplit split{(unsigned)ntx, {pm.n[0] / ntx, pm.n[0] % ntx}, {pm.n[1] / nty, pm.n[1] % nty}};
  if (tm) tm->begin(KIND_PASS_X, s);
  // chunks of 2^22 blocks keep the work-items of a launch below 2^32
  constexpr unsigned kChunk = 1u << 22;
  hipError_t e = hipSuccess;
  for (unsigned base = 0; base < tiles && e == hipSuccess; base += kChunk) {
    const unsigned end = (tiles - base < kChunk) ? tiles : base + kChunk;
    hipLaunchKernelGGL((plane_kernel<NF, Real, MODE, WV, RS>), dim3((end - base + 7) / 8 * 8), dim3(TL::NT), 0, s, pm, qk,
                       acc, qn, qout, st, sig ? *sig : SignalFuse{}, flag, split, base, end);
    e = hipGetLastError();
  }
  if (tm) tm->end(KIND_PASS_X, s);
  return e;
}

// One evaluation.  sig: a CFL step's first stage.
template <int NF, typename Real, int WV, int RS>
static hipError_t plane_rhs(const Params& pm, const Real* qk, Real* acc, const Real* qn, Real* qout, StageArgs st,
                            bool final_step, int* flag, hipStream_t s, PassTimer* tm, const SignalFuse* sig) {
  if (!final_step) return launch_plane<NF, Real, MODE_WRITE, WV, RS>(pm, qk, acc, qn, qout, st, flag, s, tm, nullptr);
  if (!sig) return launch_plane<NF, Real, MODE_STEP, WV, RS>(pm, qk, acc, qn, qout, st, flag, s, tm, nullptr);
  if (tm) tm->begin(KIND_SIGNAL, s);
  const hipError_t e = launch_signal_partials<Real>(NF, 2, pm, qk, sig->partial, flag, s);
  if (tm) tm->end(KIND_SIGNAL, s);
  if (e != hipSuccess) return e;
  return launch_plane<NF, Real, MODE_STEP | MODE_SIGNAL, WV, RS>(pm, qk, acc, qn, qout, st, flag, s, tm, sig);
}

}  // namespace mfc
