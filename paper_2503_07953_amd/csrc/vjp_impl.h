// vjp_impl.h -- the RHS adjoint, one pass per axis, templated on the
// reconstruction variant WV; each vjp_wv*.hip instantiates one variant and
// vjp.hip dispatches among them.
//
// For rhs = L(q) and a cotangent rbar, mfc_rhs_vjp forms qbar = (dL/dq)^T rbar
// in deterministic passes (no atomics).  A pass over axis DIR does, per wave,
// for 64 consecutive positions along the axis:
//   (a) the primitives of the 68 positions that the stencils touch are staged
//       in LDS (ghosts remapped, one conversion per position, rounded as the
//       forward passes round it, so that every face takes the forward's side);
//   (b) WENO at every position's centre (both biased values at once);
//   (c) at every position's low face the face cotangents Fbar = rbar_f/h_f -
//       rbar_{f-1}/h_{f-1} and ufbar = sum_j (alpha_j rbar_alpha_j/h)_{f-1} -
//       (...)_f through HLLC^T;
//   (d) WENO^T at every centre (both sides at once), as cotangents of the four
//       differences of its stencil, summed per edge between positions;
//   (e) the primitive cotangent of every cell: its centre's share plus the edge
//       below minus the edge above, plus those of the ghost positions that the
//       boundary condition fills from it, plus the direct term rbar_alpha div u
//       of this axis.  The first pass writes it, the others add to it, and the
//       last one applies cons->prim^T and writes qbar.
// Neighbouring positions are adjacent lanes: everything between (b) and (e)
// moves by DPP and nothing but the cell's sum goes to memory.
//
// What it replaces: a face pass that wrote the cotangents of all six stencil
// positions of every face (48 doubles a face and axis for two fluids in 3D)
// and a cell pass that gathered them: 2.3 KB per cell through memory, and the
// indicators of a centre formed four times.  RHS adjoint, two fluids: 96 x 80 x
// 72 cells 440 -> 185 us, 128^3 1666 -> 690, 256^2 47.5 -> 28.7, 64^2 25.2 ->
// 20.2.
//
// Lanes 3..60 of a wave are outputs (a cell needs the centres two below to two
// above it and their faces); a line's positions run from -pad to n + pad - 1,
// one line after the other, so that no lane is lost to the grid's size.  Three
// ghost positions a side do, with the fold of (e); a periodic axis wraps its
// positions, and takes five so that every stencil of a cell's centres is whole.
// A ghost holds the state of its source cell (normal momentum negated at a
// slip wall), so the ghost's primitive cotangent reaches the source through
// the source's own cons->prim^T once its normal-velocity entry is negated.
#pragma once

#include "adjoint.h"
#include "internal.h"
#include "lanes.h"

namespace mfc {

static_assert(kWvTable == kWvNonUniform, "one number for the tabulated variant");

// Lines of a block, one per wave: four neighbouring x for the y and z axes, so
// that the block's loads run along x.  (Eight, whole 64-byte runs, leave one
// block to a CU at these registers.)  Blocks go to the eight XCDs in turn; four
// neighbours, which share the 128-byte lines, are kept on one.
struct VjpTile {
  static constexpr int TB = 4;
  static constexpr int NT = 64 * TB;
  static constexpr int SLOTS = 68;  // staged positions of a wave
  static constexpr int LS = 69;     // LDS stride of a line (odd: lines start on different banks)
  static constexpr int OUT = 58;
  static constexpr unsigned GROUP = 4;
};

struct VjpGeom {
  int pad;              // ghost positions a side
  long long lines;      // lines along the axis that a wave's positions run through
  long long segments;   // waves along them
  unsigned xgroups;     // blocks across x (y and z axes)
  unsigned blocks;
};

template <int DIR>
inline VjpGeom vjp_geom(const Params& pm) {
  using TL = VjpTile;
  VjpGeom g;
  g.pad = pm.bc_lo[DIR] == BC_PERIODIC ? 5 : 3;
  const long long P = pm.n[DIR] + 2 * g.pad;
  g.lines = DIR == 0 ? (long long)pm.n[1] * pm.n[2] : (DIR == 1 ? pm.n[2] : pm.n[1]);
  g.segments = (P * g.lines - g.pad - 3 + TL::OUT - 1) / TL::OUT;
  g.xgroups = DIR == 0 ? 1u : (unsigned)((pm.n[0] + TL::TB - 1) / TL::TB);
  const long long blocks = DIR == 0 ? (g.segments + TL::TB - 1) / TL::TB : g.segments * g.xgroups;
  // work-items of a launch stay below 2^32 (0: too many)
  g.blocks = blocks < (1ll << 32) / TL::NT - 64 ? (unsigned)blocks : 0u;
  return g;
}

// Position `pos` of an axis of n cells: the cell whose state it holds and
// whether the normal momentum is negated.  Positions beyond the ghosts (of the
// neighbouring line, or past the last) stay on the last ghost: their state is
// physical and nothing of theirs is used.
template <int DIR>
__device__ __forceinline__ int vjp_cell(const Params& pm, int pos, bool& flip) {
  const int n = pm.n[DIR];
  if (pm.bc_lo[DIR] == BC_PERIODIC) {
    flip = false;
    int c = pos;
    while (c < 0) c += n;
    while (c >= n) c -= n;
    return c;
  }
  const int p = pos < -3 ? -3 : (pos > n + 2 ? n + 2 : pos);
  return ghost_index(p, n, pm.bc_lo[DIR], pm.bc_hi[DIR], flip);
}

// Offset of cell `c` of line `line` (x = `x` for the y and z axes).
template <int DIR>
__device__ __forceinline__ long long vjp_offset(const Params& pm, long long line, int c, int x) {
  const long long nx = pm.n[0], ny = pm.n[1];
  if constexpr (DIR == 0)
    return line * nx + c;
  else if constexpr (DIR == 1)
    return (line * ny + c) * nx + x;
  else
    return ((long long)c * ny + line) * nx + x;
}

template <int NF, int D, int DIR, int WV, int RS>
__global__ __launch_bounds__((VjpTile::NT)) void vjp_axis_kernel(Params pm, VjpGeom gm,
                                                                         const double* __restrict__ q,
                                                                         const double* __restrict__ rbar,
                                                                         double* __restrict__ wsum, int first, int last,
                                                                         double* __restrict__ qbar, int accumulate,
                                                                         StageEpi epi) {
  using R = Rows<NF, D>;
  using TL = VjpTile;
  constexpr int NEQ = R::NEQ;
  constexpr int TB = TL::TB, LS = TL::LS;
  constexpr bool kNU = WV == kWvNonUniform;
  // primitives by row, line and slot (slot = lane + 2); the rows of rbar, and
  // later of the cell sums, of the y and z axes by row, line and lane
  __shared__ double sw[NEQ * TB * LS];
  __shared__ double sp[TB * LS];  // the pressure that WENO^T of its row is taken at
  __shared__ double sr[DIR == 0 ? 1 : NEQ * TB * LS];
  const int tid = threadIdx.x;
  const int lane = tid & 63, b = tid >> 6;
  const int nd = pm.n[DIR];
  const long long nc = pm.ncell;
  const int P = nd + 2 * gm.pad;
  const unsigned j8 = blockIdx.x >> 3;
  const unsigned block = ((j8 / TL::GROUP) * 8u + (blockIdx.x & 7u)) * TL::GROUP + j8 % TL::GROUP;
  if (block >= gm.blocks) return;
  // x axis: each wave a segment of its own; y, z: one segment, TB neighbouring x
  const int x0 = DIR == 0 ? 0 : (int)(block % gm.xgroups) * TB;
  const long long seg = DIR == 0 ? (long long)block * TB + b : block / gm.xgroups;
  const long long line0 = seg * TL::OUT / P;
  const int rem0 = (int)(seg * TL::OUT - line0 * P);
  // line and position of the element k (-2 .. 65) places into the segment; past
  // either end of the grid: the end's ghost
  auto place = [&](int k, long long& line, int& pos) -> bool {
    const unsigned r = (unsigned)(rem0 + k + P);
    const unsigned dl = r / (unsigned)P;
    line = line0 + dl - 1;
    pos = (int)(r - dl * (unsigned)P) - gm.pad;
    if (line < 0) {
      line = 0;
      pos = -gm.pad;
    } else if (line >= gm.lines) {
      line = gm.lines - 1;
      pos = nd + gm.pad - 1;
      return false;
    }
    return true;
  };

  // ---- (a) stage the primitives (and rbar) --------------------------------------
  // x axis: a line's slots are its wave's lanes; y, z: neighbouring threads are
  // neighbouring lines
#pragma unroll 1
  for (int e = DIR == 0 ? lane : tid; e < TL::SLOTS * (DIR == 0 ? 1 : TB); e += DIR == 0 ? 64 : TL::NT) {
    const int bb = DIR == 0 ? b : e % TB;
    const int s = DIR == 0 ? e : e / TB;
    long long line;
    int pos;
    place(s - 2, line, pos);
    bool flip;
    const int c = vjp_cell<DIR>(pm, pos, flip);
    const int x = x0 + bb < pm.n[0] ? x0 + bb : pm.n[0] - 1;
    const long long cell = vjp_offset<DIR>(pm, line, c, x);
    double U[NEQ], W[NEQ];
#pragma unroll
    for (int v = 0; v < NEQ; ++v) U[v] = q[v * nc + cell];
    if constexpr (DIR != 0) {
      if (s >= 2 && s < 66) {
#pragma unroll
        for (int v = 0; v < NEQ; ++v) sr[(v * TB + bb) * LS + s - 2] = rbar[v * nc + cell];
      }
    }
    if (flip) U[R::MOM + DIR] = -U[R::MOM + DIR];
    cons_to_prim<NF, D, double>(pm, U, W);
    sp[bb * LS + s] = pressure_energy_first<NF, D>(pm, U, W);
#pragma unroll
    for (int v = 0; v < NEQ; ++v) sw[(v * TB + bb) * LS + s] = W[v];
  }
  __syncthreads();

  // this lane's position, its cell and what is real about it
  long long line;
  int pos;
  const bool on_grid = place(lane, line, pos);
  const bool wrap = pm.bc_lo[DIR] == BC_PERIODIC;
  bool flip0;
  const int cell_i = vjp_cell<DIR>(pm, pos, flip0);
  const bool x_ok = DIR == 0 || x0 + b < pm.n[0];
  const bool inside = pos >= 0 && pos < nd;
  const bool real_cell = wrap || inside;             // its rbar counts
  const bool real_face = wrap || (pos >= 0 && pos <= nd);  // its low face is one of the grid's
  const bool out_ok = x_ok && inside && on_grid && lane >= 3 && lane <= 60;
  const double ih = kNU ? inv_width(pm, DIR, cell_i) : pm.inv_dx[DIR];
  auto Wat = [&](int v, int k) -> double { return sw[(v * TB + b) * LS + lane + k]; };  // k = 2: own position

  const WenoK<double> K = weno_consts(pm.eps);
  const long long nst = (long long)nd + 6;
  const double* cf = nullptr;
  NuK<double> KN;
  if constexpr (kNU) {
    // table entries of the centres -1 .. n (wrapped positions: their cell's)
    const int ct = wrap ? cell_i : (pos < -1 ? -1 : (pos > nd ? nd : pos));
    cf = pm.nu[DIR] + (ct + 3);
    KN = nu_entry<double>(pm, DIR, ct);
  }

  // ---- (b) WENO at the centre; the left state of the low face from the lane below
  double WL[NEQ], WR[NEQ];
#pragma unroll
  for (int v = 0; v < NEQ; ++v) {
    double wl;
    if constexpr (kNU)
      weno5_nu(Wat(v, 0), Wat(v, 1), Wat(v, 2), Wat(v, 3), Wat(v, 4), pm.eps, KN, wl, WR[v]);
    else
      weno5<WV>(Wat(v, 0), Wat(v, 1), Wat(v, 2), Wat(v, 3), Wat(v, 4), K, wl, WR[v]);
    WL[v] = lane_shift<kFromPrev>(wl);
  }

  // ---- (c) face cotangents and HLLC^T ------------------------------------------------
  double Fb[NEQ], ra[2] = {0.0, 0.0};
  double ufb = 0.0, Kc = 0.0;
  if constexpr (NF == 2 && (RS & RS_KAPILA) != 0) Kc = kapila_K(pm, Wat(R::E, 2), Wat(R::ALPHA, 2), Wat(R::ALPHA + 1, 2));
  {
    const long long cell = vjp_offset<DIR>(pm, line, cell_i, 0);
#pragma unroll
    for (int v = 0; v < NEQ; ++v) {
      double r;
      if constexpr (DIR == 0)
        r = rbar[v * nc + cell];
      else
        r = sr[(v * TB + b) * LS + lane];
      r = real_cell ? r : 0.0;
      if constexpr (NF == 2) {
        // the alpha rows' source factors: alpha_i, or alpha_i +- K (RS_KAPILA)
        if (v == R::ALPHA) {
          ra[0] = r;
          ufb -= ih * ((Wat(v, 2) + Kc) * r);
        }
        if (v == R::ALPHA + 1) {
          ra[1] = r;
          ufb -= ih * ((Wat(v, 2) - Kc) * r);
        }
      }
      const double hr = ih * r;
      Fb[v] = hr - lane_shift<kFromPrev>(hr);
    }
    ufb = ufb - lane_shift<kFromPrev>(ufb);
  }
  double WLb[NEQ], WRb[NEQ], uf;
#pragma unroll
  for (int v = 0; v < NEQ; ++v) WLb[v] = WRb[v] = 0.0;
  // the low-Mach correction precedes the face solver; its adjoint follows the
  // solver's
  double uL0 = 0.0, uR0 = 0.0;
  if constexpr ((RS & RS_THORNBER) != 0) {
    uL0 = WL[R::MOM + DIR];
    uR0 = WR[R::MOM + DIR];
    thornber<NF, D, DIR, double>(pm, WL, WR);
  }
  riemann_vjp<RS, NF, D, DIR>(pm, WL, WR, Fb, ufb, WLb, WRb, &uf);
  if constexpr ((RS & RS_THORNBER) != 0) thornber_vjp<NF, D, DIR>(pm, WL, WR, uL0, uR0, WLb, WRb);
  const double div = ih * (lane_shift<kFromNext>(uf) - uf);

  // compiler-only memory barrier: the stencil values are read from LDS again
  // below instead of being kept live in registers across the HLLC adjoint
  asm volatile("" ::: "memory");

  // ---- (d), (e) WENO^T, edge sums, cell sums ------------------------------------------
  // boundary folds are formed by the waves that hold a boundary cell
  const bool fold = !wrap && __any(inside && (pos < 3 || pos >= nd - 3));
  const bool wall_lo = pm.bc_lo[DIR] == BC_SLIPWALL, wall_hi = pm.bc_hi[DIR] == BC_SLIPWALL;
  double wb[NEQ];
#pragma unroll
  for (int v = 0; v < NEQ; ++v) {
    // a face that is none of the grid's gives nothing, whatever its states
    const double gR = real_face ? WRb[v] : 0.0;
    const double gL = lane_shift<kFromNext>(real_face ? WLb[v] : 0.0);
    double gD[4];
    const double* f = (v == R::E) ? &sp[b * LS + lane] : &sw[(v * TB + b) * LS + lane];
    weno_centre_vjp<WV>(f[0], f[1], f[2], f[3], f[4], K, cf, nst, gL, gR, gD);
    const double ctr = gL + gR;
    // difference k of the centre c is the edge above position c - 2 + k: the
    // edge above this position collects gD[2] of its own centre, gD[1] and
    // gD[0] of the two above and gD[3] of the one below
    double t = lane_shift<kFromNext>(gD[0]) + gD[1];
    t = lane_shift<kFromNext>(t) + gD[2];
    const double G = t + lane_shift<kFromPrev>(gD[3]);
    double s = (ctr + lane_shift<kFromPrev>(G)) - G;
    if (fold) {
      // cotangent of ghost position p: ctr_p + G_{p-1} - G_p, with G_{-3} =
      // gD[0] of centre -1 and G_{n+1} = gD[3] of centre n the outermost edges
      const double sg = (v == R::MOM + DIR) ? -1.0 : 1.0;
      const double G1 = lane_shift<kFromPrev>(G), G2 = lane_shift<kFromPrev>(G1), G3 = lane_shift<kFromPrev>(G2);
      const double a1 = lane_shift<kFromPrev>(gD[0]), a2 = lane_shift<kFromPrev>(a1), a3 = lane_shift<kFromPrev>(a2);
      const double c1 = lane_shift<kFromPrev>(ctr);
      const double H1 = lane_shift<kFromNext>(G), H2 = lane_shift<kFromNext>(H1);
      const double b1 = lane_shift<kFromNext>(gD[3]), b2 = lane_shift<kFromNext>(b1), b3 = lane_shift<kFromNext>(b2);
      const double d1 = lane_shift<kFromNext>(ctr);
      double lo = 0.0, hi = 0.0;
      if (wall_lo) {
        if (pos == 0) lo = sg * ((c1 + G2) - G1);
        if (pos == 1) lo = sg * (a2 - G3);
        if (pos == 2) lo = sg * -a3;
      } else {
        // extrapolation: the three ghosts' sum telescopes
        if (pos == 0) lo = c1 - G1;
      }
      if (wall_hi) {
        if (pos == nd - 1) hi = sg * ((d1 + G) - H1);
        if (pos == nd - 2) hi = sg * (H2 - b2);
        if (pos == nd - 3) hi = sg * b3;
      } else {
        if (pos == nd - 1) hi = d1 + G;
      }
      s += lo + hi;
    }
    if constexpr (NF == 2) {
      if (v == R::ALPHA) s += ra[0] * div;
      if (v == R::ALPHA + 1) s += ra[1] * div;
    }
    wb[v] = s;
  }
  if constexpr (NF == 2 && (RS & RS_KAPILA) != 0) {
    // Kapila's K of the cell scales the divergence on both alpha rows, (alpha_1
    // + K) and (alpha_2 - K): Kbar = div (rbar_alpha1 - rbar_alpha2)
    double dp, da1, da2;
    kapila_K_grad(pm, Wat(R::E, 2), Wat(R::ALPHA, 2), Wat(R::ALPHA + 1, 2), dp, da1, da2);
    const double Kb = div * (ra[0] - ra[1]);
    wb[R::E] += Kb * dp;
    wb[R::ALPHA] += Kb * da1;
    wb[R::ALPHA + 1] += Kb * da2;
  }

  // ---- the cell's sum joins the other axes'; the last pass ends in qbar --------------
  auto finish = [&](long long cell, const double* ws, const double* Wc) {
    double t[NEQ];
#pragma unroll
    for (int v = 0; v < NEQ; ++v) t[v] = first ? ws[v] : wsum[v * nc + cell] + ws[v];
    if (!last) {
#pragma unroll
      for (int v = 0; v < NEQ; ++v) wsum[v * nc + cell] = t[v];
      return;
    }
    double Ub[NEQ];
    cons_to_prim_vjp_at_prim<NF, D>(pm, Wc, t, Ub);
    // qbar, or (epi.stage > 0) the reverse stage combination of v = Ub
#pragma unroll
    for (int v = 0; v < NEQ; ++v) {
      const long long e = v * nc + cell;
      if (epi.stage == 3) {
        const double x = epi.x[e];
        epi.out[e] = (2.0 / 3.0) * (x + epi.dt * Ub[v]);
        epi.qnb[e] = (1.0 / 3.0) * x;
      } else if (epi.stage == 2) {
        const double x = epi.x[e];
        epi.out[e] = 0.25 * (x + epi.dt * Ub[v]);
        epi.qnb[e] = epi.qnb[e] + 0.75 * x;
      } else if (epi.stage == 1) {
        epi.qnb[e] = epi.qnb[e] + (epi.x[e] + epi.dt * Ub[v]);
      } else {
        qbar[e] = accumulate ? qbar[e] + Ub[v] : Ub[v];
      }
    }
  };
  if constexpr (DIR == 0) {
    if (!out_ok) return;
    double Wc[NEQ];
#pragma unroll
    for (int v = 0; v < NEQ; ++v) Wc[v] = Wat(v, 2);
    finish(vjp_offset<DIR>(pm, line, pos, 0), wb, Wc);
  } else {
    // through LDS, so that neighbouring threads write neighbouring x
#pragma unroll
    for (int v = 0; v < NEQ; ++v) sr[(v * TB + b) * LS + lane] = wb[v];
    __syncthreads();
    const int bb = tid % TB, s = tid / TB;
    long long line2;
    int pos2;
    const bool on2 = place(s, line2, pos2);
    if (x0 + bb >= pm.n[0] || !on2 || s < 3 || s > 60 || pos2 < 0 || pos2 >= nd) return;
    double ws[NEQ], Wc[NEQ];
#pragma unroll
    for (int v = 0; v < NEQ; ++v) {
      ws[v] = sr[(v * TB + bb) * LS + s];
      Wc[v] = sw[(v * TB + bb) * LS + s + 2];
    }
    finish(vjp_offset<DIR>(pm, line2, pos2, x0 + bb), ws, Wc);
  }
}

template <int NF, int D, int DIR, int WV, int RS>
static hipError_t launch_vjp_axis(const Params& pm, const double* q, const double* rbar, double* wsum, bool first,
                                  bool last, double* qbar, bool accumulate, const StageEpi& epi, hipStream_t s) {
  using TL = VjpTile;
  const VjpGeom g = vjp_geom<DIR>(pm);
  if (g.blocks == 0) return hipErrorInvalidConfiguration;
  const unsigned span = 8 * TL::GROUP;
  hipLaunchKernelGGL((vjp_axis_kernel<NF, D, DIR, WV, RS>), dim3((g.blocks + span - 1) / span * span), dim3(TL::NT), 0, s,
                     pm, g, q, rbar, wsum, first ? 1 : 0, last ? 1 : 0, qbar, accumulate ? 1 : 0, epi);
  return hipGetLastError();
}

template <int NF, int D, int WV, int RS>
static hipError_t launch_rhs_vjp_t(const Params& pm, const double* q, const double* rbar, double* qbar, double* wsum,
                                   bool accumulate, hipStream_t s, PassTimer* tm, const StageEpi& epi) {
  hipError_t e = hipSuccess;
  if (tm) tm->begin(KIND_VJP, s);
  // from the highest axis down, x last
  if constexpr (D > 2) e = launch_vjp_axis<NF, D, 2, WV, RS>(pm, q, rbar, wsum, true, false, qbar, accumulate, epi, s);
  if constexpr (D > 1) {
    if (e == hipSuccess) e = launch_vjp_axis<NF, D, 1, WV, RS>(pm, q, rbar, wsum, D == 2, false, qbar, accumulate, epi, s);
  }
  if (e == hipSuccess) e = launch_vjp_axis<NF, D, 0, WV, RS>(pm, q, rbar, wsum, D == 1, true, qbar, accumulate, epi, s);
  if (tm) tm->end(KIND_VJP, s);
  return e;
}

// The face options are compile-time choices, as in the forward passes.
template <int NF, int D, int WV>
static hipError_t vjp_by_riemann(const Params& pm, const double* q, const double* rbar, double* qbar, double* wsum,
                                 bool accumulate, hipStream_t s, PassTimer* tm, const StageEpi& epi) {
#define MFC_RS(B) \
  case B: return launch_rhs_vjp_t<NF, D, WV, B>(pm, q, rbar, qbar, wsum, accumulate, s, tm, epi);
  switch (option_bits(pm)) {
    MFC_RS(0)
    MFC_RS(RS_HLL)
    MFC_RS(RS_THORNBER)
    MFC_RS(RS_HLL | RS_THORNBER)
    MFC_RS(RS_APC)
    default: break;
  }
  if constexpr (NF == 2) {
    switch (option_bits(pm)) {
      MFC_RS(RS_KAPILA)
      MFC_RS(RS_KAPILA | RS_HLL)
      MFC_RS(RS_KAPILA | RS_THORNBER)
      MFC_RS(RS_KAPILA | RS_HLL | RS_THORNBER)
      MFC_RS(RS_KAPILA | RS_APC)
      default: break;
    }
  }
#undef MFC_RS
  return hipErrorInvalidValue;
}

// Every grid of one reconstruction variant.
template <int WV>
hipError_t launch_rhs_vjp_wv(int nf, int ndim, const Params& pm, const double* q, const double* rbar, double* qbar,
                             double* wsum, bool accumulate, hipStream_t s, PassTimer* tm, const StageEpi& epi) {
#define MFC_CASE(NF, D) \
  if (nf == NF && ndim == D) return vjp_by_riemann<NF, D, WV>(pm, q, rbar, qbar, wsum, accumulate, s, tm, epi);
  MFC_CASE(1, 1)
  MFC_CASE(1, 2)
  MFC_CASE(1, 3)
  MFC_CASE(2, 1)
  MFC_CASE(2, 2)
  MFC_CASE(2, 3)
#undef MFC_CASE
  return hipErrorInvalidValue;
}

#define MFC_VJP_DECL(KW, WV)                                                                                   \
  KW template hipError_t launch_rhs_vjp_wv<WV>(int, int, const Params&, const double*, const double*, double*, \
                                               double*, bool, hipStream_t, PassTimer*, const StageEpi&);
#define MFC_INSTANTIATE_VJP(WV) MFC_VJP_DECL(, WV)
#define MFC_EXTERN_VJP(WV) MFC_VJP_DECL(extern, WV)

}  // namespace mfc
