// march_impl.h -- the x and y axes of large 3D grids in one pass, the last of an
// RHS evaluation.
//
// Every wave walks along y.  Its 64 lanes are consecutive cells across y: the
// rows of all x lines of one y, each with its three ghost cells on both sides,
// one z after the other, so that no lane is lost to the grid's size.  Step j
// loads row j, completes the x axis of row j - 3 while the loads are in flight,
// converts row j, reconstructs the y centre j - 2, solves the face below it
// and finishes the cell j - 3 behind that face.  Lanes 3..60 are outputs; the
// others repeat cells of the neighbouring waves as x halo.
//
// What it replaces: a y pass and an x pass that each read q and converted it,
// and handed the RHS accumulator from one to the other through memory.  At
// 256^3 in FP64 (two fluids) the two passes moved 428 B per cell and took 668 +
// 775 us, at the rate of a large copy; this one moves 268 B and takes 1060 us.
// The FP32 form takes 915 us instead of 409 + 529: 1849 instructions a cell, for
// which its two waves per SIMD issue in 60 % of their cycles (FP64: 1463 and 50 %,
// 28 % waiting for memory).  It rounds as the separate passes do, bit for bit; in
// FP64 the accumulator joins the x axis first.
//
// Why this shape: a tile in LDS with y and x halos around it fits twice into a
// CU, and its load phase then finds too little other work (1.88 ms).  Marching
// needs no barrier and no halo along y; its price is state per lane: the y
// stencil (five rows), the last biased values and the last fluxes.  In FP64
// that spills at two waves per SIMD (2.36 ms), so the two oldest rows, the
// fluxes and the x contribution wait in LDS (17 KB a wave, eight waves per CU)
// and the registers hold three rows.  With it nothing spills.
#pragma once

#include "device.h"
#include "internal.h"
#include "lanes.h"

namespace mfc {

// Geometry of a launch: `chunk` output rows per wave, `cols` waves across,
// `waves` = cols times chunks.
struct MarchGeom {
  int chunk;
  int cols;
  unsigned waves;
};
// Blocks are dispatched to the eight XCDs in turn: waves (numbered across,
// then chunk by chunk) go to them in groups of kGroup neighbours, which share
// cache lines and x halo.
constexpr unsigned kGroup = 8;
constexpr int kMarchOut = 58;  // outputs of a wave's 64 lanes

// Element at a wave-uniform pointer plus a lane's byte offset: the pointer is
// made an opaque scalar, so that the access takes its scalar-base form and the
// row offsets are scalar additions (the compiler otherwise adds them to a
// 64-bit vector address for every row).
template <typename Real>
__device__ __forceinline__ Real load_at(const Real* p, unsigned off) {
  using G = const __attribute__((address_space(1))) char*;
  G g = (G)p;
  asm("" : "+s"(g));
  return *(const __attribute__((address_space(1))) Real*)(g + off);
}
template <typename Real>
__device__ __forceinline__ void store_at(Real* p, unsigned off, Real v) {
  using G = __attribute__((address_space(1))) char*;
  G g = (G)p;
  asm("" : "+s"(g));
  *(__attribute__((address_space(1))) Real*)(g + off) = v;
}
// The same offset as a value that is born here: the access pattern above is
// matched within a basic block, where the 32-bit value has to be seen.
__device__ __forceinline__ unsigned here(unsigned off) {
  asm("" : "+v"(off));
  return off;
}

template <int NF, typename Real, int MODE, int WV, int RS>
__global__ __launch_bounds__(64, 2) void march_kernel(Params pm, const Real* __restrict__ qk, Real* __restrict__ acc,
                                                      const Real* __restrict__ qn, Real* __restrict__ qout,
                                                      StageArgs st, int* __restrict__ flag, MarchGeom mg) {
  constexpr int D = 3;
  using R = Rows<NF, D>;
  constexpr int NEQ = R::NEQ;
  constexpr bool kF64 = sizeof(Real) == 8;
  constexpr bool kStep = (MODE & MODE_STEP) != 0;
  static_assert((MODE & MODE_ACC) != 0, "the z pass comes first");
  static_assert(WV != kWvNonUniform, "uniform grids only");
  // two rows of primitives (j - 4 and j - 3), by the parity of the step that
  // wrote them, with two pad cells on both sides for the x stencil
  constexpr int LW = 68;
  __shared__ Real sx[2][NEQ * LW];
  // double: the fluxes of the face below and the x contribution wait here
  // while the other axis has the registers
  __shared__ Real sF[kF64 ? (NEQ + 1) * 64 : 1], sD[kF64 ? NEQ * 64 : 1];
  const int lane = threadIdx.x;
  const int own = lane + 2;
  const unsigned j8 = blockIdx.x >> 3;
  const unsigned wave = ((j8 / kGroup) * 8u + (blockIdx.x & 7u)) * kGroup + j8 % kGroup;
  if (wave >= mg.waves) return;
  const unsigned chunk_id = wave / (unsigned)mg.cols;
  const unsigned col = wave - chunk_id * (unsigned)mg.cols;

  const int nx = pm.n[0], ny = pm.n[1];
  const long long nc = pm.ncell;
  const long long plane = (long long)nx * ny;
  const int m0 = (int)chunk_id * mg.chunk;
  const int m1 = (m0 + mg.chunk < ny) ? m0 + mg.chunk : ny;

  // this lane's cell across y: the wave's first z plane as scalar base, a
  // 32-bit byte offset from it (march_pays checks that it suffices)
  const unsigned P = (unsigned)nx + 6u;
  const long long g0 = (long long)col * kMarchOut;
  const long long z0 = g0 / P;
  const unsigned r0 = (unsigned)(g0 - z0 * P) + (unsigned)lane;
  unsigned dz = r0 / P;
  const int xpos = (int)(r0 - dz * P) - 3;
  const bool valid = g0 + lane < (long long)P * pm.n[2];
  if (!valid) dz = (unsigned)(pm.n[2] - 1 - z0);
  bool flipx;
  const int gx = ghost_index(xpos, nx, pm.bc_lo[0], pm.bc_hi[0], flipx);
  const double sgnx = flipx ? -1.0 : 1.0;
  const long long base = z0 * plane;
  const unsigned off = (unsigned)((dz * (unsigned long long)plane + (unsigned)gx) * sizeof(Real));
  const bool out_lane = valid && lane >= 3 && lane <= 60 && xpos >= 0 && xpos < nx;
  const bool xface = valid && lane >= 3 && lane <= 61 && xpos >= 0 && xpos <= nx;

  // SSP-RK3, Shu-Osher form (Sec. 3.4): next state = ka q^n + kb (q_k + dt r),
  // rounded as rk3_stage rounds it (q^n counts as 0 in stage 1)
  double dt = 0.0, ka = 0.0, kb = 1.0;
  if constexpr (kStep) {
    dt = st.dt_ptr ? *st.dt_ptr : st.dt;
    if (st.stage == 2) {
      ka = 0.75;
      kb = 0.25;
    } else if (st.stage == 3) {
      ka = 1.0 / 3.0;
      kb = 2.0 / 3.0;
    }
  }
  const WenoK<Real> K = weno_consts(Real(pm.eps));
  const Real ihx = Real(pm.inv_dx[0]);

  // The y stencil of step j: rows j - 4 and j - 3 in LDS, j - 2 .. j in w;
  // wo is row j - 3 on its way into LDS.
  Real w[3][NEQ], wo[NEQ], raw[NEQ], WLp[NEQ], Fp[NEQ];
  Real ufp = Real(0);
  bool bad_any = false;

  auto load_row = [&](int j, Real* r) -> bool {
    bool flip;
    const long long rb = base + (long long)ghost_index(j, ny, pm.bc_lo[1], pm.bc_hi[1], flip) * nx;
    const unsigned o = here(off);
#pragma unroll
    for (int v = 0; v < NEQ; ++v) r[v] = load_at(qk + v * nc + rb, o);
    return flip;
  };
  auto arrive = [&](bool flip, const Real* r, Real* dst) {
    double U[NEQ], W[NEQ];
#pragma unroll
    for (int v = 0; v < NEQ; ++v) U[v] = double(r[v]);
    U[R::MOM] *= sgnx;
    U[R::MOM + 1] *= flip ? -1.0 : 1.0;
    cons_to_prim<NF, D, Real>(pm, U, W);
#pragma unroll
    for (int v = 0; v < NEQ; ++v) dst[v] = Real(W[v]);
  };
  // the first four rows, all loads in flight together
  {
    Real r4[4][NEQ];
    bool f4[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) f4[k] = load_row(m0 - 3 + k, r4[k]);
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      Real* dst = k == 1 ? wo : w[k == 0 ? 0 : k - 2];
      arrive(f4[k], r4[k], dst);
      if (k == 0) {
#pragma unroll
        for (int v = 0; v < NEQ; ++v) sx[m0 & 1][v * LW + own] = dst[v];
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  }
#pragma unroll
  for (int v = 0; v < NEQ; ++v) WLp[v] = Fp[v] = Real(0);

  // step j: row j arrives, y centre c = j - 2, face c - 1/2 (a face of this
  // chunk from j = m0 + 2 on), output cell j - 3 (from j = m0 + 3 on)
#pragma unroll 1
  for (int j = m0 + 1; j <= m1 + 2; ++j) {
    const bool full = j >= m0 + 3;
    const long long ob = base + (long long)(j - 3) * nx;
    Real* const so = sx[j & 1];         // row j - 3
    const Real* const s4 = sx[~j & 1];  // row j - 4
    const bool flipy = load_row(j, raw);
#pragma unroll
    for (int v = 0; v < NEQ; ++v) so[v * LW + own] = wo[v];
    Real a0[NEQ];
    if (full) {
      const unsigned o = here(off);
#pragma unroll
      for (int v = 0; v < NEQ; ++v) a0[v] = load_at((const Real*)acc + v * nc + ob, o);
    }

    // volume fractions of the output cell for the alpha source; with RS_KAPILA
    // they carry Kapila's K of the cell, (alpha_1 + K, alpha_2 - K)
    Real al[2] = {Real(0), Real(0)};
    if constexpr (NF == 2) {
      al[0] = wo[R::ALPHA];
      al[1] = wo[R::ALPHA + 1];
      if constexpr ((RS & RS_KAPILA) != 0) {
        const double Kc = kapila_K(pm, double(wo[R::E]), double(al[0]), double(al[1]));
        al[0] = Real(double(al[0]) + Kc);
        al[1] = Real(double(al[1]) - Kc);
      }
    }

    // ---- x axis of row j - 3 ----------------------------------------------------
    // F_{-1/2} - F_{+1/2} (conservative rows), the whole contribution (alpha rows)
    Real dx[NEQ];
    if (full) {
      __syncthreads();  // one wave: orders its LDS accesses
      Real WL[NEQ], WR[NEQ];
#pragma unroll
      for (int v = 0; v < NEQ; ++v) {
        const Real* f = so + v * LW + lane;
        Real wl;
        weno5<WV>(f[0], f[1], f[2], f[3], f[4], K, wl, WR[v]);
        WL[v] = lane_shift<kFromPrev>(wl);
        // one row at a time: interleaved rows cost more registers than there are
        if constexpr (kF64) __builtin_amdgcn_sched_barrier(0);
      }
      Real F[NEQ], uf;
      if constexpr ((RS & RS_THORNBER) != 0) thornber<NF, D, 0, Real>(pm, WL, WR);
      const bool bad = riemann<RS, NF, D, 0, Real>(pm, WL, WR, F, uf);
      bad_any |= bad && xface;
      const Real divx = ihx * (lane_shift<kFromNext>(uf) - uf);
#pragma unroll
      for (int v = 0; v < NEQ; ++v) {
        const Real fhi = lane_shift<kFromNext>(F[v]);
        dx[v] = F[v] - fhi;
        if constexpr (NF == 2) {
          if (v == R::ALPHA) dx[v] = ihx * (F[v] - fhi) + al[0] * divx;
          if (v == R::ALPHA + 1) dx[v] = ihx * (F[v] - fhi) + al[1] * divx;
        }
        // double: joined with the accumulator at once; float adds it last, the
        // order of its separate passes
        if constexpr (kF64) {
          if (NF != 2 || v < R::ALPHA) dx[v] = ihx * dx[v];
          sD[v * 64 + lane] = a0[v] + dx[v];
        }
      }
    }

    // ---- row j arrives ------------------------------------------------------------
    arrive(flipy, raw, w[2]);

    // ---- y axis: centre j - 2 and the face below it -------------------------------
    Real WLn[NEQ], WR[NEQ];
#pragma unroll
    for (int v = 0; v < NEQ; ++v) {
      const Real f0 = s4[v * LW + own], f1 = so[v * LW + own];
      weno5<WV>(f0, f1, w[0][v], w[1][v], w[2][v], K, WLn[v], WR[v]);
      if constexpr (kF64) {
        // formed here: moved to its use behind the face solver it would keep its
        // six inputs alive instead (30 registers more, and spills)
        asm volatile("" : "+v"(WLn[v]));
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    Real F[NEQ], uf;
    if constexpr ((RS & RS_THORNBER) != 0) thornber<NF, D, 1, Real>(pm, WLp, WR);
    const bool bad = riemann<RS, NF, D, 1, Real>(pm, WLp, WR, F, uf);
    bad_any |= bad && out_lane && j >= m0 + 2;
    if (full) {
      // ---- output cell j - 3 between the faces j - 7/2 and j - 5/2 ----------------
      Real qv[NEQ], uk[NEQ];
      if constexpr (kStep) {
#pragma unroll
        for (int v = 0; v < NEQ; ++v) qv[v] = Real(0);
        if (st.stage != 1) {
          const unsigned o = here(off);
#pragma unroll
          for (int v = 0; v < NEQ; ++v) qv[v] = load_at(qn + v * nc + ob, o);
        }
        if constexpr (!kF64) {
          const unsigned o = here(off);
#pragma unroll
          for (int v = 0; v < NEQ; ++v) uk[v] = load_at(qk + v * nc + ob, o);
        }
      }
      const Real ih = Real(pm.inv_dx[1]);
      if constexpr (kF64) ufp = sF[NEQ * 64 + lane];
      const Real div = ih * (uf - ufp);
      double Uc[NEQ];
      if constexpr (kF64 && kStep) {
        // the conservative values of the cell from its primitives
        double Wc[NEQ];
#pragma unroll
        for (int v = 0; v < NEQ; ++v) Wc[v] = double(so[v * LW + own]);
        prim_to_cons<NF, D, Real>(pm, Wc, Uc);
      }
      const unsigned o = here(off);
#pragma unroll
      for (int v = 0; v < NEQ; ++v) {
        if constexpr (kF64) {
          Fp[v] = sF[v * 64 + lane];
          dx[v] = sD[v * 64 + lane];
        }
        Real Dv = ih * (Fp[v] - F[v]);
        if constexpr (NF == 2) {
          if (v == R::ALPHA) Dv = Dv + al[0] * div;
          if (v == R::ALPHA + 1) Dv = Dv + al[1] * div;
        }
        Real r = Dv;
        if constexpr (kF64) {
          r = r + dx[v];
        } else {
          r = a0[v] + Dv;
          // the fused operation of the separate x pass, whatever the compiler
          // would contract here
          r = (NF == 2 && v >= R::ALPHA) ? r + dx[v] : fmaf(ihx, dx[v], r);
        }
        if constexpr (kStep) {
          // combined in double, the fused products written out
          const double ukv = kF64 ? Uc[v] : double(uk[v]);
          const double out = fma(ka, double(qv[v]), kb * fma(dt, double(r), ukv));
          if (out_lane) store_at(qout + v * nc + ob, o, Real(out));
        } else {
          if (out_lane) store_at(acc + v * nc + ob, o, r);
        }
      }
    }
    if constexpr (kF64) {
#pragma unroll
      for (int v = 0; v < NEQ; ++v) sF[v * 64 + lane] = F[v];
      sF[NEQ * 64 + lane] = uf;
    } else {
#pragma unroll
      for (int v = 0; v < NEQ; ++v) Fp[v] = F[v];
      ufp = uf;
    }
#pragma unroll
    for (int v = 0; v < NEQ; ++v) {
      WLp[v] = WLn[v];
      wo[v] = w[0][v];
      w[0][v] = w[1][v];
      w[1][v] = w[2][v];
    }
  }
  if (bad_any) atomicOr(flag, 1);
}

// ---------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------
// Waves that fill the chip: two per SIMD, what the registers leave room for.
constexpr long long kMarchSlots = 2 * 4 * 256;

inline long long march_cols(const int* n) {
  return ((long long)(n[0] + 6) * n[2] - 6 + kMarchOut - 1) / kMarchOut;
}

// Output rows per wave.  A chunk costs about 1.5 rows more than it gives (six
// rows loaded, a centre and a face solved twice), so long chunks are better
// while enough waves remain; the last waves to finish idle half a chunk's time
// of the others.
inline MarchGeom march_geom(const int* n) {
  const long long cols = march_cols(n);
  double best = 1e300;
  int chunk = 1;
  for (int c = 1; c <= 64 && c <= n[1]; ++c) {
    const double rounds = double(cols * ((n[1] + c - 1) / c)) / kMarchSlots;
    const double cost = ((rounds < 1.0 ? 1.0 : rounds) + 0.5) * (c + 1.5);
    if (cost < best) {
      best = cost;
      chunk = c;
    }
  }
  return MarchGeom{chunk, (int)cols, (unsigned)(cols * ((n[1] + chunk - 1) / chunk))};
}

// Reconstructions that the marching pass is built for: WENO5-JS and WENO5-Z.
// The double TENO5, WENO5-M and tabulated ones spill 200 to 650 bytes a lane
// there; they keep the separate passes.
template <int WV>
constexpr bool kMarchVariant = WV <= 1;

// Whether the marching pass is taken.  It needs waves enough to fill the chip
// with long walks; below that its 1.5 extra rows a chunk and its two waves per
// SIMD cost more than the traffic it saves.  Measured, separate passes against
// marching, us per two-fluid step: FP64 64^3 129 / 141, 96^3 313 / 308, 150 x 98
// x 61 452 / 362, 14 x 250 x 250 498 / 422, 128^3 788 / 709, 256^3 5887 / 4801:
// from 2^19 cells on.  FP32, which the instructions bound: 128^3 561 / 569,
// 160^3 1007 / 1079, 256^3 4058 / 3905, 512^3 32399 / 29745: from 2^23 on.  Since
// the x pass runs from line to line: FP64 200^3 2913 / 2400, 256^3 5872 / 4772,
// FP32 256^3 4065 / 3926.
template <typename Real>
inline bool march_pays(const Params& pm) {
  const int* n = pm.n;
  // 32-bit lane offsets: a wave spans at most 64 / (nx + 6) + 2 z planes
  const double span = double(n[0]) * n[1] * (64 / (n[0] + 6) + 2) * sizeof(Real);
  return pm.ncell >= (sizeof(Real) == 8 ? 1ll << 19 : 1ll << 23) && span < 4294967296.0 &&
         march_geom(n).waves < (1u << 25);  // work-items of a launch stay below 2^32
}

template <int NF, typename Real, int MODE, int WV, int RS>
static hipError_t launch_march(const Params& pm, const Real* qk, Real* acc, const Real* qn, Real* qout, StageArgs st,
                               int* flag, hipStream_t s, PassTimer* tm) {
  const MarchGeom mg = march_geom(pm.n);
  const unsigned blocks = (mg.waves + 8 * kGroup - 1) / (8 * kGroup) * (8 * kGroup);
  if (tm) tm->begin(KIND_PASS_X, s);
  hipLaunchKernelGGL((march_kernel<NF, Real, MODE, WV, RS>), dim3(blocks), dim3(64), 0, s, pm, qk, acc, qn, qout, st,
                     flag, mg);
  if (tm) tm->end(KIND_PASS_X, s);
  return hipGetLastError();
}

}  // namespace mfc
