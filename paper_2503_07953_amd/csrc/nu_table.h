// nu_table.h -- reconstruction tables of a non-uniform grid, built on the host.
#pragma once

#include <cmath>
#include <utility>
#include <vector>

#include "device.h"

namespace mfc {

// ---------------------------------------------------------------------------
// Non-uniform grids (Sec. 4.2.2): reconstruction tables built on the host.
// For the centre cell at position c of an axis, with unit coordinate
// xi = (x - x_c)/h_c, candidate r (cells c - 2 + r .. c + r) is the quadratic
// m0 + m1 xi + m2 xi^2 with the data as its cell averages: m = A^-1 f, A the
// 3 x 3 matrix of cell averages of 1, xi, xi^2 over the stencil's cells.  The
// ideal weights at a face are the least-squares (here exact) solution of
// sum_r d_r v_r = v5, v_r the candidate's value functional at the face and v5
// that of the quartic with the five cells' averages.  Ghost cells take the
// width of the cell whose state they hold (ghost_index).
// ---------------------------------------------------------------------------

// Solve the n x n system M X = B for X (k right-hand sides), Gaussian
// elimination with partial pivoting; M and B are overwritten.  False if singular.
inline bool solve_dense(int n, int k, double* M, double* B) {
  for (int col = 0; col < n; ++col) {
    int piv = col;
    for (int r = col + 1; r < n; ++r)
      if (fabs(M[r * n + col]) > fabs(M[piv * n + col])) piv = r;
    if (!(fabs(M[piv * n + col]) > 0.0)) return false;
    if (piv != col) {
      for (int j = 0; j < n; ++j) std::swap(M[col * n + j], M[piv * n + j]);
      for (int j = 0; j < k; ++j) std::swap(B[col * k + j], B[piv * k + j]);
    }
    for (int r = col + 1; r < n; ++r) {
      const double f = M[r * n + col] / M[col * n + col];
      for (int j = col; j < n; ++j) M[r * n + j] -= f * M[col * n + j];
      for (int j = 0; j < k; ++j) B[r * k + j] -= f * B[col * k + j];
    }
  }
  for (int col = n - 1; col >= 0; --col) {
    for (int j = 0; j < k; ++j) {
      double v = B[col * k + j];
      for (int c2 = col + 1; c2 < n; ++c2) v -= M[col * n + c2] * B[c2 * k + j];
      B[col * k + j] = v / M[col * n + col];
    }
  }
  return true;
}

// Inverse of the moment matrix of `deg + 1` cells with unit-coordinate faces
// e[0..deg+1]: row k of the result maps the cell averages to m_k.
inline bool moment_inverse(int deg, const double* e, double* inv) {
  const int n = deg + 1;
  double M[25], B[25];
  for (int j = 0; j < n; ++j)
    for (int k = 0; k < n; ++k) {
      const double a = e[j], b = e[j + 1];
      M[j * n + k] = (std::pow(b, k + 1) - std::pow(a, k + 1)) / ((k + 1) * (b - a));
      B[j * n + k] = (j == k) ? 1.0 : 0.0;
    }
  // M X = I gives X = M^-1 with X[k][j] the weight of average j in m_k
  if (!solve_dense(n, n, M, B)) return false;
  for (int i = 0; i < n * n; ++i) inv[i] = B[i];
  return true;
}

// Rows NU_B .. of one table entry from its candidates and ideal weights.
inline void fold_entry(double* t, long long st) {
  auto at = [&](int row) -> double& { return t[row * st]; };
  for (int r = 0; r < 3; ++r) {
    // o: the difference inside the square alone (D_0, D_1, D_3)
    const int o = r == 2 ? 1 : 0;
    double m1[2], m2[2];
    for (int j = 0; j < 2; ++j) {
      const double m0 = at(NU_MU0 + 2 * r + j);
      m1[j] = at(NU_M1 + 2 * r + j);
      m2[j] = at(NU_M2 + 2 * r + j);
      at(NU_VR + 2 * r + j) = at(NU_DR + r) * (m0 + 0.25 * m2[j] + 0.5 * m1[j]);
      at(NU_VL + 2 * r + j) = at(NU_DL + r) * (m0 + 0.25 * m2[j] - 0.5 * m1[j]);
    }
    const double k = 13.0 / 3.0, p = std::hypot(m1[o], std::sqrt(k) * m2[o]);
    const double c1 = m1[o] / p, c2 = m2[o] / p, det = c1 * m2[1 - o] - c2 * m1[1 - o];
    at(NU_B + 3 * r) = p;
    at(NU_B + 3 * r + 1) = c1 * m1[1 - o] + k * (c2 * m2[1 - o]);
    at(NU_B + 3 * r + 2) = k * (det * det);
  }
}

// Table of one axis: kNuCoefs rows of n + 6 entries (positions -3 .. n + 2).
inline bool build_axis_table(const Params& pm, int d, const std::vector<double>& faces, double dx,
                      std::vector<double>& tab) {
  const int n = pm.n[d];
  const long long st = n + 6;
  tab.assign((size_t)kNuCoefs * st, 0.0);
  auto width = [&](int pos) {
    if (faces.empty()) return dx;
    bool flip;
    const int i = ghost_index(pos, n, pm.bc_lo[d], pm.bc_hi[d], flip);
    return faces[i + 1] - faces[i];
  };
  for (int pos = -3; pos <= n + 2; ++pos) tab[NU_INVW * st + pos + 3] = 1.0 / width(pos);
  for (int pos = -1; pos <= n; ++pos) {
    const double hc = width(pos);
    double e[6];
    e[2] = -0.5;
    e[3] = 0.5;
    e[1] = e[2] - width(pos - 1) / hc;
    e[0] = e[1] - width(pos - 2) / hc;
    e[4] = e[3] + width(pos + 1) / hc;
    e[5] = e[4] + width(pos + 2) / hc;
    double inv3[3][9];
    for (int r = 0; r < 3; ++r) {
      if (!moment_inverse(2, &e[r], inv3[r])) return false;
      // m_k = sum_j inv[k][j] f_{r+j}; m0 - f_2 subtracts the centre (j = 2 - r)
      for (int k = 0; k < 3; ++k) {
        double w[3] = {inv3[r][k * 3 + 0], inv3[r][k * 3 + 1], inv3[r][k * 3 + 2]};
        if (k == 0) w[2 - r] -= 1.0;
        // zero-sum w: w . f = -w_0 (f_1 - f_0) + w_2 (f_2 - f_1) over the stencil
        const int row = (k == 0 ? NU_MU0 : k == 1 ? NU_M1 : NU_M2) + 2 * r;
        tab[row * st + pos + 3] = -w[0];
        tab[(row + 1) * st + pos + 3] = w[2];
      }
    }
    double inv5[25];
    if (!moment_inverse(4, e, inv5)) return false;
    for (int side = 0; side < 2; ++side) {
      const double xi = side == 0 ? 0.5 : -0.5;
      double v5[5] = {0, 0, 0, 0, 0}, V[3][5] = {};
      for (int j = 0; j < 5; ++j)
        for (int k = 0; k < 5; ++k) v5[j] += std::pow(xi, k) * inv5[k * 5 + j];
      for (int r = 0; r < 3; ++r)
        for (int j = 0; j < 3; ++j)
          for (int k = 0; k < 3; ++k) V[r][r + j] += std::pow(xi, k) * inv3[r][k * 3 + j];
      double N[9], rhs[3];
      for (int a = 0; a < 3; ++a) {
        rhs[a] = 0.0;
        for (int j = 0; j < 5; ++j) rhs[a] += V[a][j] * v5[j];
        for (int b = 0; b < 3; ++b) {
          N[a * 3 + b] = 0.0;
          for (int j = 0; j < 5; ++j) N[a * 3 + b] += V[a][j] * V[b][j];
        }
      }
      if (!solve_dense(3, 1, N, rhs)) return false;
      const int row = side == 0 ? NU_DR : NU_DL;
      for (int r = 0; r < 3; ++r) tab[(row + r) * st + pos + 3] = rhs[r];
    }
    fold_entry(&tab[pos + 3], st);
  }
  return true;
}

}  // namespace mfc
