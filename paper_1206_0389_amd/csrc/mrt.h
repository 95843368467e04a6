// D3Q19 MRT collision with a Smagorinsky eddy viscosity, for gfx950.
//
// Eq. (12) read as a relaxation, f* = f - M^-1 S (M f - m_eq), m_eq = M f_eq
// with the incompressible equilibrium of Eq. (2) (deviation form, rho0 = 1).
// The shear rows relax with 1/tau_total from the closed form Eqs. (20)-(21),
// Q = sqrt(2 Pi:Pi), Pi = sum_i e_i e_i (f_i - f_eq_i) (Eq. (19)).
//
// Both moment bases and their inverses are built at compile time for the
// adjoint and the interface rescaling, which unroll the matrix-vector
// products so that zero entries vanish and +-1 entries become additions. The
// collision itself works on raw moments (mrt_collide). Only the shear rate
// is per node.
#pragma once

#include "stencil.h"

namespace lbm {

// One moment row: a radial polynomial r0 + r1 |e|^2 + r2 |e|^4 times a sum
// of monomials coef * ex^a ey^b ez^c.
struct Mono {
  double coef;
  int a, b, c;
};
struct Row {
  double r[3];
  int n;
  Mono t[3];
  int group;  // 0 conserved, 1 shear (1/tau_total), 2+k runtime rate k
};

constexpr double ipow_c(int v, int p) {
  double r = 1.0;
  for (int k = 0; k < p; ++k) r *= v;
  return r;
}

// Moments grouped as in Table 1 (the s1..s7 groups that exist on D3Q19).
constexpr Row kTable1Rows[19] = {
    {{1, 0, 0}, 1, {{1, 0, 0, 0}}, 0},
    {{1, 0, 0}, 1, {{1, 1, 0, 0}}, 0},
    {{1, 0, 0}, 1, {{1, 0, 1, 0}}, 0},
    {{1, 0, 0}, 1, {{1, 0, 0, 1}}, 0},
    {{1, 0, 0}, 1, {{1, 1, 1, 0}}, 1},                         // mu_12
    {{1, 0, 0}, 1, {{1, 1, 0, 1}}, 1},                         // mu_13
    {{1, 0, 0}, 1, {{1, 0, 1, 1}}, 1},                         // mu_23
    {{1, 0, 0}, 2, {{1, 2, 0, 0}, {-1, 0, 2, 0}}, 1},          // mu_11 - mu_22
    {{1, 0, 0}, 2, {{1, 2, 0, 0}, {-1, 0, 0, 2}}, 1},          // mu_11 - mu_33
    {{0, 1, 0}, 1, {{1, 0, 0, 0}}, 2},                         // s2: trace
    {{1, 0, 0}, 2, {{1, 1, 2, 0}, {1, 1, 0, 2}}, 3},           // s3
    {{1, 0, 0}, 2, {{1, 2, 1, 0}, {1, 0, 1, 2}}, 3},
    {{1, 0, 0}, 2, {{1, 2, 0, 1}, {1, 0, 2, 1}}, 3},
    {{1, 0, 0}, 2, {{1, 1, 2, 0}, {-1, 1, 0, 2}}, 4},          // s4
    {{1, 0, 0}, 2, {{1, 2, 1, 0}, {-1, 0, 1, 2}}, 4},
    {{1, 0, 0}, 2, {{1, 2, 0, 1}, {-1, 0, 2, 1}}, 4},
    {{1, 0, 0}, 3, {{1, 2, 2, 0}, {-2, 2, 0, 2}, {1, 0, 2, 2}}, 5},  // s7
    {{1, 0, 0}, 3, {{1, 2, 2, 0}, {1, 2, 0, 2}, {-2, 0, 2, 2}}, 5},
    {{1, 0, 0}, 3, {{1, 2, 2, 0}, {1, 2, 0, 2}, {1, 0, 2, 2}}, 5},
};

// d'Humieres, Ginzburg, Krafczyk, Lallemand & Luo (2002) orthogonal D3Q19
// basis: energy, energy squared, heat flux, viscous stress, 4th-order
// stress and the antisymmetric 3rd-order moments.
constexpr Row kDhumieresRows[19] = {
    {{1, 0, 0}, 1, {{1, 0, 0, 0}}, 0},
    {{-30, 19, 0}, 1, {{1, 0, 0, 0}}, 2},                       // e
    {{12, -26.5, 10.5}, 1, {{1, 0, 0, 0}}, 3},                  // eps
    {{1, 0, 0}, 1, {{1, 1, 0, 0}}, 0},                          // j_x
    {{-9, 5, 0}, 1, {{1, 1, 0, 0}}, 4},                         // q_x
    {{1, 0, 0}, 1, {{1, 0, 1, 0}}, 0},                          // j_y
    {{-9, 5, 0}, 1, {{1, 0, 1, 0}}, 4},                         // q_y
    {{1, 0, 0}, 1, {{1, 0, 0, 1}}, 0},                          // j_z
    {{-9, 5, 0}, 1, {{1, 0, 0, 1}}, 4},                         // q_z
    {{1, 0, 0}, 3, {{2, 2, 0, 0}, {-1, 0, 2, 0}, {-1, 0, 0, 2}}, 1},   // 3 p_xx
    {{-5, 3, 0}, 3, {{2, 2, 0, 0}, {-1, 0, 2, 0}, {-1, 0, 0, 2}}, 5},  // 3 pi_xx
    {{1, 0, 0}, 2, {{1, 0, 2, 0}, {-1, 0, 0, 2}}, 1},           // p_ww
    {{-5, 3, 0}, 2, {{1, 0, 2, 0}, {-1, 0, 0, 2}}, 5},          // pi_ww
    {{1, 0, 0}, 1, {{1, 1, 1, 0}}, 1},                          // p_xy
    {{1, 0, 0}, 1, {{1, 0, 1, 1}}, 1},                          // p_yz
    {{1, 0, 0}, 1, {{1, 1, 0, 1}}, 1},                          // p_xz
    {{1, 0, 0}, 2, {{1, 1, 2, 0}, {-1, 1, 0, 2}}, 6},           // m_x
    {{1, 0, 0}, 2, {{1, 0, 1, 2}, {-1, 2, 1, 0}}, 6},           // m_y
    {{1, 0, 0}, 2, {{1, 2, 0, 1}, {-1, 0, 2, 1}}, 6},           // m_z
};

struct Mat19 {
  double a[19][19];
};

constexpr double eval_row(const Row& r, int i) {
  const double e2 = cx(i) * cx(i) + cy(i) * cy(i) + cz(i) * cz(i);
  double s = 0.0;
  for (int k = 0; k < r.n; ++k)
    s += r.t[k].coef * ipow_c(cx(i), r.t[k].a) * ipow_c(cy(i), r.t[k].b) *
         ipow_c(cz(i), r.t[k].c);
  return (r.r[0] + r.r[1] * e2 + r.r[2] * e2 * e2) * s;
}

constexpr Mat19 build_basis(int basis) {
  Mat19 M{};
  for (int k = 0; k < 19; ++k)
    for (int i = 0; i < 19; ++i)
      M.a[k][i] = eval_row(basis == 0 ? kTable1Rows[k] : kDhumieresRows[k], i);
  return M;
}

constexpr double abs_c(double v) { return v < 0 ? -v : v; }

// Gauss-Jordan inverse with partial pivoting, evaluated by the compiler.
constexpr Mat19 invert19(const Mat19& A) {
  double w[19][38] = {};
  for (int r = 0; r < 19; ++r) {
    for (int c = 0; c < 19; ++c) w[r][c] = A.a[r][c];
    w[r][19 + r] = 1.0;
  }
  for (int c = 0; c < 19; ++c) {
    int p = c;
    for (int r = c + 1; r < 19; ++r)
      if (abs_c(w[r][c]) > abs_c(w[p][c])) p = r;
    if (p != c)
      for (int k = 0; k < 38; ++k) {
        const double t = w[c][k];
        w[c][k] = w[p][k];
        w[p][k] = t;
      }
    const double piv = w[c][c];
    for (int k = 0; k < 38; ++k) w[c][k] /= piv;
    for (int r = 0; r < 19; ++r)
      if (r != c && w[r][c] != 0.0) {
        const double l = w[r][c];
        for (int k = 0; k < 38; ++k) w[r][k] -= l * w[c][k];
      }
  }
  Mat19 R{};
  for (int r = 0; r < 19; ++r)
    for (int c = 0; c < 19; ++c) R.a[r][c] = w[r][19 + c];
  return R;
}

constexpr int row_group(int basis, int k) {
  return basis == 0 ? kTable1Rows[k].group : kDhumieresRows[k].group;
}

template <int BASIS>
struct MrtTables {
  static constexpr Mat19 M = build_basis(BASIS);
  static constexpr Mat19 Minv = invert19(M);
};

// Entries below this magnitude are exact zeros of the rational inverse.
constexpr bool is_nonzero(double v) { return abs_c(v) > 1e-12; }

struct MrtParams {
  double tau0;     // 3 nu + 1/2
  double cs18;     // 18 C_S^2
  double rates[5]; // runtime non-shear rates (groups 2+k)
};

// The collision of one node, on raw moments. Both bases relax linear
// combinations of the same raw non-equilibrium moments of order 2 to 4,
//   n_ab = sum e_a e_b d,  a_ab = sum e_a e_b^2 d,  b_ab = sum e_a^2 e_b^2 d
// (d = f - f_eq; the equilibrium's moments of Eq. (2) are drho/3 + j_a j_b,
// j_a/3 and drho/9 + (j_a^2 + j_b^2)/3 - j_c^2/6), so the relaxation gives
// the change of each raw moment, and D3Q19's inverse is a few sums: the four
// diagonal populations of a plane are the only ones in its b, n_ab and a.
//   Table 1:    n's deviator at 1/tau, trace at s2, a_ab +- a_ac at s3, s4,
//               every b at s7.
//   d'Humieres: eps = 21 (b sum) - 16 (trace) and the deviator of pi, 3 b' -
//               2 n' with b'_yz paired to n'_xx, mix orders 2 and 4.
// Small moments are formed from differences in which what the populations
// have in common (drho / 3, j_a / 3) has dropped out, never by subtracting
// it from sums that carry it: the deviators from differences of two axes,
// the trace from (b sum) - f_0. The shear rate near 2 (tau0 < 1) is used as
// 2 - gap: rounding 1/tau itself shifts the viscosity by up to 6e-8 tau /
// (tau - 1/2), which adds up over the steps. FP32 against 64 bits, velocity,
// 24^3 periodic waves at nu 1e-3, this form / the unrolled 19 x 19 products:
// Table 1 3.3e-8 / 7.5e-8 after 6 steps, 2.7e-7 / 9.2e-7 after 300,
// d'Humieres 4.5e-8 / 6.9e-8 and 3.3e-7 / 1.2e-6.
// 289 VALU instructions per node in the FP32 even step, 558 with the
// products; the steps, bound by memory, take the same time as before the
// differences (131x97x211 jet, ten steps and populations: 687 us).
template <typename real, int BASIS>
__device__ __forceinline__ void mrt_collide(real (&f)[19], const MrtParams& p) {
  // the four diagonals of the xy, xz and yz planes: ++, --, +-, -+
  constexpr int P[3][4] = {
      {index_of(1, 1, 0), index_of(-1, -1, 0), index_of(1, -1, 0), index_of(-1, 1, 0)},
      {index_of(1, 0, 1), index_of(-1, 0, -1), index_of(1, 0, -1), index_of(-1, 0, 1)},
      {index_of(0, 1, 1), index_of(0, -1, -1), index_of(0, 1, -1), index_of(0, -1, 1)}};
  // per plane: e_a^2 e_b^2, e_a e_b, e_a e_b^2 and e_a^2 e_b moments
  real B[3], X[3], A1[3], A2[3];
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    const real s = f[P[k][0]] + f[P[k][1]], t = f[P[k][2]] + f[P[k][3]];
    const real d = f[P[k][0]] - f[P[k][1]], e = f[P[k][2]] - f[P[k][3]];
    B[k] = s + t;
    X[k] = s - t;
    A1[k] = d + e;
    A2[k] = d - e;
  }
  const real sx = f[1] + f[2], sy = f[3] + f[4], sz = f[5] + f[6];
  const real ax = A1[0] + A1[1], ay = A2[0] + A1[2], az = A2[1] + A2[2];
  const real gx = f[1] - f[2], gy = f[3] - f[4], gz = f[5] - f[6];
  const real jx = gx + ax, jy = gy + ay, jz = gz + az;
  const real drho = f[0] + ((sx + sy + sz) + (B[0] + B[1] + B[2]));
  const real third = real(1.0 / 3.0), sixth = real(1.0 / 6.0), two3 = real(2.0 / 3.0);
  const real xx = jx * jx, yy = jy * jy, zz = jz * jz;
  const real r9 = real(1.0 / 9.0) * drho;
  const real d1 = (sx - sy) + (B[1] - B[2]) - (xx - yy);
  const real d2 = (sx - sz) + (B[0] - B[2]) - (xx - zz);
  const real dxx = third * (d1 + d2), dyy = third * (d2 - real(2) * d1),
             dzz = third * (d1 - real(2) * d2);
  const real tr = ((B[0] + B[1] + B[2]) - f[0]) - (xx + yy + zz), t3 = third * tr;
  const real nxy = X[0] - jx * jy, nxz = X[1] - jx * jz, nyz = X[2] - jy * jz;
  // the strain-dependent relaxation time, Eqs. (19)-(21)
  const real pi2 = dxx * dxx + dyy * dyy + dzz * dzz + tr * t3 +
                   real(2) * (nxy * nxy + nxz * nxz + nyz * nyz);
  const real Qs = sqrt(real(2) * pi2);
  const real tau0 = real(p.tau0), les = real(p.cs18) * Qs;
  const real i2t = real(1) / (tau0 + sqrt(tau0 * tau0 + les));  // 1 / (2 tau)
  // 1 / tau = top - gap, gap = (2 tau - 1) / tau, 2 tau - 1 = 2 tau0 - 1 +
  // les / (2 tau) for rates near 2, else the rate itself
  const bool low = p.tau0 < 1.0;
  const real top = low ? real(2) : real(0);
  const real gap = real(2) * i2t * (low ? real(2.0 * p.tau0 - 1.0) + les * i2t : real(-1));
  const real bxy = B[0] - (r9 + third * (xx + yy) - sixth * zz);
  const real bxz = B[1] - (r9 + third * (xx + zz) - sixth * yy);
  const real byz = B[2] - (r9 + third * (yy + zz) - sixth * xx);
  // changes c of the raw moments
  const real s_tr = real(p.rates[0]);
  const real ct = s_tr * t3;
  const real cxx = top * dxx + (ct - gap * dxx), cyy = top * dyy + (ct - gap * dyy),
             czz = top * dzz + (ct - gap * dzz);
  const real q4 = real(0.25), t4 = q4 * top, g4 = q4 * gap;
  const real hs = real(0.5) * real(BASIS == 0 ? p.rates[1] : p.rates[2]);
  const real ha = real(0.5) * real(BASIS == 0 ? p.rates[2] : p.rates[4]);
  // c of a, per plane (first and second axis odd); the equilibrium's j_a/3
  // drops out of the differences, and a_ab + a_ac - 2 j_a / 3 is a third of
  // a_ab + a_ac - 2 g_a, g_a the axis populations' difference
  const real x0 = hs * (third * (ax - real(2) * gx)), x1 = ha * (A1[0] - A1[1]);
  const real y0 = hs * (third * (ay - real(2) * gy)), y1 = ha * (A2[0] - A1[2]);
  const real z0 = hs * (third * (az - real(2) * gz)), z1 = ha * (A2[1] - A2[2]);
  const real c1[3] = {x0 + x1, x0 - x1, y0 - y1}, c2[3] = {y0 + y1, z0 + z1, z0 - z1};
  real cb[3], cbs;  // c of b and their sum
  if constexpr (BASIS == 0) {
    const real s7 = real(p.rates[3]);
    cb[0] = s7 * bxy;
    cb[1] = s7 * bxz;
    cb[2] = s7 * byz;
    cbs = cb[0] + cb[1] + cb[2];
  } else {
    const real s_eps = real(p.rates[1]), s_pi = real(p.rates[3]);
    cbs = s_eps * (bxy + bxz + byz) + real(16.0 / 21.0) * (s_tr - s_eps) * tr;
    const real mix = two3 * ((s_pi - top) + gap), base = third * cbs;
    const real g1 = (B[0] - B[1]) - real(0.5) * (yy - zz);
    const real g2 = (B[0] - B[2]) - real(0.5) * (xx - zz);
    cb[0] = base + s_pi * (third * (g1 + g2)) + mix * dzz;
    cb[1] = base + s_pi * (third * (g2 - real(2) * g1)) + mix * dyy;
    cb[2] = base + s_pi * (third * (g1 - real(2) * g2)) + mix * dxx;
  }
  // D3Q19 inverse of the changes
  f[0] += real(3) * ct - cbs;
  const real h = real(0.5);
  const real ex = h * (cxx - cb[0] - cb[1]);
  const real ey = h * (cyy - cb[0] - cb[2]);
  const real ez = h * (czz - cb[1] - cb[2]);
  f[1] -= ex - x0;
  f[2] -= ex + x0;
  f[3] -= ey - y0;
  f[4] -= ey + y0;
  f[5] -= ez - z0;
  f[6] -= ez + z0;
  const real x[3] = {t4 * nxy - g4 * nxy, t4 * nxz - g4 * nxz, t4 * nyz - g4 * nyz};
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    const real e = q4 * cb[k] + x[k], o = q4 * cb[k] - x[k];
    const real d = q4 * (c1[k] + c2[k]), g = q4 * (c1[k] - c2[k]);
    f[P[k][0]] -= e + d;
    f[P[k][1]] -= e - d;
    f[P[k][2]] -= o + g;
    f[P[k][3]] -= o - g;
  }
}

}  // namespace lbm
