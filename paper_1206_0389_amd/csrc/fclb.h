// D3Q27 factorized cascaded (FCLB) collision for gfx950.
//
// Central moments (Eqs. (14)-(15)) are taken per unit mass about the local
// velocity u = j / rho (Eqs. (6)-(8)). The shear part of the second order
// relaxes with omega = 1/tau0, every other group with rate 1 (Section 2:
// s_i = 1 for i != 1): the trace goes to 1, orders 3 and 5 to 0, and the
// fourth and sixth orders to the factorized equilibria of Table 2, products
// of the relaxed second-order central moments. The whole post-collision
// moment set is recomputed and transformed back (the paper's "recompute"
// variant).
//
// In central form both transforms factor over the axes (the adjoint in
// adjoint.h differentiates this form): with D3Q27 = {-1,0,1}^3 the central
// moment matrix is a Kronecker product of three 3x3 matrices, so each
// transform is three sweeps of nine 3-point transforms held in registers.
// The arithmetic runs on deviations f_i - w_i: the rest weights factor as
// w = phi(ex) phi(ey) phi(ez) with phi = (1/6, 2/3, 1/6), whose central
// moments about u are c0 = 1, c1 = -u, c2 = 1/3 + u^2, so the rest part is
// added in closed form and every quantity in the registers stays small.
// That keeps FP32 arithmetic at the accuracy of FP32 storage.
#pragma once

#include "stencil.h"

namespace lbm {

// (f(-1), f(0), f(+1)) -> central moments of order 0, 1, 2 about u.
template <typename real>
__device__ __forceinline__ void central3(real& a0, real& a1, real& a2, real u) {
  const real s = a0 + a1 + a2;
  const real dif = a2 - a0;
  const real sum = a2 + a0;
  a0 = s;
  a1 = dif - u * s;
  a2 = sum - real(2) * u * dif + u * u * s;
}

// Inverse of central3.
template <typename real>
__device__ __forceinline__ void uncentral3(real& a0, real& a1, real& a2, real u) {
  const real m1 = a1 + u * a0;
  const real m2 = a2 + u * (real(2) * a1 + u * a0);
  const real m0 = a0;
  a0 = real(0.5) * (m2 - m1);
  a1 = m0 - m2;
  a2 = real(0.5) * (m2 + m1);
}

// Macroscopic quantities and relaxed second-order central moments of one
// node: everything the post-collision moment set depends on.
template <typename real>
struct FclbState {
  real drho, inv, ux, uy, uz;
  real ax, ay, az, bxy, bxz, byz;  // relaxed rho (kappa_aa - T/3), rho kappa_ab
};

// Forward central transform of the deviations (only the second order is
// used: every other group relaxes with rate 1) and the shear relaxation.
template <typename real>
__device__ __forceinline__ FclbState<real> fclb_relax(const real (&f)[27], real omega) {
  real A[3][3][3];
  real drho = 0, jx = 0, jy = 0, jz = 0;
#pragma unroll
  for (int i = 0; i < 27; ++i) {
    A[cx(i) + 1][cy(i) + 1][cz(i) + 1] = f[i];
    drho += f[i];
    if (cx(i)) jx += cx(i) > 0 ? f[i] : -f[i];
    if (cy(i)) jy += cy(i) > 0 ? f[i] : -f[i];
    if (cz(i)) jz += cz(i) > 0 ? f[i] : -f[i];
  }
  FclbState<real> s;
  s.drho = drho;
  const real rho = real(1) + drho;
  s.inv = real(1) / rho;
  s.ux = jx * s.inv;
  s.uy = jy * s.inv;
  s.uz = jz * s.inv;
  const real ux = s.ux, uy = s.uy, uz = s.uz;

  // Central moments D_abc of the deviations about u.
#pragma unroll
  for (int a = 0; a < 3; ++a)
#pragma unroll
    for (int b = 0; b < 3; ++b) central3(A[a][b][0], A[a][b][1], A[a][b][2], uz);
#pragma unroll
  for (int a = 0; a < 3; ++a)
#pragma unroll
    for (int c = 0; c < 3; ++c) central3(A[a][0][c], A[a][1][c], A[a][2][c], uy);
#pragma unroll
  for (int b = 0; b < 3; ++b)
#pragma unroll
    for (int c = 0; c < 3; ++c) central3(A[0][b][c], A[1][b][c], A[2][b][c], ux);

  const real third = real(1.0 / 3.0);
  const real omc = real(1) - omega;
  const real uu = ux * ux + uy * uy + uz * uz;
  const real dtr = A[2][0][0] + A[0][2][0] + A[0][0][2];
  // rho (kappa_aa - T/3) relaxed with omega; rho kappa_ab relaxed with omega
  s.ax = omc * ((ux * ux + A[2][0][0]) - third * (uu + dtr));
  s.ay = omc * ((uy * uy + A[0][2][0]) - third * (uu + dtr));
  s.az = omc * ((uz * uz + A[0][0][2]) - third * (uu + dtr));
  s.bxy = omc * (ux * uy + A[1][1][0]);
  s.bxz = omc * (ux * uz + A[1][0][1]);
  s.byz = omc * (uy * uz + A[0][1][1]);
  return s;
}

// Post-collision central moments G = rho kappa* minus the central moments
// of the rest weights about u, then the inverse transform to deviations.
template <typename real>
__device__ __forceinline__ void fclb_post(const FclbState<real>& s, real (&A)[3][3][3]) {
  const real drho = s.drho, inv = s.inv, ux = s.ux, uy = s.uy, uz = s.uz;
  const real ax = s.ax, ay = s.ay, az = s.az, bxy = s.bxy, bxz = s.bxz, byz = s.byz;
  const real third = real(1.0 / 3.0);
  const real ux2 = ux * ux, uy2 = uy * uy, uz2 = uz * uz;
  const real uu = ux2 + uy2 + uz2;
  const real c2x = third + ux2, c2y = third + uy2, c2z = third + uz2;
  A[0][0][0] = drho;
  A[1][0][0] = ux;
  A[0][1][0] = uy;
  A[0][0][1] = uz;
  A[2][0][0] = third * drho + ax - ux2;
  A[0][2][0] = third * drho + ay - uy2;
  A[0][0][2] = third * drho + az - uz2;
  A[1][1][0] = bxy - ux * uy;
  A[1][0][1] = bxz - ux * uz;
  A[0][1][1] = byz - uy * uz;
  A[2][1][0] = c2x * uy;
  A[2][0][1] = c2x * uz;
  A[1][2][0] = ux * c2y;
  A[0][2][1] = c2y * uz;
  A[1][0][2] = ux * c2z;
  A[0][1][2] = uy * c2z;
  A[1][1][1] = ux * uy * uz;
  const real ninth = real(1.0 / 9.0);
  A[2][2][0] = ninth * drho + third * (ax + ay - ux2 - uy2) + ax * ay * inv - ux2 * uy2;
  A[2][0][2] = ninth * drho + third * (ax + az - ux2 - uz2) + ax * az * inv - ux2 * uz2;
  A[0][2][2] = ninth * drho + third * (ay + az - uy2 - uz2) + ay * az * inv - uy2 * uz2;
  A[2][1][1] = third * (byz - uy * uz) + ax * inv * byz - ux2 * uy * uz;
  A[1][2][1] = third * (bxz - ux * uz) + ay * inv * bxz - uy2 * ux * uz;
  A[1][1][2] = third * (bxy - ux * uy) + az * inv * bxy - uz2 * ux * uy;
  A[2][2][1] = c2x * c2y * uz;
  A[2][1][2] = c2x * uy * c2z;
  A[1][2][2] = ux * c2y * c2z;
  A[2][2][2] = real(1.0 / 27.0) * drho + ninth * (ax + ay + az - uu) +
               third * inv * (ax * ay + ax * az + ay * az) + ax * ay * az * inv * inv -
               third * (ux2 * uy2 + ux2 * uz2 + uy2 * uz2) - ux2 * uy2 * uz2;

#pragma unroll
  for (int b = 0; b < 3; ++b)
#pragma unroll
    for (int c = 0; c < 3; ++c) uncentral3(A[0][b][c], A[1][b][c], A[2][b][c], ux);
#pragma unroll
  for (int a = 0; a < 3; ++a)
#pragma unroll
    for (int c = 0; c < 3; ++c) uncentral3(A[a][0][c], A[a][1][c], A[a][2][c], uy);
#pragma unroll
  for (int a = 0; a < 3; ++a)
#pragma unroll
    for (int b = 0; b < 3; ++b) uncentral3(A[a][b][0], A[a][b][1], A[a][b][2], uz);
}

// ---------------------------------------------------------------- collision
// The collision itself runs on raw moments. With j = rho u, the central
// second moments of f + w are k_aa = R_aa - j_a u_a, k_ab = R_ab - j_a u_b (R
// the raw moments of the deviations, the rest part cancelling), so the
// forward side needs ten sums and no u-dependent sweep. Central moments that
// are products of the second order make the raw ones products too (P_a =
// rho (kappa_aa + u_a^2), b_ab = rho kappa_ab after the relaxation):
//   M_110 = b_xy + j_x u_y              M_210 = P_x u_y + 2 u_x b_xy
//   M_111 = u_x b_yz + u_y b_xz + u_z M_110
//   M_220 = P_x P_y / rho + 4 u_x u_y b_xy
//   M_211 = P_x M_011 / rho + 2 u_x (u_y b_xz + u_z b_xy)
//   M_221 = u_z M_220 + 2 (u_y b_yz P_x + u_x b_xz P_y) / rho
//   M_222 = P_x P_y P_z / rho^2 + 4 (u_x u_y b_xy P_z + ...) / rho
// less the rest moments 1, 1/3, 1/9, 1/27, expanded so that only deviations
// are summed. The CLB's independent Gaussian fourth and sixth orders change
// the M with two or more even orders (GAUSS). The inverse is three sweeps of
// (m0, m1, m2) -> (m2 - m1, m0 - 2 m2, m2 + m1) on moments scaled by 1/2 per
// non-zero order: three operations a line and no velocity.
// Measured: 344 VALU instructions per node in the FP32 even step, 631 with
// the u-dependent sweeps of both directions. FP16 storage, which is bound by
// them, gains 9 % (256x256x512 jet, 10 steps and a snapshot: 8.13 to 7.45
// ms); FP32 is bound by its memory accesses (14.44 and 14.53 ms with the
// populations read out). Error after 10 steps against 64 bits 2.3e-7 to
// 1.7e-7 of the populations.

// Raw moments of one node: density, momentum, velocity and the relaxed
// second-order central moments (rho kappa_aa - T/3, rho kappa_ab).
template <typename real>
struct FclbRaw {
  real drho, inv, jx, jy, jz, ux, uy, uz;
  real ax, ay, az, bxy, bxz, byz;
};

template <typename real>
__device__ __forceinline__ FclbRaw<real> fclb_raw(const real (&f)[27], real omega) {
  // sums along z of the nine lines (all, first and second order), then along
  // y, then along x
  real s[3][3], d[3][3], q[3][3];
#pragma unroll
  for (int a = 0; a < 3; ++a)
#pragma unroll
    for (int b = 0; b < 3; ++b) {
      const real lo = f[index_of(a - 1, b - 1, -1)], mid = f[index_of(a - 1, b - 1, 0)],
                 hi = f[index_of(a - 1, b - 1, 1)];
      q[a][b] = lo + hi;
      d[a][b] = hi - lo;
      s[a][b] = mid + q[a][b];
    }
  real s0[3], s1[3], s2[3], d0[3], d1[3], q0[3];
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    s2[a] = s[a][0] + s[a][2];
    s1[a] = s[a][2] - s[a][0];
    s0[a] = s[a][1] + s2[a];
    d0[a] = d[a][0] + d[a][1] + d[a][2];
    d1[a] = d[a][2] - d[a][0];
    q0[a] = q[a][0] + q[a][1] + q[a][2];
  }
  FclbRaw<real> m;
  const real rxx = s0[0] + s0[2], ryy = s2[0] + s2[1] + s2[2], rzz = q0[0] + q0[1] + q0[2];
  const real rxy = s1[2] - s1[0], rxz = d0[2] - d0[0], ryz = d1[0] + d1[1] + d1[2];
  m.drho = s0[1] + rxx;
  m.jx = s0[2] - s0[0];
  m.jy = s1[0] + s1[1] + s1[2];
  m.jz = d0[0] + d0[1] + d0[2];
  m.inv = real(1) / (real(1) + m.drho);
  m.ux = m.jx * m.inv;
  m.uy = m.jy * m.inv;
  m.uz = m.jz * m.inv;
  const real omc = real(1) - omega;
  const real kx = rxx - m.jx * m.ux, ky = ryy - m.jy * m.uy, kz = rzz - m.jz * m.uz;
  const real tr = real(1.0 / 3.0) * (kx + ky + kz);
  m.ax = omc * (kx - tr);
  m.ay = omc * (ky - tr);
  m.az = omc * (kz - tr);
  m.bxy = omc * (rxy - m.jx * m.uy);
  m.bxz = omc * (rxz - m.jx * m.uz);
  m.byz = omc * (ryz - m.jy * m.uz);
  return m;
}

// One line of the inverse transform (scaled moments to populations).
template <typename real>
__device__ __forceinline__ void raw_line(real& m0, real& m1, real& m2) {
  const real lo = m2 - m1, hi = m2 + m1, mid = m0 - real(2) * m2;
  m0 = lo;
  m1 = mid;
  m2 = hi;
}

template <typename real, bool GAUSS = false>
__device__ __forceinline__ void fclb_collide(real (&f)[27], real omega) {
  const FclbRaw<real> m = fclb_raw(f, omega);
  const real drho = m.drho, inv = m.inv, ux = m.ux, uy = m.uy, uz = m.uz;
  const real ax = m.ax, ay = m.ay, az = m.az, bxy = m.bxy, bxz = m.bxz, byz = m.byz;
  const real third = real(1.0 / 3.0), ninth = real(1.0 / 9.0), t27 = real(1.0 / 27.0);
  const real px = third * drho + ax + m.jx * ux, py = third * drho + ay + m.jy * uy,
             pz = third * drho + az + m.jz * uz;
  const real Px = third + px, Py = third + py, Pz = third + pz;
  const real qxy = bxy + m.jx * uy, qxz = bxz + m.jx * uz, qyz = byz + m.jy * uz;
  const real vx = real(2) * ux, vy = real(2) * uy, vz = real(2) * uz;
  real A[3][3][3];
  A[0][0][0] = drho;
  A[1][0][0] = real(0.5) * m.jx;
  A[0][1][0] = real(0.5) * m.jy;
  A[0][0][1] = real(0.5) * m.jz;
  A[2][0][0] = real(0.5) * px;
  A[0][2][0] = real(0.5) * py;
  A[0][0][2] = real(0.5) * pz;
  A[1][1][0] = real(0.25) * qxy;
  A[1][0][1] = real(0.25) * qxz;
  A[0][1][1] = real(0.25) * qyz;
  A[2][1][0] = real(0.25) * (Px * uy + vx * bxy);
  A[2][0][1] = real(0.25) * (Px * uz + vx * bxz);
  A[1][2][0] = real(0.25) * (Py * ux + vy * bxy);
  A[0][2][1] = real(0.25) * (Py * uz + vy * byz);
  A[1][0][2] = real(0.25) * (Pz * ux + vz * bxz);
  A[0][1][2] = real(0.25) * (Pz * uy + vz * byz);
  A[1][1][1] = real(0.125) * (ux * byz + uy * bxz + uz * qxy);
  if constexpr (!GAUSS) {
    const real exy = inv * (third * (px + py) + px * py - ninth * drho);
    const real exz = inv * (third * (px + pz) + px * pz - ninth * drho);
    const real eyz = inv * (third * (py + pz) + py * pz - ninth * drho);
    const real wxy = vx * vy * bxy, wxz = vx * vz * bxz, wyz = vy * vz * byz;
    const real mxy = exy + wxy, mxz = exz + wxz, myz = eyz + wyz;
    A[2][2][0] = real(0.25) * mxy;
    A[2][0][2] = real(0.25) * mxz;
    A[0][2][2] = real(0.25) * myz;
    const real Ix = Px * inv, Iy = Py * inv, Iz = Pz * inv;
    A[2][1][1] = real(0.125) * (Ix * qyz + vx * (uy * bxz + uz * bxy));
    A[1][2][1] = real(0.125) * (Iy * qxz + vy * (ux * byz + uz * bxy));
    A[1][1][2] = real(0.125) * (Iz * qxy + vz * (ux * byz + uy * bxz));
    A[2][2][1] = real(0.125) * (uz * (ninth + mxy) + vy * byz * Ix + vx * bxz * Iy);
    A[2][1][2] = real(0.125) * (uy * (ninth + mxz) + vz * byz * Ix + vx * bxy * Iz);
    A[1][2][2] = real(0.125) * (ux * (ninth + myz) + vz * bxz * Iy + vy * bxy * Iz);
    A[2][2][2] = real(0.125) * (inv * (third * exy + ninth * pz + exy * pz - t27 * drho) +
                                wxy * Iz + wxz * Iy + wyz * Ix);
  } else {
    // rho kappa_aa
    const real rho3 = third + third * drho;
    const real Kx = rho3 + ax, Ky = rho3 + ay, Kz = rho3 + az;
    const real ux2 = ux * ux, uy2 = uy * uy, uz2 = uz * uz;
    const real sx = m.jx * ux, sy = m.jy * uy;  // rho u_a^2
    const real wxy = vx * vy * bxy, wxz = vx * vz * bxz, wyz = vy * vz * byz;
    const real mxy = ninth * drho + ux2 * Ky + uy2 * Kx + sx * uy2 + wxy;
    const real mxz = ninth * drho + ux2 * Kz + uz2 * Kx + sx * uz2 + wxz;
    const real myz = ninth * drho + uy2 * Kz + uz2 * Ky + sy * uz2 + wyz;
    A[2][2][0] = real(0.25) * mxy;
    A[2][0][2] = real(0.25) * mxz;
    A[0][2][2] = real(0.25) * myz;
    A[2][1][1] = real(0.125) * (Px * uy * uz + ux2 * byz + vx * (uy * bxz + uz * bxy));
    A[1][2][1] = real(0.125) * (Py * ux * uz + uy2 * bxz + vy * (ux * byz + uz * bxy));
    A[1][1][2] = real(0.125) * (Pz * ux * uy + uz2 * bxy + vz * (ux * byz + uy * bxz));
    A[2][2][1] = real(0.125) * (uz * (ninth + mxy) + vx * uy2 * bxz + vy * ux2 * byz);
    A[2][1][2] = real(0.125) * (uy * (ninth + mxz) + vx * uz2 * bxy + vz * ux2 * byz);
    A[1][2][2] = real(0.125) * (ux * (ninth + myz) + vy * uz2 * bxy + vz * uy2 * bxz);
    A[2][2][2] = real(0.125) * (t27 * drho + ninth * (real(1) + drho) * (ux2 + uy2 + uz2) +
        ux2 * uy2 * Kz + ux2 * uz2 * Ky + uy2 * uz2 * Kx + sx * uy2 * uz2 +
        wxy * uz2 + wxz * uy2 + wyz * ux2);
  }
#pragma unroll
  for (int a = 0; a < 3; ++a)
#pragma unroll
    for (int b = 0; b < 3; ++b) raw_line(A[a][b][0], A[a][b][1], A[a][b][2]);
#pragma unroll
  for (int a = 0; a < 3; ++a)
#pragma unroll
    for (int c = 0; c < 3; ++c) raw_line(A[a][0][c], A[a][1][c], A[a][2][c]);
#pragma unroll
  for (int b = 0; b < 3; ++b)
#pragma unroll
    for (int c = 0; c < 3; ++c) raw_line(A[0][b][c], A[1][b][c], A[2][b][c]);
#pragma unroll
  for (int i = 0; i < 27; ++i) f[i] = A[cx(i) + 1][cy(i) + 1][cz(i) + 1];
}

}  // namespace lbm
