// The collision and the wall force of one node, shared by the collide-stream
// kernels.
#pragma once

#include "internal.h"
#include "stream.h"

namespace lbm {

// Reichardt wall force of a first off-wall cell (Sec. II.C, Eq. (16)-(21)):
// base vector from the tangential part of u_2, projected speed u_hat, u_tau
// from a fixed number of Newton steps on u_tau u+(y u_tau / nu0) = |u_hat|,
// F_w = -sign(u_hat) rho u_tau^2 e_x.  The wall normal is along y.
//
// With the line-averaged model (wall_line set) u_tau is the signed value of
// the cell's wall line, computed by wall_line_kernel from the z-mean of u_hat.
__device__ __forceinline__ void wall_force(const CollideArgs& a, float rho, float uwx, float uwz, float u2x,
                                           float u2z, float& fx, float& fz, float& ut_out, int w, int x) {
  fx = 0.f;
  fz = 0.f;
  ut_out = 0.f;
  const float line = a.wall_line ? a.wall_line[w * a.nx + x] : 0.f;
  if (a.wall_line) ut_out = fabsf(line);
  const float tn2 = u2x * u2x + u2z * u2z;
  if (!(tn2 > 0.f)) return;
  const float itn = 1.f / sqrtf(tn2);
  const float ex = u2x * itn, ez = u2z * itn;
  if (a.wall_line) {
    const float tw = (line > 0.f ? -1.f : 1.f) * rho * line * line;
    fx = tw * ex;
    fz = tw * ez;
    return;
  }
  const float uhat = uwx * ex + uwz * ez;
  if (uhat == 0.f) return;
  const float ut = newton_utau(a, fabsf(uhat));
  const float tw = (uhat > 0.f ? -1.f : 1.f) * rho * ut * ut;
  fx = tw * ex;
  fz = tw * ez;
  ut_out = ut;
}

// MRT collision with Guo forcing in moment space and the Smagorinsky
// relaxation time (Sec. II.A-II.B, Eq. (6)-(15)), written as
// f* = f + M^-1 delta with delta_k = -s_k (m_k - m_eq_k) + (1 - s_k/2) F_k.
// The moment transform uses the even/odd split of the basis over the
// opposite-direction pairs (i, 18 - i).  Returns the force-corrected velocity.
//
// DEV: f holds the deviations h_i = f_i - w_i and is updated as h* = h + M^-1
// delta; pr are the pair sums of h and rhoh = rho - 1.  The weights add only
// to m_0 = rho, m_1 (-11) and m_2 (3), which enter through e_1 and e_2.
template <bool FORCE, bool DEV = false>
__device__ __forceinline__ void collide(const CollideArgs& a, const Tau0& t0, float f[Q], const Pairs& pr, float rho,
                                        float jx, float jy, float jz, float Fx, float Fy, float Fz, float& ux,
                                        float& uy, float& uz, float rhoh = 0.f) {
  const float* s = pr.s;
  const float* d = pr.d;
  const float f9 = f[9];
  const float A = pr.A;
  const float Bx = pr.Bx;
  const float T04 = s[0] + s[4], T26 = s[2] + s[6], T1357 = s[1] + s[3] + s[5] + s[7];
  const float m1 = 8.f * A - 11.f * Bx - 30.f * f9;
  const float m2 = A - 4.f * Bx + 12.f * f9;
  const float m9 = 2.f * (s[8] - T04) + T1357 - T26;
  const float m10 = -2.f * T04 + T1357 + 2.f * T26 - 4.f * s[8];
  const float m11 = (s[5] + s[6] + s[7]) - (s[1] + s[2] + s[3]);
  const float m12 = (s[5] + s[7] - 2.f * s[6]) - (s[1] + s[3] - 2.f * s[2]);
  const float m13 = s[5] - s[7], m14 = s[0] - s[4], m15 = s[1] - s[3];
  const float m4 = (d[3] + d[7]) - (d[1] + d[5]) + 4.f * d[8];
  const float m6 = d[4] - (d[0] + d[5] + d[7]) + 4.f * d[6];
  const float m8 = 4.f * d[2] - (d[0] + d[1] + d[3] + d[4]);
  const float m16 = (d[1] + d[7]) - (d[3] + d[5]);
  const float m17 = (d[4] + d[5] + d[7]) - d[0];
  const float m18 = (d[0] + d[4]) - (d[1] + d[3]);

  // Eq. (11): rho u = j + F/2;  Eq. (8) equilibria (with the readings of m2, m4,6,8)
  const float ir = rcp_fast(rho);
  const float px = FORCE ? jx + 0.5f * Fx : jx;
  const float py = FORCE ? jy + 0.5f * Fy : jy;
  const float pz = FORCE ? jz + 0.5f * Fz : jz;
  ux = px * ir;
  uy = py * ir;
  uz = pz * ir;
  const float uxx = ux * ux, uyy = uy * uy, uzz = uz * uz, uu = uxx + uyy + uzz;
  const float e1 = DEV ? m1 + 11.f * rhoh - 19.f * rho * uu : m1 - rho * (19.f * uu - 11.f);
  const float e2 = DEV ? m2 - 3.f * rhoh + 5.5f * rho * uu : m2 - rho * (3.f - 5.5f * uu);
  const float e4 = m4 + (2.f / 3.f) * px;
  const float e6 = m6 + (2.f / 3.f) * py;
  const float e8 = m8 + (2.f / 3.f) * pz;
  const float q9 = rho * (2.f * uxx - uyy - uzz);
  const float q11 = rho * (uyy - uzz);
  const float e9 = m9 - q9, e10 = m10 + 0.5f * q9;
  const float e11 = m11 - q11, e12 = m12 + 0.5f * q11;
  const float e13 = m13 - px * uy, e14 = m14 - py * uz, e15 = m15 - px * uz;

  // Sec. II.B: Pi_neq from the non-equilibrium moments, Q^(1/2) = |Pi_neq|,
  // tau_eff = tau0/2 + sqrt(tau0^2 + 18 sqrt(2) C_smag Q^(1/2) / rho)/2
  const float dc2 = e1 * (1.f / 19.f);
  const float pxx = (e9 + dc2) * (1.f / 3.f);
  const float pyy = 0.5f * (dc2 - pxx + e11), pzz = 0.5f * (dc2 - pxx - e11);
  const float q2 = pxx * pxx + pyy * pyy + pzz * pzz + 2.f * (e13 * e13 + e14 * e14 + e15 * e15);
  const float tau = 0.5f * t0.tau0 + 0.5f * sqrt_fast(t0.tau0sq + a.smag * sqrt_fast(q2) * ir);
  const float sv = rcp_fast(tau);
  const float hv = 1.f - 0.5f * sv;

  // Guo forcing moments M Fbar = (1/rho) d m_eq/du . F
  float F1 = 0.f, F2 = 0.f, F4 = 0.f, F6 = 0.f, F8 = 0.f, F9 = 0.f, F10 = 0.f, F11 = 0.f, F12 = 0.f;
  float F13 = 0.f, F14 = 0.f, F15 = 0.f;
  if (FORCE) {
    const float uF = ux * Fx + uy * Fy + uz * Fz;
    F1 = 38.f * uF;
    F2 = -11.f * uF;
    F4 = (-2.f / 3.f) * Fx;
    F6 = (-2.f / 3.f) * Fy;
    F8 = (-2.f / 3.f) * Fz;
    F9 = 2.f * (2.f * ux * Fx - uy * Fy - uz * Fz);
    F10 = -0.5f * F9;
    F11 = 2.f * (uy * Fy - uz * Fz);
    F12 = -0.5f * F11;
    F13 = ux * Fy + uy * Fx;
    F14 = uy * Fz + uz * Fy;
    F15 = ux * Fz + uz * Fx;
  }
  // delta_k / D_k
  const float a1 = FORCE ? -a.rs[1] * e1 + a.rf[1] * F1 : -a.rs[1] * e1;
  const float a2 = FORCE ? -a.rs[2] * e2 + a.rf[2] * F2 : -a.rs[2] * e2;
  const float a9 = (FORCE ? -sv * e9 + hv * F9 : -sv * e9) * (1.f / 36.f);
  const float a10 = FORCE ? -a.rs[10] * e10 + a.rf[10] * F10 : -a.rs[10] * e10;
  const float a11 = (FORCE ? -sv * e11 + hv * F11 : -sv * e11) * (1.f / 12.f);
  const float a12 = FORCE ? -a.rs[12] * e12 + a.rf[12] * F12 : -a.rs[12] * e12;
  const float a13 = (FORCE ? -sv * e13 + hv * F13 : -sv * e13) * 0.25f;
  const float a14 = (FORCE ? -sv * e14 + hv * F14 : -sv * e14) * 0.25f;
  const float a15 = (FORCE ? -sv * e15 + hv * F15 : -sv * e15) * 0.25f;
  const float b3 = 0.1f * Fx, b5 = 0.1f * Fy, b7 = 0.1f * Fz;
  const float b4 = FORCE ? -a.rs[4] * e4 + a.rf[4] * F4 : -a.rs[4] * e4;
  const float b6 = FORCE ? -a.rs[6] * e6 + a.rf[6] * F6 : -a.rs[6] * e6;
  const float b8 = FORCE ? -a.rs[8] * e8 + a.rf[8] * F8 : -a.rs[8] * e8;
  const float b16 = -a.rs[16] * m16, b17 = -a.rs[17] * m17, b18 = -a.rs[18] * m18;

  // f* = f + M^T diag(1/D) delta, assembled per opposite pair
  const float P = 8.f * a1 + a2, Qx = -11.f * a1 - 4.f * a2, R9 = -30.f * a1 + 12.f * a2;
  const float b910 = a9 + a10, c1112 = a11 + a12;
  const float h = 2.f * a10 - a9, kk = 2.f * a12 - a11;
  float E[9], O[9];
  E[0] = P - 2.f * b910 + a14;
  E[4] = P - 2.f * b910 - a14;
  E[1] = P + b910 - c1112 + a15;
  E[3] = P + b910 - c1112 - a15;
  E[5] = P + b910 + c1112 + a13;
  E[7] = P + b910 + c1112 - a13;
  E[2] = Qx + h + kk;
  E[6] = Qx + h - kk;
  E[8] = Qx + 2.f * a9 - 4.f * a10;
  const float B34 = FORCE ? b3 + b4 : b4, B56 = FORCE ? b5 + b6 : b6, B78 = FORCE ? b7 + b8 : b8;
  O[0] = -B56 - B78 - b17 + b18;
  O[4] = B56 - B78 + b17 + b18;
  O[1] = -B34 - B78 + b16 - b18;
  O[3] = B34 - B78 - b16 - b18;
  O[5] = -B34 - B56 - b16 + b17;
  O[7] = B34 - B56 + b16 + b17;
  O[2] = 4.f * b8 - (FORCE ? b7 : 0.f);
  O[6] = 4.f * b6 - (FORCE ? b5 : 0.f);
  O[8] = 4.f * b4 - (FORCE ? b3 : 0.f);
#pragma unroll
  for (int k = 0; k < 9; ++k) {
    const float lo = f[k], hi = f[18 - k];
    f[k] = lo + E[k] + O[k];
    f[18 - k] = hi + E[k] - O[k];
  }
  f[9] = f9 + R9;
}

}  // namespace lbm
