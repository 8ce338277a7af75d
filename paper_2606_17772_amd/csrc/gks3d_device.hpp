// Device arithmetic of the 3D gas-kinetic solvers for gfx950: the BGK
// interface solver and the smooth nodal solver of App. A with the collision
// invariants psi = (1, u, v, w, (u^2 + v^2 + w^2 + xi^2)/2), in FP64.
//
// The form is that of the 2D solver (gks_device.hpp): slopes of a Maxwellian
// as derivatives of its logarithm in the primitive variables, everything but
// the normal velocity u integrated in closed form, 1D moment sums of cubics of
// u; nodal fluxes in closed form.  Bound by FP64 issue and registers: the
// moment vectors of psi of the earlier form took 440 registers (one wave per
// SIMD) and 4,797 flop per solve at stage 1.
#pragma once

#include "gks_device.hpp"

namespace fdk3 {

using fdk::Consts;
using fdk::TimeCoef;
using fdk::m_abs;
using fdk::m_recip;

struct Prim {
  double rho, irho, U, V, Wv, p, lam, i2l, ip;  // i2l = 1/(2 lambda) = p/rho = theta, ip = 1/p
};
FDK_HD Prim prim(const double* W, double gamma) {
  Prim s;
  s.rho = W[0];
  s.irho = m_recip(W[0]);
  s.U = W[1] * s.irho;
  s.V = W[2] * s.irho;
  s.Wv = W[3] * s.irho;
  s.p = (gamma - 1.0) * (W[4] - 0.5 * s.rho * (s.U * s.U + s.V * s.V + s.Wv * s.Wv));
  s.i2l = s.p * s.irho;
  s.ip = m_recip(s.p);
  s.lam = 0.5 * s.rho * s.ip;
  return s;
}

// rho_x / rho, U_x, V_x, W_x, theta_x of a slope (or the time derivatives)
struct PSlope {
  double r, u, v, w, th;
};
// Slopes of the primitive variables from the derivative d of the conservative ones.
FDK_HD PSlope prim_slope(const Prim& s, double g1, const double* d) {
  PSlope o;
  o.r = d[0] * s.irho;
  o.u = d[1] * s.irho - s.U * o.r;
  o.v = d[2] * s.irho - s.V * o.r;
  o.w = d[3] * s.irho - s.Wv * o.r;
  const double k2 = 0.5 * (s.U * s.U + s.V * s.V + s.Wv * s.Wv);
  const double e = d[4] * s.irho - k2 * o.r - s.U * o.u - s.V * o.v - s.Wv * o.w;  // (p_x / rho) / (gamma - 1)
  o.th = g1 * e - s.i2l * o.r;
  return o;
}
// Euler time derivatives of the primitive variables
FDK_HD PSlope euler_slope(const Prim& s, double g1, const PSlope& a, const PSlope& b, const PSlope& c) {
  PSlope t;
  const double div = a.u + b.v + c.w, th = s.i2l;
  t.r = -(div + s.U * a.r + s.V * b.r + s.Wv * c.r);
  t.u = -(a.th + th * a.r + s.U * a.u + s.V * b.u + s.Wv * c.u);
  t.v = -(b.th + th * b.r + s.U * a.v + s.V * b.v + s.Wv * c.v);
  t.w = -(c.th + th * c.r + s.U * a.w + s.V * b.w + s.Wv * c.w);
  t.th = -(g1 * th * div + s.U * a.th + s.V * b.th + s.Wv * c.th);
  return t;
}
// a(u) of a slope: <a.psi> over the full lines of v, w, xi (see gks_device.hpp)
FDK_HD void slope_poly(const Prim& s, double ith, const PSlope& a, double* o) {
  const double ux = a.u * ith;
  o[2] = 0.5 * a.th * (ith * ith);
  o[1] = ux - 2.0 * s.U * o[2];
  o[0] = a.r - s.i2l * o[2] - s.U * (o[1] + s.U * o[2]);
}
// Conservative time derivative of a state from the primitive one
FDK_HD void cons_t(const Prim& s, double hK, const PSlope& t, double* Wt) {
  const double rt = s.rho * t.r;
  Wt[0] = rt;
  Wt[1] = s.rho * t.u + s.U * rt;
  Wt[2] = s.rho * t.v + s.V * rt;
  Wt[3] = s.rho * t.w + s.Wv * rt;
  Wt[4] = s.U * Wt[1] + s.V * Wt[2] + s.Wv * Wt[3] + hK * (s.rho * t.th) +
          (hK * s.i2l - 0.5 * (s.U * s.U + s.V * s.V + s.Wv * s.Wv)) * rt;
}

// Local frame: the normal velocity is component 1 (u); v and w are the
// tangential velocities, Wt and Wt2 the tangential slopes along their axes.
struct GksIO3 {
  double WL[5], WR[5], nL[5], nR[5], Wt[5], Wt2[5];
  double F[5], Ft[5], Wl[5], Wr[5], Wlt[5], Wrt[5];
};

// One state's contribution (a side over its half line, or the equilibrium
// over the full line; m0, m1 its <1>, <u>): adds the moments
// rho <phi [k0 + kA A.psi + kg ((a.psi) u + (b.psi) v + (c.psi) w)]> for phi =
// psi to We / Wet and for phi = u psi to F / Ft, with the coefficients ca (of
// f^n, VALUES) and cb (of f_t^n); F[0] = We[1] and Ft[0] = Wet[1] are left to
// the caller.  Wt receives the state's Euler time derivative (conservative).
template <bool VALUES>
FDK_HD void state_terms(const Prim& s, double kappa, double hK, double g1, double m0, double m1, const double* n,
                        const double* tv, const double* tw, const double* ca, const double* cb, double* We, double* F,
                        double* Wet, double* Ft, double* Wt) {
  const double th = s.i2l, ith = 2.0 * s.lam;
  const double hE = kappa * th + 0.5 * (s.V * s.V + s.Wv * s.Wv);
  const PSlope a = prim_slope(s, g1, n), b = prim_slope(s, g1, tv), c = prim_slope(s, g1, tw);
  const PSlope t = euler_slope(s, g1, a, b, c);
  cons_t(s, hK, t, Wt);
  double mu[7], A[3], g[4], nv[2], nw[2], eg[2];
  mu[0] = m0;
  mu[1] = m1;
  fdk::mu_rec(mu, s.U, th);
  slope_poly(s, ith, t, A);
  {
    double pa[3], pb[3], pc[3];
    slope_poly(s, ith, a, pa);
    slope_poly(s, ith, b, pb);
    slope_poly(s, ith, c, pc);
    // weight 1: cubic of u; weights v' and w': quadratics; weight e' = (v'^2 + w'^2 + xi^2) / 2
    g[0] = b.v + c.w + s.V * pb[0] + s.Wv * pc[0];
    g[1] = pa[0] + s.V * pb[1] + s.Wv * pc[1];
    g[2] = pa[1] + s.V * pb[2] + s.Wv * pc[2];
    g[3] = pa[2];
    const double v0 = b.th + s.V * b.v + s.Wv * c.v + th * pb[0], v1 = a.v + th * pb[1], v2 = th * pb[2];
    const double w0 = c.th + s.V * b.w + s.Wv * c.w + th * pc[0], w1 = a.w + th * pc[1], w2 = th * pc[2];
    const double e0 = th * (b.v + c.w) + kappa * (s.V * b.th + s.Wv * c.th), e1 = kappa * a.th;
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      nv[q] = v0 * mu[q] + v1 * mu[q + 1] + v2 * mu[q + 2];
      nw[q] = w0 * mu[q] + w1 * mu[q + 1] + w2 * mu[q + 2];
      eg[q] = e0 * mu[q] + e1 * mu[q + 1] + s.V * nv[q] + s.Wv * nw[q];
    }
  }
  const double et = kappa * t.th + s.V * t.v + s.Wv * t.w;
  auto add = [&](const double* cf, double* W, double* G) {
    const double k0 = s.rho * cf[0], kA = s.rho * cf[1], kg = s.rho * cf[2];
    const double p0 = k0 + kA * A[0] + kg * g[0], p1 = kA * A[1] + kg * g[1], p2 = kA * A[2] + kg * g[2];
    const double p3 = kg * g[3];
    double M[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) M[q] = p0 * mu[q] + p1 * mu[q + 1] + p2 * mu[q + 2] + p3 * mu[q + 3];
    const double av = kA * t.v, aw = kA * t.w, ae = kA * et;
    W[0] = W[0] + M[0];
    W[1] = W[1] + M[1];
    G[1] = G[1] + M[2];
    W[2] = W[2] + s.V * M[0] + av * mu[0] + kg * nv[0];
    G[2] = G[2] + s.V * M[1] + av * mu[1] + kg * nv[1];
    W[3] = W[3] + s.Wv * M[0] + aw * mu[0] + kg * nw[0];
    G[3] = G[3] + s.Wv * M[1] + aw * mu[1] + kg * nw[1];
    W[4] = W[4] + 0.5 * M[2] + hE * M[0] + ae * mu[0] + kg * eg[0];
    G[4] = G[4] + 0.5 * M[3] + hE * M[1] + ae * mu[1] + kg * eg[1];
  };
  if (VALUES) add(ca, We, F);
  add(cb, Wet, Ft);
}

// Interface solver (App. A1-A2): flux, its time derivative and the values of
// Eq. W-model with their time derivatives.  VALUES = false skips F and the
// values (stage 2 uses only time derivatives).
template <bool VALUES> FDK_HD void gks_iface(const Consts& k, double dt, GksIO3& io) {
  const double gam = k.gamma, g1 = gam - 1.0, kappa = 0.5 * (k.K + 2.0), hK = 0.5 * (k.K + 3.0);
  const Prim sL = prim(io.WL, gam), sR = prim(io.WR, gam);
  // half-line moments <1> and x = <u> - U <1>, and the compatibility state
  double mL, mR, xL, xR, W0[5];
  fdk::half_moms(sL.lam, sL.i2l, sL.U, 1.0, mL, xL);
  fdk::half_moms(sR.lam, sR.i2l, sR.U, -1.0, mR, xR);
  {
    const double XL = sL.rho * xL, XR = sR.rho * xR;
#pragma unroll
    for (int i = 0; i < 5; ++i) W0[i] = mL * io.WL[i] + mR * io.WR[i];
    W0[1] = W0[1] + (XL + XR);
    W0[4] = W0[4] + 0.5 * (sL.U * XL + sR.U * XR);
  }
  const Prim s0 = prim(W0, gam);
  const double tau = (k.mu > 0 ? k.mu * s0.ip : k.tau_c1 * dt) +
                     k.tau_c2 * dt * m_abs(sL.p - sR.p) * m_recip(sL.p + sR.p);
  const TimeCoef<double> tc = fdk::time_coef(dt, tau);
  double F[5], Ft[5], We[5], Wet[5], WtL[5], WtR[5];
  // equilibrium: its leading terms are W0 and the Euler flux of W0
  {
    const double H = W0[4] + s0.p;
    const double fe[5] = {W0[1], s0.p + s0.U * W0[1], s0.V * W0[1], s0.Wv * W0[1], s0.U * H};
    double nm[5], Wt0[5];
#pragma unroll
    for (int i = 0; i < 5; ++i) {
      F[i] = VALUES ? tc.c[0] * fe[i] : 0.0;
      We[i] = VALUES ? tc.c[0] * W0[i] : 0.0;
      Ft[i] = tc.ct[0] * fe[i];
      Wet[i] = tc.ct[0] * W0[i];
      nm[i] = 0.5 * (io.nL[i] + io.nR[i]);
    }
    const double ca[3] = {0.0, tc.c[2], tc.c[1]}, cb[3] = {0.0, tc.ct[2], tc.ct[1]};
    state_terms<VALUES>(s0, kappa, hK, g1, 1.0, s0.U, nm, io.Wt, io.Wt2, ca, cb, We, F, Wet, Ft, Wt0);
  }
  // non-equilibrium initial parts of both sides
  {
    const double ca[3] = {tc.c[3], -tau * tc.c[3], tc.c[4]}, cb[3] = {tc.ct[3], -tau * tc.ct[3], tc.ct[4]};
    state_terms<VALUES>(sL, kappa, hK, g1, mL, sL.U * mL + xL, io.nL, io.Wt, io.Wt2, ca, cb, We, F, Wet, Ft, WtL);
    state_terms<VALUES>(sR, kappa, hK, g1, mR, sR.U * mR + xR, io.nR, io.Wt, io.Wt2, ca, cb, We, F, Wet, Ft, WtR);
  }
  F[0] = We[1];
  Ft[0] = Wet[1];
  // Prandtl-number correction: (1/Pr - 1) times the heat flux
  // 1/2 <(u-U0)((u-U0)^2 + (v-V0)^2 + (w-W0)^2 + xi^2)>, written with the
  // moments of psi (We) and u psi (F) of the same distribution.
  if (k.mu > 0) {
    const double U = s0.U, V = s0.V, Wv = s0.Wv, f = k.prfix;
    const double q2 = U * U + V * V + Wv * Wv;
    const double a = U * U + 0.5 * q2, b = 0.5 * U * q2, UV = U * V, UW = U * Wv;
    if (VALUES)
      F[4] = F[4] + f * (F[4] - U * F[1] - V * F[2] - Wv * F[3] + a * F[0] - U * We[4] + UV * We[2] + UW * We[3] -
                         b * We[0]);
    Ft[4] = Ft[4] + f * (Ft[4] - U * Ft[1] - V * Ft[2] - Wv * Ft[3] + a * Ft[0] - U * Wet[4] + UV * Wet[2] +
                         UW * Wet[3] - b * Wet[0]);
  }
  const double e = tc.e1, oe = 1.0 - tc.e1;
#pragma unroll
  for (int i = 0; i < 5; ++i) {
    io.Ft[i] = Ft[i];
    io.Wlt[i] = oe * Wet[i] + e * WtL[i];
    io.Wrt[i] = oe * Wet[i] + e * WtR[i];
    if (VALUES) {
      io.F[i] = F[i];
      io.Wl[i] = oe * We[i] + e * io.WL[i];
      io.Wr[i] = oe * We[i] + e * io.WR[i];
    }
  }
}

// Smooth nodal solver: f^n = g [1 - tauN ((a.psi) u + (b.psi) v + (c.psi) w
// + A.psi)], f_t = (A.psi) g, in closed form: Euler fluxes, their time
// derivatives from the Euler equations, and the Navier-Stokes stress and heat
// flux of the BGK model (with the Prandtl correction).  F[a], Ft[a]: flux along
// axis a (x, y, z) and its time derivative.  VALUES = false: F skipped.
template <bool VALUES>
FDK_HD void gks_node(const Consts& k, const double* W, const double* Wx, const double* Wy, const double* Wz,
                     double F[3][5], double Ft[3][5]) {
  const double g1 = k.gamma - 1.0, hK = 0.5 * (k.K + 3.0), h1 = hK + 1.0;
  const Prim s = prim(W, k.gamma);
  const PSlope a = prim_slope(s, g1, Wx), b = prim_slope(s, g1, Wy), c = prim_slope(s, g1, Wz);
  const PSlope t = euler_slope(s, g1, a, b, c);
  double Wt[5];
  cons_t(s, hK, t, Wt);
  const bool visc = k.mu > 0;
  const double f = k.prfix;
  const double pt = s.rho * t.th + s.i2l * Wt[0];
  const double H = W[4] + s.p, Ht = Wt[4] + pt;
  const double u[3] = {s.U, s.V, s.Wv}, ut[3] = {t.u, t.v, t.w};
#pragma unroll
  for (int ax = 0; ax < 3; ++ax) {
    Ft[ax][0] = Wt[1 + ax];
#pragma unroll
    for (int m = 0; m < 3; ++m) {
      // (rho u_ax u_m)_t, formed the same way for both of (ax, m) and (m, ax)
      const int lo = ax < m ? ax : m, hi = ax < m ? m : ax;
      const double x = u[hi] * Wt[1 + lo] + W[1 + lo] * ut[hi];
      Ft[ax][1 + m] = ax == m ? pt + x : x;
    }
    Ft[ax][4] = u[ax] * Ht + ut[ax] * H;
    if (visc) Ft[ax][4] = Ft[ax][4] + f * (h1 * s.p * ut[ax]);
  }
  if (VALUES) {
    const double tp = k.mu, kap = tp * h1 * (1.0 + f), div = g1 * (a.u + b.v + c.w);
    const double sd[3] = {tp * (2.0 * a.u - div), tp * (2.0 * b.v - div), tp * (2.0 * c.w - div)};
    const double sxy = tp * (b.u + a.v), sxz = tp * (c.u + a.w), syz = tp * (c.v + b.w);
    const double S[3][3] = {{sd[0], sxy, sxz}, {sxy, sd[1], syz}, {sxz, syz, sd[2]}};
    const double q[3] = {a.th, b.th, c.th};
#pragma unroll
    for (int ax = 0; ax < 3; ++ax) {
      F[ax][0] = W[1 + ax];
#pragma unroll
      for (int m = 0; m < 3; ++m) {
        const int lo = ax < m ? ax : m, hi = ax < m ? m : ax;
        const double x = u[hi] * W[1 + lo];
        F[ax][1 + m] = ax == m ? s.p + x : x;
        if (visc) F[ax][1 + m] = F[ax][1 + m] - S[ax][m];
      }
      F[ax][4] = u[ax] * H;
      if (visc) F[ax][4] = F[ax][4] - (u[0] * S[ax][0] + u[1] * S[ax][1] + u[2] * S[ax][2] + kap * q[ax]);
    }
  }
}

}  // namespace fdk3
