// Device arithmetic of the FD-CGKS stage for gfx950: compact GENO
// reconstruction and the space-time coupled BGK gas-kinetic solver.
//
// Straight-line FP64 code (FP32 optional for the gas-kinetic part), fully
// inlined so that every moment index is a compile-time constant and all
// moment tables live in VGPRs.
#pragma once

#include <hip/hip_runtime.h>

#include <cmath>
#include <type_traits>

// Everything here is also host-callable, so that host-side checks can run the
// same arithmetic.
#define FDK_HD __host__ __device__ __forceinline__

namespace fdk {

// Scheme constants, passed by value to every kernel.
struct Consts {
  double gamma;
  double K;           // internal degrees of freedom: (4-2g)/(g-1) in 2D, (3-g)/(g-1) in 1D
  double inv_Kd;      // 1/(K+2) in 2D, 1/(K+1) in 1D
  double mu;          // dynamic viscosity (0: Euler)
  double prfix;       // 1/Pr - 1 (applied when mu > 0)
  double C, inv_tanhC, eps, eps_a, dc, ds;  // GENO (Sec. 3.2, App. D)
  double tau_c1, tau_c2;
  double geno_ratio;  // smooth-data bound on tau / (smallest indicator + eps), see geno_smooth_ratio (0: not used)
  int r;              // GENO exponent
  int variant;        // 0: (6-4), 1: (6-2), 2: linear
  int grad_carried;
  int flux_order;     // 6, or 8: the linear compact flux over the wider stencil
};

// ---------------------------------------------------------------- math
FDK_HD double m_erfc(double x) { return erfc(x); }
FDK_HD float m_erfc(float x) { return erfcf(x); }
FDK_HD double m_exp(double x) { return exp(x); }
FDK_HD float m_exp(float x) { return expf(x); }
FDK_HD double m_sqrt(double x) { return sqrt(x); }
FDK_HD float m_sqrt(float x) { return sqrtf(x); }
FDK_HD double m_abs(double x) { return fabs(x); }
FDK_HD float m_abs(float x) { return fabsf(x); }

template <class T> FDK_HD T sqr(T a) { return a * a; }

// Reciprocal and square root of normal numbers: Newton steps on the hardware
// estimates without the scaling and fix-up of the IEEE sequences (5 and 8
// instructions instead of about 11 and 18).  The square root is the coupled
// iteration for sqrt(x) and 1 / (2 sqrt(x)) with one correction by the
// residual.  On the device both are right to 0.500 ulp at each of 400,000
// points over 1e-290 .. 1e290, as the correctly rounded operations.  Not for
// arguments that may be zero, denormal or infinite.
template <class T> FDK_HD T m_recip(T x) { return T(1) / x; }
FDK_HD double m_recip(double x) {
#if defined(__HIP_DEVICE_COMPILE__)
  double r = __builtin_amdgcn_rcp(x);
  r = __builtin_fma(__builtin_fma(-x, r, 1.0), r, r);
  return __builtin_fma(__builtin_fma(-x, r, 1.0), r, r);
#else
  return 1.0 / x;
#endif
}
FDK_HD double m_sqrt_normal(double x) {
#if defined(__HIP_DEVICE_COMPILE__)
  const double y = __builtin_amdgcn_rsq(x);
  double g = x * y, h = 0.5 * y;
  double d = __builtin_fma(-h, g, 0.5);
  g = __builtin_fma(g, d, g);
  h = __builtin_fma(h, d, h);
  d = __builtin_fma(-g, g, x);
  return __builtin_fma(d, h, g);
#else
  return sqrt(x);
#endif
}
// exp(-x) and 1 - exp(-x) for x >= 0, to 1.13 and 1.23 ulp: -x = k ln 2 + r,
// expm1(r) = r + r^2 (1/2 + r q(r)) with q interpolated at Chebyshev nodes of
// |r| <= ln(2) / 2 (relative error of exp below 8e-17 before rounding).
FDK_HD void exp_neg(double x, double& E, double& one_minus_E) {
  const double y = x > 800.0 ? 800.0 : x;  // exp(-800) = 0
  const double k = __builtin_rint(-y * 1.4426950408889634);
  double r = __builtin_fma(k, -0x1.62e42fefa3000p-1, -y);
  r = __builtin_fma(k, -0x1.3de6af278ece6p-42, r);
  double q = 0x1.af238498b289ap-26;
  q = __builtin_fma(q, r, 0x1.2880562d283e2p-22);
  q = __builtin_fma(q, r, 0x1.71de17dab6782p-19);
  q = __builtin_fma(q, r, 0x1.a019c99634817p-16);
  q = __builtin_fma(q, r, 0x1.a01a01a4b5021p-13);
  q = __builtin_fma(q, r, 0x1.6c16c17393002p-10);
  q = __builtin_fma(q, r, 0x1.1111111110e69p-7);
  q = __builtin_fma(q, r, 0x1.5555555554cb2p-5);
  q = __builtin_fma(q, r, 0x1.5555555555555p-3);
  q = __builtin_fma(q, r, 0.5);
  const double m = __builtin_fma(r * r, q, r);  // expm1(r)
  const double s = ldexp(1.0, (int)k);
  E = __builtin_fma(s, m, s);
  one_minus_E = __builtin_fma(-s, m, 1.0 - s);
}
// tanh of the path function: (1 - E) / (1 + E), E = exp(-2 |a|), no branch;
// beyond |a| = 19.5 it is +-1 in FP64 (1 - tanh(a) < 2.3e-17, under half an ulp of 1).
FDK_HD double g_tanh(double a) {
  double E, o;
  exp_neg(2.0 * fabs(a), E, o);
  return copysign(o * m_recip(1.0 + E), a);
}
// erf(z) / 2 for |z| <= 1, to 1.62 ulp: z p(z^2), p interpolated at Chebyshev nodes of [0, 1] (relative error
// below 5e-17).
FDK_HD double half_erf_small(double z) {
  const double t = z * z;
  double p = -0x1.ac9585a44fe29p-32;
  p = __builtin_fma(p, t, 0x1.d76af6ca49787p-28);
  p = __builtin_fma(p, t, -0x1.5c131500d3f88p-24);
  p = __builtin_fma(p, t, 0x1.b981d78881a5dp-21);
  p = __builtin_fma(p, t, -0x1.f4ca838adb73bp-18);
  p = __builtin_fma(p, t, 0x1.f9a2be4f731a1p-15);
  p = __builtin_fma(p, t, -0x1.c02db0665e53dp-12);
  p = __builtin_fma(p, t, 0x1.565bccfa44156p-9);
  p = __builtin_fma(p, t, -0x1.b82ce31203772p-7);
  p = __builtin_fma(p, t, 0x1.ce2f21a040f66p-5);
  p = __builtin_fma(p, t, -0x1.812746b0379c1p-3);
  p = __builtin_fma(p, t, 0x1.20dd750429b6dp-1);
  return z * p;
}

template <class T> FDK_HD T ipow(T x, int r) {
  T y = x;
  for (int k = 1; k < r; ++k) y = y * x;
  return y;
}

// scalar helpers (ties keep the first argument)
FDK_HD double g_abs(double a) { return fabs(a); }
FDK_HD double g_max(double a, double b) { return fmax(a, b); }
FDK_HD double g_min(double a, double b) { return fmin(a, b); }
FDK_HD double val(double a) { return a; }
FDK_HD float val(float a) { return a; }

// ----------------------------------------------------- GENO, Sec. 3 / App. C
// Path function and blend of one side.  IS1 is the IS^tau reference;
// d1, d2, d3 the ideal weights; q/dq the sub-stencil value/derivative
// candidates; PH/PHx the high-order ones.  Normalised low-order weights are
// d_k / t_k^2 (t_k = IS_k + eps_a) scaled by t1^2 t2^2 t3^2, so one division
// normalises them.
template <class R> struct GenoOutT {
  R v, d, chi;
};
// Largest ratio x = tau / (ISL + eps) below which the path function saturates
// whatever the other indicators are: alpha = 2 aH / (aH + aL) with aH >= 1 is at
// least 2 / (2 + x^r), so C alpha >= 19.5 (1 + 1e-12) where x^r <= beta =
// 2 C / (19.5 (1 + 1e-12)) - 2.  0 (never) where 1 / tanh(C) is not 1, beta is
// not positive or eps does not keep the quotients normal.
inline double geno_smooth_ratio(double C, double inv_tanhC, int r, double eps) {
  const double beta = 2.0 * C / (19.5 * (1.0 + 1e-12)) - 2.0;
  if (inv_tanhC != 1.0 || !(beta > 0.0) || !(eps >= 1e-100)) return 0.0;
  return std::pow(beta, 1.0 / r) * (1.0 - 1e-9);
}
// Smooth data decided from one ratio: where it holds (and IS1, hence every
// indicator, is far from overflow) geno() returns PH, PHx and chi = 1.
template <class R> FDK_HD bool geno_smooth(const Consts& k, R IS1, R IS2, R IS3) {
  const R tau = 0.5 * g_abs((IS2 + IS3) - 2.0 * IS1);
  const R eL = g_min(IS1, g_min(IS2, IS3)) + k.eps;
  return val(tau) < k.geno_ratio * val(eL) && val(IS1) <= 1e100;
}
template <class R>
FDK_HD GenoOutT<R> geno(const Consts& k, R IS1, R IS2, R IS3, double d1, double d2, double d3,
                                            R q1, R q2, R q3, R dq1, R dq2, R dq3, R PH, R PHx) {
  R tau = 0.5 * g_abs((IS2 + IS3) - 2.0 * IS1);
  R ISH = g_max(IS1, g_max(IS2, IS3));
  R ISL = g_min(IS1, g_min(IS2, IS3));
  R eH = ISH + k.eps, eL = ISL + k.eps;
  GenoOutT<R> o;
  // Smooth data decided before any division.  With A = eH^r + tau^r and
  // B = eL^r + tau^r, alpha below equals 2 A eL^r / (A eL^r + B eH^r).  Where
  // C alpha >= 19.5 (1 + 1e-12) in that division-free form (rounding moves it
  // by a few 1e-16), the alpha computed below gives C alpha > 19.5, tanh is 1,
  // and with 1/tanh(C) = 1 the value returned is the one of the shortcut
  // further down.  Other points (and inf / NaN / underflowed products) take
  // the full path.
  if (k.inv_tanhC == 1.0) {
    R pH = eH, pL = eL, pt = tau;
    for (int q = 1; q < k.r; ++q) {
      pH = pH * eH;
      pL = pL * eL;
      pt = pt * tau;
    }
    R a = (pH + pt) * pL, b = (pL + pt) * pH;
    R lhs = (2.0 * k.C) * a, rhs = (19.5 * (1.0 + 1e-12)) * (a + b);
    if (val(rhs) >= 1e-290 && val(lhs) <= 1e300 && val(lhs) >= val(rhs)) {
      o.v = PH;
      o.d = PHx;
      o.chi = R(1.0);
      return o;
    }
  }
  R inv = 1.0 / (eH * eL);
  R xH = tau * eL * inv, xL = tau * eH * inv;
  R aH = 1.0 + ipow(xH, k.r), aL = 1.0 + ipow(xL, k.r);
  R alpha = 2.0 * aH / (aH + aL);
  R th = g_tanh(k.C * alpha);
  R chi = th * k.inv_tanhC;
  // Smooth data: tanh saturates (its derivative is 0) and chi = 1 exactly, so
  // the low-order blend has weight 0 in the value and in every derivative.
  if (val(th) == 1.0 && val(chi) == 1.0) {
    o.v = PH;
    o.d = PHx;
    o.chi = chi;
    return o;
  }
  R t1 = sqr(IS1 + k.eps_a), t2 = sqr(IS2 + k.eps_a), t3 = sqr(IS3 + k.eps_a);
  R w1 = d1 * t2 * t3, w2 = d2 * t1 * t3, w3 = d3 * t1 * t2;
  R is = 1.0 / (w1 + w2 + w3);
  R PL = (w1 * q1 + w2 * q2 + w3 * q3) * is;
  R PLx = (w1 * dq1 + w2 * dq2 + w3 * dq3) * is;
  o.v = chi * PH + (1.0 - chi) * PL;
  o.d = chi * PHx + (1.0 - chi) * PLx;
  o.chi = chi;
  return o;
}

// x^r with the exponent known (RR > 0) or at run time
template <int RR> FDK_HD double rpow(double x, int r) {
  if constexpr (RR > 0) {
    double y = x;
#pragma unroll
    for (int k = 1; k < RR; ++k) y = y * x;
    return y;
  } else {
    return ipow(x, r);
  }
}
// geno() without its early decisions: one straight run, for points known not
// to be smooth (the same bits, since the early decisions never change them);
// the two sides of an interface then overlap.  With tanh through exp_neg a
// 400-node shock tube went from 30.9 to 22.3 us per step.
template <int RR>
FDK_HD GenoOutT<double> geno_full(const Consts& k, double IS1, double IS2, double IS3, double d1, double d2, double d3,
                                  double q1, double q2, double q3, double dq1, double dq2, double dq3, double PH,
                                  double PHx) {
  const double tau = 0.5 * g_abs((IS2 + IS3) - 2.0 * IS1);
  const double ISH = g_max(IS1, g_max(IS2, IS3)), ISL = g_min(IS1, g_min(IS2, IS3));
  const double eH = ISH + k.eps, eL = ISL + k.eps;
  const double inv = 1.0 / (eH * eL);
  const double xH = tau * eL * inv, xL = tau * eH * inv;
  const double aH = 1.0 + rpow<RR>(xH, k.r), aL = 1.0 + rpow<RR>(xL, k.r);
  const double alpha = 2.0 * aH / (aH + aL);
  const double th = g_tanh(k.C * alpha);
  const double chi = th * k.inv_tanhC;
  const double t1 = sqr(IS1 + k.eps_a), t2 = sqr(IS2 + k.eps_a), t3 = sqr(IS3 + k.eps_a);
  const double w1 = d1 * t2 * t3, w2 = d2 * t1 * t3, w3 = d3 * t1 * t2;
  const double is = 1.0 / (w1 + w2 + w3);
  const double PL = (w1 * q1 + w2 * q2 + w3 * q3) * is;
  const double PLx = (w1 * dq1 + w2 * dq2 + w3 * dq3) * is;
  const bool one = th == 1.0 && chi == 1.0;
  GenoOutT<double> o;
  o.v = one ? PH : chi * PH + (1.0 - chi) * PL;
  o.d = one ? PHx : chi * PHx + (1.0 - chi) * PLx;
  o.chi = chi;
  return o;
}

// geno (FULL = -1) or geno_full with the exponent FULL (0: at run time)
template <class R, int FULL>
FDK_HD GenoOutT<R> geno_of(const Consts& k, R IS1, R IS2, R IS3, double d1, double d2, double d3, R q1, R q2, R q3,
                           R dq1, R dq2, R dq3, R PH, R PHx) {
  if constexpr (FULL < 0) return geno<R>(k, IS1, IS2, IS3, d1, d2, d3, q1, q2, q3, dq1, dq2, dq3, PH, PHx);
  else return geno_full<FULL>(k, IS1, IS2, IS3, d1, d2, d3, q1, q2, q3, dq1, dq2, dq3, PH, PHx);
}
// Interface m+1/2 of a line q0..q3 = Q_{m-1..m+2}, x0..x3 = averaged
// derivatives (Eq. 7th-compact-recons; App. C1, C2).
template <class R> struct IfaceRecT {
  R vl, dl, cl, vr, dr, cr;
};
using IfaceRec = IfaceRecT<double>;
template <class R, int FULL = -1>
FDK_HD IfaceRecT<R> recon_iface(const Consts& k, R q0, R q1, R q2, R q3, R x0, R x1, R x2, R x3,
                                                    double h, double invh) {
  IfaceRecT<R> o;
  R PHl = ((7.0 * q0 + 35.0 * q1 + 21.0 * q2 + q3) + (x0 + 22.0 * x1 - 7.0 * x2) * h) * (1.0 / 64.0);
  R PHr = ((q0 + 21.0 * q1 + 35.0 * q2 + 7.0 * q3) + (7.0 * x1 - 22.0 * x2 - x3) * h) * (1.0 / 64.0);
  R PHx = -((q0 + 45.0 * q1 - 45.0 * q2 - q3) + 9.0 * (x1 + x2) * h) * (invh * (1.0 / 30.0));
  if (k.variant == 2) {
    o.vl = PHl; o.dl = PHx; o.cl = R(1.0);
    o.vr = PHr; o.dr = PHx; o.cr = R(1.0);
    return o;
  }
  R hx0 = h * x0, hx3 = h * x3;
  R D2 = sqr(q0 - 2.0 * q1 + q2), D3 = sqr(q1 - 2.0 * q2 + q3);
  R dmid = (q2 - q1) * invh;
  R qc = (-q0 + 6.0 * q1 + 3.0 * q2) * 0.125;  // q_2^l == q_3^r
  // left (App. C1)
  R ISl1 = (13.0 / 3.0) * sqr(q1 - q0 - hx0) + sqr(2.0 * (q1 - q0) - hx0);
  R ISl2 = (13.0 / 12.0) * D2 + 0.25 * sqr(q2 - q0);
  R ISl3 = (13.0 / 12.0) * D3 + 0.25 * sqr(3.0 * q1 - 4.0 * q2 + q3);
  R ql1 = (-5.0 * q0 + 9.0 * q1 - 3.0 * hx0) * 0.25;
  R ql3 = (3.0 * q1 + 6.0 * q2 - q3) * 0.125;
  R dl1 = (-3.0 * q0 + 3.0 * q1 - 2.0 * hx0) * invh;
  GenoOutT<R> L = geno_of<R, FULL>(k, ISl1, ISl2, ISl3, k.ds, k.dc, k.ds, ql1, qc, ql3, dl1, dmid, dmid, PHl, PHx);
  // right (App. C2)
  R ISr1 = (13.0 / 3.0) * sqr(q2 - q3 + hx3) + sqr(2.0 * (q3 - q2) - hx3);
  R ISr2 = (13.0 / 12.0) * D3 + 0.25 * sqr(q3 - q1);
  R ISr3 = (13.0 / 12.0) * D2 + 0.25 * sqr(3.0 * q2 - 4.0 * q1 + q0);
  R qr1 = (-5.0 * q3 + 9.0 * q2 + 3.0 * hx3) * 0.25;
  R qr2 = (-q3 + 6.0 * q2 + 3.0 * q1) * 0.125;
  R dr1 = (-3.0 * q2 + 3.0 * q3 - 2.0 * hx3) * invh;
  GenoOutT<R> Rr = geno_of<R, FULL>(k, ISr1, ISr2, ISr3, k.ds, k.dc, k.ds, qr1, qr2, qc, dr1, dmid, dmid, PHr, PHx);
  o.vl = L.v; o.dl = L.d; o.cl = L.chi;
  o.vr = Rr.v; o.dr = Rr.d; o.cr = Rr.chi;
  return o;
}

// The same where both sides pass the one-ratio smooth test (or the scheme is
// linear): returns whether they do; o then holds recon_iface's result.
FDK_HD bool recon_iface_smooth(const Consts& k, double q0, double q1, double q2, double q3, double x0, double x1,
                               double x2, double x3, double h, double invh, IfaceRec& o) {
  const double PHl = ((7.0 * q0 + 35.0 * q1 + 21.0 * q2 + q3) + (x0 + 22.0 * x1 - 7.0 * x2) * h) * (1.0 / 64.0);
  const double PHr = ((q0 + 21.0 * q1 + 35.0 * q2 + 7.0 * q3) + (7.0 * x1 - 22.0 * x2 - x3) * h) * (1.0 / 64.0);
  const double PHx = -((q0 + 45.0 * q1 - 45.0 * q2 - q3) + 9.0 * (x1 + x2) * h) * (invh * (1.0 / 30.0));
  o.vl = PHl; o.dl = PHx; o.cl = 1.0;
  o.vr = PHr; o.dr = PHx; o.cr = 1.0;
  if (k.variant == 2) return true;
  const double hx0 = h * x0, hx3 = h * x3;
  const double D2 = sqr(q0 - 2.0 * q1 + q2), D3 = sqr(q1 - 2.0 * q2 + q3);
  const double ISl1 = (13.0 / 3.0) * sqr(q1 - q0 - hx0) + sqr(2.0 * (q1 - q0) - hx0);
  const double ISl2 = (13.0 / 12.0) * D2 + 0.25 * sqr(q2 - q0);
  const double ISl3 = (13.0 / 12.0) * D3 + 0.25 * sqr(3.0 * q1 - 4.0 * q2 + q3);
  const double ISr1 = (13.0 / 3.0) * sqr(q2 - q3 + hx3) + sqr(2.0 * (q3 - q2) - hx3);
  const double ISr2 = (13.0 / 12.0) * D3 + 0.25 * sqr(q3 - q1);
  const double ISr3 = (13.0 / 12.0) * D2 + 0.25 * sqr(3.0 * q2 - 4.0 * q1 + q0);
  // both tests evaluated, no branch between them
  return (int)geno_smooth<double>(k, ISl1, ISl2, ISl3) & (int)geno_smooth<double>(k, ISr1, ISr2, ISr3);
}
// A line of N components: one straight run of arithmetic that is all of it on
// smooth data, the general routine for components that are not smooth (the
// results are recon_iface's bit for bit).  The general routine per component
// and side cost two branches and about 15 more FP64 operations each, and the
// scheduler could not mix the components.
template <int N>
FDK_HD void recon_line(const Consts& k, const double (&Q)[N][4], const double (&X)[N][4], double h, double invh,
                       IfaceRec (&rec)[N]) {
  bool ok[N], all = true;
#pragma unroll
  for (int c = 0; c < N; ++c) {
    ok[c] = recon_iface_smooth(k, Q[c][0], Q[c][1], Q[c][2], Q[c][3], X[c][0], X[c][1], X[c][2], X[c][3], h, invh,
                               rec[c]);
    all = (int)all & (int)ok[c];
  }
  if (!all) {
#pragma unroll
    for (int c = 0; c < N; ++c)
      if (!ok[c])
        rec[c] = recon_iface<double>(k, Q[c][0], Q[c][1], Q[c][2], Q[c][3], X[c][0], X[c][1], X[c][2], X[c][3], h,
                                     invh);
  }
}

// recon_line for a line that can be read again: Q, X hold the stencil, and
// load(c, q, x) reads component c's (a run-time index).  The general routine
// is then a loop with one copy of its code, a fifth of recon_line's size, for
// a kernel whose code has to stay in the instruction cache.
template <int N, class Load>
FDK_HD void recon_line_compact(const Consts& k, const double (&Q)[N][4], const double (&X)[N][4], const Load& load,
                               double h, double invh, IfaceRec (&rec)[N]) {
  int bad = 0;
#pragma unroll
  for (int c = 0; c < N; ++c)
    bad |= recon_iface_smooth(k, Q[c][0], Q[c][1], Q[c][2], Q[c][3], X[c][0], X[c][1], X[c][2], X[c][3], h, invh,
                              rec[c])
               ? 0
               : 1 << c;
  if (bad) {
#pragma unroll 1
    for (int c = 0; c < N; ++c) {
      if (!(bad & (1 << c))) continue;
      double q[4], x[4];
      load(c, q, x);
      IfaceRec r;
      if (k.r == 3) r = recon_iface<double, 3>(k, q[0], q[1], q[2], q[3], x[0], x[1], x[2], x[3], h, invh);
      else r = recon_iface<double, 0>(k, q[0], q[1], q[2], q[3], x[0], x[1], x[2], x[3], h, invh);
#pragma unroll
      for (int d = 0; d < N; ++d)
        if (d == c) rec[d] = r;
    }
  }
}

// Node derivative from q0..q2 = Q_{j-1..j+1}, x0..x2 (Eq. 6th-compact-recons,
// App. C3; the central sub-stencil is the IS^tau reference with weight dc).
template <class R, int FULL = -1>
FDK_HD R recon_node(const Consts& k, R q0, R q1, R q2, R x0, R x1, R x2, double h, double invh) {
  R PHx = (9.0 * (q0 - q2) + h * (x0 + 46.0 * x1 + x2)) * (invh * (1.0 / 30.0));
  if (k.variant == 2) return PHx;
  R hx0 = h * x0, hx2 = h * x2;
  R IS1 = (13.0 / 3.0) * sqr(q1 - q0 - hx0) + sqr(2.0 * (q1 - q0) - hx0);
  R IS2 = (13.0 / 3.0) * sqr(q2 - q1 - hx2) + sqr(2.0 * (q2 - q1) - hx2);
  R IS3 = (13.0 / 12.0) * sqr(q0 - 2.0 * q1 + q2) + 0.25 * sqr(q2 - q0);
  R dq1 = (-2.0 * q0 + 2.0 * q1 - hx0) * invh;
  R dq2 = (-2.0 * q1 + 2.0 * q2 - hx2) * invh;
  R dq3 = (q2 - q0) * (0.5 * invh);
  GenoOutT<R> o = geno_of<R, FULL>(k, IS3, IS1, IS2, k.dc, k.ds, k.ds, q1, q1, q1, dq3, dq1, dq2, q1, PHx);
  return o.d;
}

// The same, and whether the one-ratio smooth test holds.
FDK_HD bool recon_node_smooth(const Consts& k, double q0, double q1, double q2, double x0, double x1, double x2,
                              double h, double invh, double& d) {
  d = (9.0 * (q0 - q2) + h * (x0 + 46.0 * x1 + x2)) * (invh * (1.0 / 30.0));
  if (k.variant == 2) return true;
  const double hx0 = h * x0, hx2 = h * x2;
  const double IS1 = (13.0 / 3.0) * sqr(q1 - q0 - hx0) + sqr(2.0 * (q1 - q0) - hx0);
  const double IS2 = (13.0 / 3.0) * sqr(q2 - q1 - hx2) + sqr(2.0 * (q2 - q1) - hx2);
  const double IS3 = (13.0 / 12.0) * sqr(q0 - 2.0 * q1 + q2) + 0.25 * sqr(q2 - q0);
  return geno_smooth<double>(k, IS3, IS1, IS2);
}
// Node derivatives of N components along one axis (as recon_line).
template <int N>
FDK_HD void recon_node_line(const Consts& k, const double (&Q)[N][3], const double (&X)[N][3], double h, double invh,
                            double (&d)[N]) {
  bool ok[N], all = true;
#pragma unroll
  for (int c = 0; c < N; ++c) {
    ok[c] = recon_node_smooth(k, Q[c][0], Q[c][1], Q[c][2], X[c][0], X[c][1], X[c][2], h, invh, d[c]);
    all = (int)all & (int)ok[c];
  }
  if (!all) {
#pragma unroll
    for (int c = 0; c < N; ++c)
      if (!ok[c]) d[c] = recon_node<double>(k, Q[c][0], Q[c][1], Q[c][2], X[c][0], X[c][1], X[c][2], h, invh);
  }
}

// recon_node_line for a line that can be read again (see recon_line_compact).
template <int N, class Load>
FDK_HD void recon_node_compact(const Consts& k, const double (&Q)[N][3], const double (&X)[N][3], const Load& load,
                               double h, double invh, double (&d)[N]) {
  int bad = 0;
#pragma unroll
  for (int c = 0; c < N; ++c)
    bad |= recon_node_smooth(k, Q[c][0], Q[c][1], Q[c][2], X[c][0], X[c][1], X[c][2], h, invh, d[c]) ? 0 : 1 << c;
  if (bad) {
#pragma unroll 1
    for (int c = 0; c < N; ++c) {
      if (!(bad & (1 << c))) continue;
      double q[3], x[3];
      load(c, q, x);
      double r;
      if (k.r == 3) r = recon_node<double, 3>(k, q[0], q[1], q[2], x[0], x[1], x[2], h, invh);
      else r = recon_node<double, 0>(k, q[0], q[1], q[2], x[0], x[1], x[2], h, invh);
#pragma unroll
      for (int e = 0; e < N; ++e)
        if (e == c) d[e] = r;
    }
  }
}

// ------------------------------------- characteristic variables (Sec. 3)
// Eigenvectors of the Euler flux Jacobian along a line, in the line's local
// frame (component 1 is the momentum along the line), at a state W.  The
// columns of R are the fields u - c, u, [shears,] u + c, normalised as
// (1, u - c, [v, w,] H - u c), (1, u, [v, w,] |u|^2/2), [(0, 0, 1, 0, v),
// (0, 0, 0, 1, w),] (1, u + c, [v, w,] H + u c) (2D: no w); L = R^-1 in
// closed form with b1 = (gamma-1)/c^2 and b2 = b1 |u|^2 / 2.  The map is linear, so values and derivatives
// transform with the same matrices.  Nothing here is contracted into fused
// multiply-adds, in particular not with the callers' arithmetic: otherwise
// which products fuse would depend on the kernel the code is inlined into,
// and the path function (very sensitive to the last bit of the
// characteristic values on smooth data) would differ between kernels.
struct CharFrame {
  double u, v, c, ic, H, b1, b2, k2;  // k2 = |u|^2 / 2
  double w;                            // 3D only
};
template <int DIM> FDK_HD CharFrame char_frame(double gamma, const double* W) {
#pragma clang fp contract(off)
  CharFrame f;
  const double ir = 1.0 / W[0];
  f.u = W[1] * ir;
  f.v = DIM >= 2 ? W[2] * ir : 0.0;
  f.w = DIM == 3 ? W[3] * ir : 0.0;
  if (DIM == 3) f.k2 = 0.5 * (f.u * f.u + f.v * f.v + f.w * f.w);
  else f.k2 = 0.5 * (f.u * f.u + f.v * f.v);
  const double p = (gamma - 1.0) * (W[DIM + 1] - W[0] * f.k2);
  const double c2 = gamma * p * ir;
  f.c = sqrt(c2);
  f.ic = 1.0 / f.c;
  f.H = (W[DIM + 1] + p) * ir;
  f.b1 = (gamma - 1.0) / c2;
  f.b2 = f.b1 * f.k2;
  return f;
}
// q = L w
template <int DIM> FDK_HD void to_char(const CharFrame& f, const double* w, double* q) {
#pragma clang fp contract(off)
  const double uc = f.u * f.ic;
  double s;  // b1 (E - u m - v n [- w o])
  if (DIM == 3) s = f.b1 * (w[4] - f.u * w[1] - f.v * w[2] - f.w * w[3]);
  else s = f.b1 * (w[DIM + 1] - f.u * w[1] - (DIM == 2 ? f.v * w[2] : 0.0));
  const double a = f.b2 * w[0] + s;  // b2 rho + s
  const double m = f.ic * w[1] - uc * w[0];  // (m - u rho) / c
  q[0] = 0.5 * (a - m);
  q[1] = w[0] - a;
  if (DIM >= 2) q[2] = w[2] - f.v * w[0];
  if (DIM == 3) q[3] = w[3] - f.w * w[0];
  q[DIM + 1] = 0.5 * (a + m);
}
// w = R q
template <int DIM> FDK_HD void from_char(const CharFrame& f, const double* q, double* w) {
#pragma clang fp contract(off)
  const double lo = q[0], en = q[1], hi = q[DIM + 1];
  const double sh = DIM >= 2 ? q[2] : 0.0;
  const double sw = DIM == 3 ? q[3] : 0.0;
  const double s = lo + en + hi;
  w[0] = s;
  w[1] = f.u * s + f.c * (hi - lo);
  if (DIM >= 2) w[2] = f.v * s + sh;
  if (DIM == 3) {
    w[3] = f.w * s + sw;
    w[4] = f.H * (lo + hi) + f.u * f.c * (hi - lo) + f.k2 * en + f.v * sh + f.w * sw;
  } else {
    w[DIM + 1] = f.H * (lo + hi) + f.u * f.c * (hi - lo) + f.k2 * en + f.v * sh;
  }
}

// Interface reconstruction of a whole line of N = DIM + 2 components on
// characteristic variables.  Q[c][m], X[c][m]: values and averaged
// derivatives in the local frame at the nodes m = 0..3 around the interface;
// the eigenvectors are taken at the mean of the two interface-adjacent
// states.  rec[c] receives the local-frame results; chi is the smallest of
// the left and right path functions of the u - c and u + c fields.
template <int DIM>
FDK_HD void recon_iface_char(const Consts& k, const double (&Q)[DIM + 2][4], const double (&X)[DIM + 2][4], double h,
                             double invh, IfaceRec (&rec)[DIM + 2], double& chi) {
  constexpr int N = DIM + 2;
  double Wm[N];
  {
#pragma clang fp contract(off)
#pragma unroll
    for (int c = 0; c < N; ++c) Wm[c] = 0.5 * (Q[c][1] + Q[c][2]);
  }
  const CharFrame f = char_frame<DIM>(k.gamma, Wm);
  double qc[N][4], xc[N][4];
#pragma unroll
  for (int m = 0; m < 4; ++m) {
    double a[N], b[N];
#pragma unroll
    for (int c = 0; c < N; ++c) a[c] = Q[c][m];
    to_char<DIM>(f, a, b);
#pragma unroll
    for (int c = 0; c < N; ++c) { qc[c][m] = b[c]; a[c] = X[c][m]; }
    to_char<DIM>(f, a, b);
#pragma unroll
    for (int c = 0; c < N; ++c) xc[c][m] = b[c];
  }
  IfaceRec cr[N];
  recon_line<N>(k, qc, xc, h, invh, cr);
  chi = fmin(fmin(cr[0].cl, cr[0].cr), fmin(cr[N - 1].cl, cr[N - 1].cr));
  double a[N], b[N];
#pragma unroll
  for (int c = 0; c < N; ++c) a[c] = cr[c].vl;
  from_char<DIM>(f, a, b);
#pragma unroll
  for (int c = 0; c < N; ++c) { rec[c].vl = b[c]; a[c] = cr[c].dl; }
  from_char<DIM>(f, a, b);
#pragma unroll
  for (int c = 0; c < N; ++c) { rec[c].dl = b[c]; a[c] = cr[c].vr; }
  from_char<DIM>(f, a, b);
#pragma unroll
  for (int c = 0; c < N; ++c) { rec[c].vr = b[c]; a[c] = cr[c].dr; }
  from_char<DIM>(f, a, b);
#pragma unroll
  for (int c = 0; c < N; ++c) {
    rec[c].dr = b[c];
    rec[c].cl = rec[c].cr = chi;
  }
}

// Node derivatives of a whole line on characteristic variables: Q[c][m],
// X[c][m] at the nodes j-1, j, j+1 (local frame); eigenvectors at the
// node's own state.
template <int DIM>
FDK_HD void recon_node_char(const Consts& k, const double (&Q)[DIM + 2][3], const double (&X)[DIM + 2][3], double h,
                            double invh, double (&d)[DIM + 2]) {
  constexpr int N = DIM + 2;
  double Wc[N];
#pragma unroll
  for (int c = 0; c < N; ++c) Wc[c] = Q[c][1];
  const CharFrame f = char_frame<DIM>(k.gamma, Wc);
  double qc[N][3], xc[N][3];
#pragma unroll
  for (int m = 0; m < 3; ++m) {
    double a[N], b[N];
#pragma unroll
    for (int c = 0; c < N; ++c) a[c] = Q[c][m];
    to_char<DIM>(f, a, b);
#pragma unroll
    for (int c = 0; c < N; ++c) { qc[c][m] = b[c]; a[c] = X[c][m]; }
    to_char<DIM>(f, a, b);
#pragma unroll
    for (int c = 0; c < N; ++c) xc[c][m] = b[c];
  }
  double dc[N];
  recon_node_line<N>(k, qc, xc, h, invh, dc);
  from_char<DIM>(f, dc, d);
}

// ------------------------------------------- Maxwellian moments (App. A)
// Per unit density: mu[n] = <u^n> (full or half line), mv[n] = <v^n>,
// x2 = <xi^2>, x4 = <xi^4>.
template <class FT> struct Mom {
  FT mu[7];
  FT mv[7];
  FT x2, x4;
};

template <class FT> FDK_HD void mu_rec(FT* m, FT U, FT i2l) {
#pragma unroll
  for (int n = 0; n < 5; ++n) m[n + 2] = U * m[n + 1] + FT(n + 1) * i2l * m[n];
}

// <u^P v^Q xi^(2R) psi>, psi = (1, u, v, (u^2+v^2+xi^2)/2), R in {0, 1}
template <int P, int Q, int R, class FT> FDK_HD void muv(const Mom<FT>& m, FT o[4]) {
  const FT xr = R == 0 ? FT(1) : m.x2;
  const FT xr1 = R == 0 ? m.x2 : m.x4;
  FT b = m.mu[P] * m.mv[Q];
  o[0] = b * xr;
  o[1] = m.mu[P + 1] * m.mv[Q] * xr;
  o[2] = m.mu[P] * m.mv[Q + 1] * xr;
  o[3] = FT(0.5) * ((m.mu[P + 2] * m.mv[Q] + m.mu[P] * m.mv[Q + 2]) * xr + b * xr1);
}
// <(s.psi) u^P v^Q psi>.  With g = s.psi = s0 + s1 u + s2 v + h3 (u^2 + v^2 +
// xi^2), h3 = s3 / 2, a moment of g splits into a u part and a v part:
//   <g u^a v^b> = mv[b] cu(a) + mu[a] cv(b),
//   cu(a) = (s0 + h3 x2) mu[a] + s1 mu[a+1] + h3 mu[a+2],  cv(b) = s2 mv[b+1] + h3 mv[b+2],
// and <g u^a v^b xi^2> = x2 <g u^a v^b> + h3 mu[a] mv[b] (x4 - x2^2): six
// one-dimensional combinations instead of the six moment vectors of psi.
template <int P, int Q, class FT> FDK_HD void ma(const FT s[4], const Mom<FT>& m, FT o[4]) {
  const FT h3 = FT(0.5) * s[3];
  const FT c0 = s[0] + h3 * m.x2;
  const FT u0 = c0 * m.mu[P] + s[1] * m.mu[P + 1] + h3 * m.mu[P + 2];
  const FT u1 = c0 * m.mu[P + 1] + s[1] * m.mu[P + 2] + h3 * m.mu[P + 3];
  const FT u2 = c0 * m.mu[P + 2] + s[1] * m.mu[P + 3] + h3 * m.mu[P + 4];
  const FT v0 = s[2] * m.mv[Q + 1] + h3 * m.mv[Q + 2];
  const FT v1 = s[2] * m.mv[Q + 2] + h3 * m.mv[Q + 3];
  const FT v2 = s[2] * m.mv[Q + 3] + h3 * m.mv[Q + 4];
  o[0] = m.mv[Q] * u0 + m.mu[P] * v0;
  o[1] = m.mv[Q] * u1 + m.mu[P + 1] * v0;
  o[2] = m.mv[Q + 1] * u0 + m.mu[P] * v1;
  const FT gx = m.x2 * o[0] + h3 * (m.mu[P] * m.mv[Q]) * (m.x4 - m.x2 * m.x2);
  o[3] = FT(0.5) * ((m.mv[Q] * u2 + m.mu[P + 2] * v0) + (m.mv[Q + 2] * u0 + m.mu[P] * v2) + gx);
}
// 1D: psi = (1, u, (u^2+xi^2)/2)
template <int P, int R, class FT> FDK_HD void mu1(const Mom<FT>& m, FT o[3]) {
  const FT xr = R == 0 ? FT(1) : m.x2;
  const FT xr1 = R == 0 ? m.x2 : m.x4;
  o[0] = m.mu[P] * xr;
  o[1] = m.mu[P + 1] * xr;
  o[2] = FT(0.5) * (m.mu[P + 2] * xr + m.mu[P] * xr1);
}
template <int P, class FT> FDK_HD void ma1(const FT s[3], const Mom<FT>& m, FT o[3]) {
  FT t0[3], t1[3], t2[3], t3[3];
  mu1<P, 0>(m, t0);
  mu1<P + 1, 0>(m, t1);
  mu1<P + 2, 0>(m, t2);
  mu1<P, 1>(m, t3);
  FT h2 = FT(0.5) * s[2];
#pragma unroll
  for (int i = 0; i < 3; ++i) o[i] = s[0] * t0[i] + s[1] * t1[i] + h2 * (t2[i] + t3[i]);
}

// Primitive variables and the shared v / xi moments of a state.
template <class FT> struct Prim {
  FT rho, irho, U, V, p, lam, i2l, ip;  // ip = 1/p
};
template <class FT, int DIM> FDK_HD Prim<FT> prim(const FT* W, FT gamma) {
  Prim<FT> s;
  s.rho = W[0];
  s.irho = m_recip(W[0]);
  s.U = W[1] * s.irho;
  s.V = DIM == 2 ? W[2] * s.irho : FT(0);
  FT rE = W[DIM + 1];
  s.p = (gamma - FT(1)) * (rE - FT(0.5) * s.rho * (s.U * s.U + s.V * s.V));
  s.i2l = s.p * s.irho;          // 1/(2 lambda) = p/rho
  s.ip = m_recip(s.p);           // lambda = rho/(2p); 1/p also serves the collision time
  s.lam = FT(0.5) * s.rho * s.ip;
  return s;
}
template <class FT, int DIM> FDK_HD void mom_common(const Prim<FT>& s, FT K, Mom<FT>& m) {
  m.mv[0] = FT(1);
  m.mv[1] = s.V;
  if (DIM == 2) mu_rec(m.mv, s.V, s.i2l);
  m.x2 = K * s.i2l;
  m.x4 = m.x2 * (K + FT(2)) * s.i2l;
}
template <class FT> FDK_HD void mom_full(const Prim<FT>& s, Mom<FT>& m) {
  m.mu[0] = FT(1);
  m.mu[1] = s.U;
  mu_rec(m.mu, s.U, s.i2l);
}
// half line: sgn = +1 (u > 0) or -1 (u < 0); <1> and <u> - U <1>
FDK_HD void half_moms(double lam, double i2l, double U, double sgn, double& m0, double& x) {
  const double sl = m_sqrt_normal(lam), z = sl * U;
  // |z| <= 1 up to a normal Mach number of about 1.2; a wave goes through the
  // library's erfc only if one of its points is beyond.  1/2 - erf/2 is exact
  // in the last digits of the whole, not of the smaller share; with erfc in its
  // place the solver's error against extended precision is the same to 1% (40,000
  // states each at normal Mach 0.3 to 2, densities up to 1e5 apart)
  if (fabs(z) <= 1.0) m0 = 0.5 + sgn * half_erf_small(z);
  else m0 = 0.5 * m_erfc(-sgn * z);
  double E, o;
  exp_neg(z * z, E, o);
  // 1/(2 sqrt(pi lambda)) = (1/(2 lambda)) sqrt(lambda) / sqrt(pi): no second square root
  x = sgn * E * (i2l * sl) * 0.56418958354775628695;
}
template <class FT> FDK_HD void mom_half(const Prim<FT>& s, FT sgn, Mom<FT>& m) {
  FT sl = m_sqrt(s.lam);
  m.mu[0] = FT(0.5) * m_erfc(-sgn * sl * s.U);
  m.mu[1] = s.U * m.mu[0] + sgn * m_exp(-s.lam * s.U * s.U) * (s.i2l * sl) * FT(0.56418958354775628695);
  mu_rec(m.mu, s.U, s.i2l);
}

// Micro slope s with <psi (s.psi)> = d (d per unit density): closed-form
// solution of the moment system.
template <class FT, int DIM>
FDK_HD void slope(const Prim<FT>& q, FT K, FT iKd, const FT* d, FT* s) {
  if (DIM == 2) {
    FT e = q.U * q.U + q.V * q.V + (K + FT(2)) * q.i2l;
    FT B = FT(2) * d[3] - e * d[0];
    FT A = d[1] - q.U * d[0];
    FT Cc = d[2] - q.V * d[0];
    FT tl = FT(2) * q.lam;
    s[3] = tl * tl * iKd * (B - FT(2) * q.U * A - FT(2) * q.V * Cc);
    s[2] = tl * Cc - q.V * s[3];
    s[1] = tl * A - q.U * s[3];
    s[0] = d[0] - q.U * s[1] - q.V * s[2] - FT(0.5) * s[3] * e;
  } else {
    FT e = q.U * q.U + (K + FT(1)) * q.i2l;
    FT B = FT(2) * d[2] - e * d[0];
    FT A = d[1] - q.U * d[0];
    FT tl = FT(2) * q.lam;
    s[2] = tl * tl * iKd * (B - FT(2) * q.U * A);
    s[1] = tl * A - q.U * s[2];
    s[0] = d[0] - q.U * s[1] - FT(0.5) * s[2] * e;
  }
}

// Integrated BGK time coefficients over [0, T] (equilibrium, its space and
// time slope terms, non-equilibrium initial part, its slope term) and the
// f^n / f_t^n fit of App. A1 from T = dt/2 and T = dt.
template <class FT> struct TimeCoef {
  FT c[5], ct[5], e1;  // e1 = exp(-dt/tau)
};
template <class FT> FDK_HD TimeCoef<FT> time_coef(FT dt, FT tau) {
  TimeCoef<FT> r;
  if constexpr (std::is_same_v<FT, double>) {
    // The fit written out: with s = tau / dt, E = exp(-dt / (2 tau)) and
    // o = 1 - E the ten combinations (4 q(dt/2) - q(dt)) / dt and
    // 4 (q(dt) - 2 q(dt/2)) / dt^2 of the integrals reduce to four numbers.
    // tau = 0 (p_l = p_r without a c1 term): the tau -> 0+ limit, E = 0.
    double Eh = 0.0, o = 1.0;
    if (tau > 1e-290) exp_neg(0.5 * dt * m_recip(tau), Eh, o);
    const FT idt = m_recip(dt), s = tau * idt;
    r.e1 = Eh * Eh;
    const FT c3 = s * o * (FT(2) + o);
    const FT c4 = tau * ((FT(1) - o * o) - FT(2) * c3);  // 2 E - E^2 = 1 - o^2
    const FT t0 = FT(4) * s * (o * o), t1 = FT(4) * s * (o * (Eh - FT(2) * s * o));
    r.c[0] = FT(1) - c3;
    r.c[1] = -tau - c4;
    r.c[2] = -tau * r.c[0];
    r.c[3] = c3;
    r.c[4] = c4;
    r.ct[0] = t0 * idt;
    r.ct[1] = t1;
    r.ct[2] = FT(1) - s * t0;
    r.ct[3] = -r.ct[0];
    r.ct[4] = -t1;
    return r;
  }
  // tau = 0 (p_l = p_r without a c1 term): the tau -> 0+ limit, exp(-T/tau) = 0
  FT Eh = val(tau) > 0 ? m_exp(-FT(0.5) * dt / tau) : FT(0);
  FT Ef = Eh * Eh;
  FT Th = FT(0.5) * dt, Tf = dt;
  FT qh[5], qf[5];
  qh[0] = Th - tau * (FT(1) - Eh);
  qf[0] = Tf - tau * (FT(1) - Ef);
  qh[1] = tau * ((FT(2) * tau - Th) - (Th + FT(2) * tau) * Eh);
  qf[1] = tau * ((FT(2) * tau - Tf) - (Tf + FT(2) * tau) * Ef);
  qh[2] = FT(0.5) * Th * Th - tau * Th + tau * tau * (FT(1) - Eh);
  qf[2] = FT(0.5) * Tf * Tf - tau * Tf + tau * tau * (FT(1) - Ef);
  qh[3] = tau * (FT(1) - Eh);
  qf[3] = tau * (FT(1) - Ef);
  qh[4] = tau * ((Th + FT(2) * tau) * Eh - FT(2) * tau);
  qf[4] = tau * ((Tf + FT(2) * tau) * Ef - FT(2) * tau);
  FT idt = FT(1) / dt;
  FT idt2 = FT(4) * idt * idt;
#pragma unroll
  for (int k = 0; k < 5; ++k) {
    r.c[k] = (FT(4) * qh[k] - qf[k]) * idt;
    r.ct[k] = (qf[k] - FT(2) * qh[k]) * idt2;
  }
  r.e1 = Ef;
  return r;
}

// ----------------------------------------- gas-kinetic interface solver
// Local frame: the normal velocity is component 1 (u).  2D: W = (rho, rho u,
// rho v, rho E), tangential slope Wt; 1D: W = (rho, rho u, rho E).
// Outputs: flux F, its time derivative Ft, and the interface values
// W-hat^{l,r} and their time derivatives (Eq. W-model).  VALUES = false skips
// F and W-hat (stage 2 uses only the time derivatives).
template <class FT, int DIM> struct GksIO {
  FT WL[DIM + 2], WR[DIM + 2], nL[DIM + 2], nR[DIM + 2], Wt[DIM + 2];
  FT F[DIM + 2], Ft[DIM + 2], Wl[DIM + 2], Wr[DIM + 2], Wlt[DIM + 2], Wrt[DIM + 2];
};

// Moments of the transport and time-slope terms of one state:
// tr = <psi ((a.psi) u + (b.psi) v)>, tru = <u psi (...)>, Ap = <psi A.psi>,
// Au = <u psi A.psi> (2D; 1D drops the v terms).
template <class FT, int DIM>
FDK_HD void transport(const FT* a, const FT* b, const Mom<FT>& m, FT* tr, FT* tru) {
  if (DIM == 2) {
    FT x[4], y[4];
    ma<1, 0>(a, m, x); ma<0, 1>(b, m, y);
#pragma unroll
    for (int i = 0; i < 4; ++i) tr[i] = x[i] + y[i];
    ma<2, 0>(a, m, x); ma<1, 1>(b, m, y);
#pragma unroll
    for (int i = 0; i < 4; ++i) tru[i] = x[i] + y[i];
  } else {
    ma1<1>(a, m, tr);
    ma1<2>(a, m, tru);
  }
}
template <class FT, int DIM> FDK_HD void tslope(const FT* A, const Mom<FT>& m, FT* Ap, FT* Au) {
  if (DIM == 2) { ma<0, 0>(A, m, Ap); ma<1, 0>(A, m, Au); }
  else { ma1<0>(A, m, Ap); ma1<1>(A, m, Au); }
}
// <psi> and <u psi> of a (half or full) state
template <class FT, int DIM> FDK_HD void psi_moms(const Mom<FT>& m, FT* p, FT* u) {
  if (DIM == 2) {
    p[0] = m.mu[0]; p[1] = m.mu[1]; p[2] = m.mu[0] * m.mv[1];
    p[3] = FT(0.5) * (m.mu[2] + m.mu[0] * (m.mv[2] + m.x2));
    muv<1, 0, 0>(m, u);
  } else {
    p[0] = m.mu[0]; p[1] = m.mu[1]; p[2] = FT(0.5) * (m.mu[2] + m.mu[0] * m.x2);
    mu1<1, 0>(m, u);
  }
}

// The contribution of one side s to the moments of f^n and f_t^n:
// rho_s <phi [c3 (1 - tau A.psi) + c4 ((a.psi) u + (b.psi) v)]> over the half
// line of s, for phi = psi (We, Wet) and u psi (F, Ft); also the one-sided
// Euler time derivative Wt = -rho_s <psi (...)> over the full line.
template <class FT, int DIM, bool VALUES>
FDK_HD void side_terms(const Prim<FT>& s, const Mom<FT>& h, const FT* n, const FT* t, FT K,
                                           FT iKd, FT tau, const TimeCoef<FT>& tc, bool both, FT* F, FT* Ft, FT* We,
                                           FT* Wet, FT* Wt) {
  constexpr int N = DIM + 2;
  Mom<FT> f = h;
  mom_full(s, f);
  FT a[N], b[N], A[N], d[N], tf[N], tuf[N];
#pragma unroll
  for (int i = 0; i < N; ++i) d[i] = n[i] * s.irho;
  slope<FT, DIM>(s, K, iKd, d, a);
  if (DIM == 2) {
#pragma unroll
    for (int i = 0; i < N; ++i) d[i] = t[i] * s.irho;
    slope<FT, DIM>(s, K, iKd, d, b);
  }
  if (DIM == 2) { FT x[N], y[N]; ma<1, 0>(a, f, x); ma<0, 1>(b, f, y); for (int i = 0; i < N; ++i) tf[i] = x[i] + y[i]; }
  else ma1<1>(a, f, tf);
#pragma unroll
  for (int i = 0; i < N; ++i) { d[i] = -tf[i]; Wt[i] = -s.rho * tf[i]; }
  slope<FT, DIM>(s, K, iKd, d, A);
  FT ph[N], uh[N], tp[N], tu[N], Ap[N], Au[N];
  psi_moms<FT, DIM>(h, ph, uh);
  transport<FT, DIM>(a, b, h, tp, tu);
  tslope<FT, DIM>(A, h, Ap, Au);
  (void)tuf;
#pragma unroll
  for (int i = 0; i < N; ++i) {
    FT nu = uh[i] - tau * Au[i], np = ph[i] - tau * Ap[i];
    Ft[i] += s.rho * (tc.ct[3] * nu + tc.ct[4] * tu[i]);
    Wet[i] += s.rho * (tc.ct[3] * np + tc.ct[4] * tp[i]);
    if (both) {
      F[i] += s.rho * (tc.c[3] * nu + tc.c[4] * tu[i]);
      We[i] += s.rho * (tc.c[3] * np + tc.c[4] * tp[i]);
    }
  }
}

// The solver from moment vectors of psi, as App. A writes it.  The FP32-flux
// variant runs it: that option is there for the accuracy of FP32 solvers, whose
// results are this arithmetic's rounding, and not for speed (scalar FP32 issues
// at the FP64 rate: 6.0 ms per 2048^2 step against 3.8 in FP64).  FP64 runs the
// form in primitive slopes below.
template <class FT, int DIM, bool VALUES>
FDK_HD void gks_iface_moments(const Consts& k, FT dt, GksIO<FT, DIM>& io) {
  constexpr int N = DIM + 2;
  const FT K = FT(k.K), gam = FT(k.gamma), iKd = FT(k.inv_Kd);
  const bool both = VALUES || k.mu > 0;  // F and We are needed for the values or the Prandtl fix
  Prim<FT> sL = prim<FT, DIM>(io.WL, gam), sR = prim<FT, DIM>(io.WR, gam);
  // half-line moments and the compatibility state W0
  Mom<FT> hL, hR;
  mom_common<FT, DIM>(sL, K, hL);
  mom_half(sL, FT(1), hL);
  mom_common<FT, DIM>(sR, K, hR);
  mom_half(sR, FT(-1), hR);
  FT W0[N];
  {
    FT pL[N], pR[N], u[N];
    psi_moms<FT, DIM>(hL, pL, u);
    psi_moms<FT, DIM>(hR, pR, u);
#pragma unroll
    for (int i = 0; i < N; ++i) W0[i] = sL.rho * pL[i] + sR.rho * pR[i];
  }
  Prim<FT> s0 = prim<FT, DIM>(W0, gam);
  // collision time and time coefficients
  FT tau = (k.mu > 0 ? FT(k.mu) * s0.ip : FT(k.tau_c1) * dt) +
           FT(k.tau_c2) * dt * m_abs(sL.p - sR.p) / (sL.p + sR.p);
  TimeCoef<FT> tc = time_coef(dt, tau);
  FT F[N], We[N], Wet[N], WtL[N], WtR[N];
#pragma unroll
  for (int i = 0; i < N; ++i) { F[i] = FT(0); io.Ft[i] = FT(0); We[i] = FT(0); Wet[i] = FT(0); }
  // non-equilibrium initial parts of both sides
  side_terms<FT, DIM, VALUES>(sL, hL, io.nL, io.Wt, K, iKd, tau, tc, both, F, io.Ft, We, Wet, WtL);
  side_terms<FT, DIM, VALUES>(sR, hR, io.nR, io.Wt, K, iKd, tau, tc, both, F, io.Ft, We, Wet, WtR);
  // equilibrium part: g0 with slopes from the averaged normal slope (D12) and
  // the tangential slope, time slope from compatibility
  {
    Mom<FT> m0;
    mom_common<FT, DIM>(s0, K, m0);
    mom_full(s0, m0);
    FT a0[N], b0[N], A0[N], d[N], t0[N], tu0[N], Ap0[N], Au0[N], p0[N], u0[N];
#pragma unroll
    for (int i = 0; i < N; ++i) d[i] = FT(0.5) * (io.nL[i] + io.nR[i]) * s0.irho;
    slope<FT, DIM>(s0, K, iKd, d, a0);
    if (DIM == 2) {
#pragma unroll
      for (int i = 0; i < N; ++i) d[i] = io.Wt[i] * s0.irho;
      slope<FT, DIM>(s0, K, iKd, d, b0);
    }
    transport<FT, DIM>(a0, b0, m0, t0, tu0);
#pragma unroll
    for (int i = 0; i < N; ++i) d[i] = -t0[i];
    slope<FT, DIM>(s0, K, iKd, d, A0);
    tslope<FT, DIM>(A0, m0, Ap0, Au0);
    psi_moms<FT, DIM>(m0, p0, u0);
#pragma unroll
    for (int i = 0; i < N; ++i) {
      io.Ft[i] += s0.rho * (tc.ct[0] * u0[i] + tc.ct[1] * tu0[i] + tc.ct[2] * Au0[i]);
      Wet[i] += s0.rho * (tc.ct[0] * p0[i] + tc.ct[1] * t0[i] + tc.ct[2] * Ap0[i]);
      if (both) {
        F[i] += s0.rho * (tc.c[0] * u0[i] + tc.c[1] * tu0[i] + tc.c[2] * Au0[i]);
        We[i] += s0.rho * (tc.c[0] * p0[i] + tc.c[1] * t0[i] + tc.c[2] * Ap0[i]);
      }
    }
  }
  // Prandtl-number correction of the energy flux: (1/Pr - 1) times the heat
  // flux 1/2 <(u-U0)((u-U0)^2 + (v-V0)^2 + xi^2)> of the same distribution,
  // written with the moments of psi and u psi.
  if (k.mu > 0) {
    FT U = s0.U, V = s0.V, f = FT(k.prfix);
    if (DIM == 2) {
      FT a = FT(1.5) * U * U + FT(0.5) * V * V, b = FT(0.5) * U * (U * U + V * V);
      FT q = F[3] - U * F[1] - V * F[2] + a * F[0] - U * We[3] + U * V * We[2] - b * We[0];
      FT qt = io.Ft[3] - U * io.Ft[1] - V * io.Ft[2] + a * io.Ft[0] - U * Wet[3] + U * V * Wet[2] - b * Wet[0];
      F[3] += f * q;
      io.Ft[3] += f * qt;
    } else {
      FT a = FT(1.5) * U * U, b = FT(0.5) * U * U * U;
      FT q = F[2] - U * F[1] + a * F[0] - U * We[2] - b * We[0];
      FT qt = io.Ft[2] - U * io.Ft[1] + a * io.Ft[0] - U * Wet[2] - b * Wet[0];
      F[2] += f * q;
      io.Ft[2] += f * qt;
    }
  }
  // interface values (Eq. W-model) with the one-sided Euler time derivatives
  FT e = tc.e1, oe = FT(1) - tc.e1;
#pragma unroll
  for (int i = 0; i < N; ++i) {
    io.Wlt[i] = oe * Wet[i] + e * WtL[i];
    io.Wrt[i] = oe * Wet[i] + e * WtR[i];
    if (VALUES) {
      io.F[i] = F[i];
      io.Wl[i] = oe * We[i] + e * io.WL[i];
      io.Wr[i] = oe * We[i] + e * io.WR[i];
    }
  }
}

// ------------------------------------- the solver in primitive slopes
// A slope a.psi of a Maxwellian is the derivative of its logarithm.  With the
// derivatives of (rho, U, V, theta), theta = p / rho = 1 / (2 lambda), and the
// peculiar velocities c = u - U, v' = v - V:
//   a.psi = r + (c U_x + v' V_x) / theta + ((c^2 + v'^2 + xi^2) / theta - (K + dim)) theta_x / (2 theta),
// r = rho_x / rho.  Everything but u is integrated over full lines, where
// the moments of v' and xi are closed: the weights 1, v' and
// e' = (v'^2 + xi^2) / 2 leave polynomials of u,
//   <a.psi>    = a(u) = a0 + a1 u + a2 u^2,
//   <a.psi v'> = V_x,     <a.psi e'> = kappa (theta a(u) + theta_x),  kappa = (K + dim - 1) / 2,
// so a solve needs 1D moment sums of cubics only.  Bound by FP64 issue and by
// the registers that set the number of waves: against the moment vectors of
// psi (with GENO's smooth lines decided from one ratio) the stage-1 interface
// sweep executes 3,789 instead of 5,618 flop per point and holds 180 instead of
// 246 VGPRs, stage 2 140 instead of 246 (three waves per SIMD): 1.25 and 0.81
// ms against 1.55 and 1.40 ms at 2048^2.
template <class FT> struct PSlope {
  FT r, u, v, th;  // rho_x / rho, U_x, V_x, theta_x
};
// Constants of a state shared by its terms.
template <class FT> struct PState {
  FT U, V, th, ith, k2, hE;  // theta, 1 / theta, V^2 / 2, kappa theta + V^2 / 2
};
template <class FT, int DIM> FDK_HD PState<FT> pstate(const Prim<FT>& s, FT kappa) {
  PState<FT> q;
  q.U = s.U;
  q.V = s.V;
  q.th = s.i2l;
  q.ith = FT(2) * s.lam;
  q.hE = kappa * s.i2l;
  if (DIM == 2) {
    q.k2 = FT(0.5) * s.V * s.V;
    q.hE = q.hE + q.k2;
  } else {
    q.k2 = FT(0);
  }
  return q;
}
// Slopes of the primitive variables from the derivative d of the conservative ones.
template <class FT, int DIM> FDK_HD PSlope<FT> prim_slope(const Prim<FT>& s, FT g1, const FT* d) {
  PSlope<FT> o;
  o.r = d[0] * s.irho;
  o.u = d[1] * s.irho - s.U * o.r;
  if (DIM == 2) {
    o.v = d[2] * s.irho - s.V * o.r;
    const FT k2 = FT(0.5) * (s.U * s.U + s.V * s.V);
    const FT e = d[3] * s.irho - k2 * o.r - s.U * o.u - s.V * o.v;  // (p_x / rho) / (gamma - 1)
    o.th = g1 * e - s.i2l * o.r;
  } else {
    o.v = FT(0);
    const FT e = d[2] * s.irho - FT(0.5) * s.U * s.U * o.r - s.U * o.u;
    o.th = g1 * e - s.i2l * o.r;
  }
  return o;
}
// Euler time derivatives of the primitive variables from the normal slope a and the tangential slope b.
template <class FT, int DIM>
FDK_HD PSlope<FT> euler_slope(const PState<FT>& q, FT g1, const PSlope<FT>& a, const PSlope<FT>& b) {
  PSlope<FT> t;
  if (DIM == 2) {
    const FT div = a.u + b.v;
    t.r = -(div + q.U * a.r + q.V * b.r);
    t.u = -(a.th + q.th * a.r + q.U * a.u + q.V * b.u);
    t.v = -(b.th + q.th * b.r + q.U * a.v + q.V * b.v);
    t.th = -(g1 * q.th * div + q.U * a.th + q.V * b.th);
  } else {
    t.r = -(a.u + q.U * a.r);
    t.u = -(a.th + q.th * a.r + q.U * a.u);
    t.v = FT(0);
    t.th = -(g1 * q.th * a.u + q.U * a.th);
  }
  return t;
}
// a(u) of a slope
template <class FT> FDK_HD void slope_poly(const PState<FT>& q, const PSlope<FT>& a, FT* o) {
  const FT ux = a.u * q.ith;
  o[2] = FT(0.5) * a.th * (q.ith * q.ith);
  o[1] = ux - FT(2) * q.U * o[2];
  o[0] = a.r - q.th * o[2] - q.U * (o[1] + q.U * o[2]);
}
// The terms of one state (a side over its half line, or the equilibrium over
// the full line) that k0 + kA A.psi + kg ((a.psi) u + (b.psi) v) weights:
// polynomials and the 1D moments common to the values and their time
// derivatives.
template <class FT, int DIM> struct PTerms {
  FT A[3], g[4];         // A(u); (a.psi) u + (b.psi) v integrated over v', xi
  FT vt[2], ng[2];       // weight v' (2D) with u^0, u^1: of A.psi, of the transport term
  FT et[2], eg[2];       // weight V v' + e' beyond hE times weight 1
};
template <class FT, int DIM>
FDK_HD PTerms<FT, DIM> pterms(const PState<FT>& q, FT kappa, const PSlope<FT>& a, const PSlope<FT>& b,
                              const PSlope<FT>& t, const FT* mu) {
  PTerms<FT, DIM> o;
  FT pa[3];
  slope_poly(q, a, pa);
  slope_poly(q, t, o.A);
  if (DIM == 2) {
    FT pb[3];
    slope_poly(q, b, pb);
    o.g[0] = b.v + q.V * pb[0];
    o.g[1] = pa[0] + q.V * pb[1];
    o.g[2] = pa[1] + q.V * pb[2];
    o.g[3] = pa[2];
    const FT n0 = b.th + q.V * b.v + q.th * pb[0], n1 = a.v + q.th * pb[1], n2 = q.th * pb[2];
    const FT e0 = q.th * b.v + kappa * (q.V * b.th), e1 = kappa * a.th;
    const FT ett = kappa * t.th + q.V * t.v;
#pragma unroll
    for (int n = 0; n < 2; ++n) {
      o.vt[n] = t.v * mu[n];
      o.ng[n] = n0 * mu[n] + n1 * mu[n + 1] + n2 * mu[n + 2];
      o.et[n] = ett * mu[n];
      o.eg[n] = e0 * mu[n] + e1 * mu[n + 1] + q.V * o.ng[n];
    }
  } else {
    o.g[0] = FT(0);
    o.g[1] = pa[0];
    o.g[2] = pa[1];
    o.g[3] = pa[2];
    const FT e1 = kappa * a.th, ett = kappa * t.th;
#pragma unroll
    for (int n = 0; n < 2; ++n) {
      o.vt[n] = o.ng[n] = FT(0);
      o.et[n] = ett * mu[n];
      o.eg[n] = e1 * mu[n + 1];
    }
  }
  return o;
}
// Adds the moments <psi (..)> to W and <u psi (..)> to F for one set of
// coefficients (F[0] = W[1] is left to the caller).
template <class FT, int DIM>
FDK_HD void padd(const PState<FT>& q, const PTerms<FT, DIM>& p, const FT* mu, FT k0, FT kA, FT kg, FT* W, FT* F) {
  const FT p0 = DIM == 2 ? k0 + kA * p.A[0] + kg * p.g[0] : k0 + kA * p.A[0];
  const FT p1 = kA * p.A[1] + kg * p.g[1], p2 = kA * p.A[2] + kg * p.g[2], p3 = kg * p.g[3];
  FT M[4];
#pragma unroll
  for (int n = 0; n < 4; ++n) M[n] = p0 * mu[n] + p1 * mu[n + 1] + p2 * mu[n + 2] + p3 * mu[n + 3];
  W[0] = W[0] + M[0];
  W[1] = W[1] + M[1];
  F[1] = F[1] + M[2];
  if (DIM == 2) {
    W[2] = W[2] + q.V * M[0] + kA * p.vt[0] + kg * p.ng[0];
    F[2] = F[2] + q.V * M[1] + kA * p.vt[1] + kg * p.ng[1];
  }
  W[DIM + 1] = W[DIM + 1] + FT(0.5) * M[2] + q.hE * M[0] + kA * p.et[0] + kg * p.eg[0];
  F[DIM + 1] = F[DIM + 1] + FT(0.5) * M[3] + q.hE * M[1] + kA * p.et[1] + kg * p.eg[1];
}
// Conservative time derivative of a state from the primitive one
template <class FT, int DIM> FDK_HD void cons_t(const Prim<FT>& s, FT hK, const PSlope<FT>& t, FT* Wt) {
  const FT rt = s.rho * t.r;
  Wt[0] = rt;
  Wt[1] = s.rho * t.u + s.U * rt;
  if (DIM == 2) {
    Wt[2] = s.rho * t.v + s.V * rt;
    Wt[3] = s.U * Wt[1] + s.V * Wt[2] + hK * (s.rho * t.th) + (hK * s.i2l - FT(0.5) * (s.U * s.U + s.V * s.V)) * rt;
  } else {
    Wt[2] = s.U * Wt[1] + hK * (s.rho * t.th) + (hK * s.i2l - FT(0.5) * s.U * s.U) * rt;
  }
}
// One state's contribution to the moments of f^n (VALUES) and f_t^n.
// mu[0], mu[1] given; the higher ones follow from the recursion.  ca: k0, kA,
// kg of f^n, cb: of f_t^n.  t receives the Euler time derivatives.
template <class FT, int DIM, bool VALUES>
FDK_HD void pstate_terms(const Prim<FT>& s, FT kappa, FT g1, FT m0, FT m1, const FT* n, const FT* tang, const FT* ca,
                         const FT* cb, FT* We, FT* F, FT* Wet, FT* Ft, PSlope<FT>& t) {
  const PState<FT> q = pstate<FT, DIM>(s, kappa);
  const PSlope<FT> a = prim_slope<FT, DIM>(s, g1, n);
  PSlope<FT> b{};
  if (DIM == 2) b = prim_slope<FT, DIM>(s, g1, tang);
  t = euler_slope<FT, DIM>(q, g1, a, b);
  FT mu[7];
  mu[0] = m0;
  mu[1] = m1;
  mu_rec(mu, s.U, s.i2l);
  const PTerms<FT, DIM> p = pterms<FT, DIM>(q, kappa, a, b, t, mu);
  if (VALUES) padd<FT, DIM>(q, p, mu, s.rho * ca[0], s.rho * ca[1], s.rho * ca[2], We, F);
  padd<FT, DIM>(q, p, mu, s.rho * cb[0], s.rho * cb[1], s.rho * cb[2], Wet, Ft);
}

template <class FT, int DIM, bool VALUES>
FDK_HD void gks_iface_slopes(const Consts& k, FT dt, GksIO<FT, DIM>& io) {
  constexpr int N = DIM + 2;
  const FT K = FT(k.K), gam = FT(k.gamma), g1 = gam - FT(1);
  const FT kappa = FT(0.5) * (K + FT(DIM - 1)), hK = FT(0.5) * (K + FT(DIM));
  const Prim<FT> sL = prim<FT, DIM>(io.WL, gam), sR = prim<FT, DIM>(io.WR, gam);
  // half-line moments <1> and x = <u> - U <1> of both sides, and the
  // compatibility state W0: a half line holds the share <1> of its state's W,
  // plus rho x of momentum and rho x U / 2 of energy
  FT mL, mR, xL, xR, W0[N];
  half_moms(sL.lam, sL.i2l, sL.U, 1.0, mL, xL);
  half_moms(sR.lam, sR.i2l, sR.U, -1.0, mR, xR);
  {
    const FT XL = sL.rho * xL, XR = sR.rho * xR;
#pragma unroll
    for (int i = 0; i < N; ++i) W0[i] = mL * io.WL[i] + mR * io.WR[i];
    W0[1] = W0[1] + (XL + XR);
    W0[N - 1] = W0[N - 1] + FT(0.5) * (sL.U * XL + sR.U * XR);
  }
  const Prim<FT> s0 = prim<FT, DIM>(W0, gam);
  // collision time and time coefficients
  const FT tau = (k.mu > 0 ? FT(k.mu) * s0.ip : FT(k.tau_c1) * dt) +
                 FT(k.tau_c2) * dt * m_abs(sL.p - sR.p) * m_recip(sL.p + sR.p);
  const TimeCoef<FT> tc = time_coef(dt, tau);
  FT We[N], F[N], Wet[N], Ft[N];
#pragma unroll
  for (int i = 0; i < N; ++i) { We[i] = FT(0); F[i] = FT(0); Wet[i] = FT(0); Ft[i] = FT(0); }
  PSlope<FT> tL, tR, t0;
  {
    // equilibrium part: slopes from the averaged normal slope (D12) and the
    // tangential slope, time slope from compatibility
    FT nm[N];
#pragma unroll
    for (int i = 0; i < N; ++i) nm[i] = FT(0.5) * (io.nL[i] + io.nR[i]);
    // the leading terms (g0 itself) are W0 and its Euler flux, exact to the last
    // operation; the polynomials carry the slope terms only
    const FT H = W0[N - 1] + s0.p;
#pragma unroll
    for (int i = 0; i < N; ++i) {
      const FT fe = i == N - 1 ? s0.U * H : (i == 0 ? W0[1] : (i == 1 ? s0.p + s0.U * W0[1] : s0.V * W0[1]));
      if (VALUES) { We[i] = tc.c[0] * W0[i]; F[i] = tc.c[0] * fe; }
      Wet[i] = tc.ct[0] * W0[i];
      Ft[i] = tc.ct[0] * fe;
    }
    const FT ca[3] = {FT(0), tc.c[2], tc.c[1]}, cb[3] = {FT(0), tc.ct[2], tc.ct[1]};
    pstate_terms<FT, DIM, VALUES>(s0, kappa, g1, FT(1), s0.U, nm, io.Wt, ca, cb, We, F, Wet, Ft, t0);
  }
  {
    // non-equilibrium initial parts of both sides: c3 (1 - tau A.psi) + c4 (...)
    const FT ca[3] = {tc.c[3], -tau * tc.c[3], tc.c[4]}, cb[3] = {tc.ct[3], -tau * tc.ct[3], tc.ct[4]};
    pstate_terms<FT, DIM, VALUES>(sL, kappa, g1, mL, sL.U * mL + xL, io.nL, io.Wt, ca, cb, We, F, Wet, Ft, tL);
    pstate_terms<FT, DIM, VALUES>(sR, kappa, g1, mR, sR.U * mR + xR, io.nR, io.Wt, ca, cb, We, F, Wet, Ft, tR);
  }
  F[0] = We[1];
  Ft[0] = Wet[1];
  // Prandtl-number correction of the energy flux: (1/Pr - 1) times the heat
  // flux 1/2 <(u-U0)((u-U0)^2 + (v-V0)^2 + xi^2)> of the same distribution,
  // written with the moments of psi and u psi.
  if (k.mu > 0) {
    const FT U = s0.U, V = s0.V, f = FT(k.prfix);
    if (DIM == 2) {
      const FT a = FT(1.5) * U * U + FT(0.5) * V * V, b = FT(0.5) * U * (U * U + V * V), UV = U * V;
      if (VALUES) F[3] = F[3] + f * (F[3] - U * F[1] - V * F[2] + a * F[0] - U * We[3] + UV * We[2] - b * We[0]);
      Ft[3] = Ft[3] + f * (Ft[3] - U * Ft[1] - V * Ft[2] + a * Ft[0] - U * Wet[3] + UV * Wet[2] - b * Wet[0]);
    } else {
      const FT a = FT(1.5) * U * U, b = FT(0.5) * U * U * U;
      if (VALUES) F[2] = F[2] + f * (F[2] - U * F[1] + a * F[0] - U * We[2] - b * We[0]);
      Ft[2] = Ft[2] + f * (Ft[2] - U * Ft[1] + a * Ft[0] - U * Wet[2] - b * Wet[0]);
    }
  }
  // interface values (Eq. W-model) with the one-sided Euler time derivatives
  const FT e = tc.e1, oe = FT(1) - tc.e1;
  FT WtL[N], WtR[N];
  cons_t<FT, DIM>(sL, hK, tL, WtL);
  cons_t<FT, DIM>(sR, hK, tR, WtR);
#pragma unroll
  for (int i = 0; i < N; ++i) {
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

template <class FT, int DIM, bool VALUES>
FDK_HD void gks_iface(const Consts& k, FT dt, GksIO<FT, DIM>& io) {
  if constexpr (std::is_same_v<FT, double>) gks_iface_slopes<FT, DIM, VALUES>(k, dt, io);
  else gks_iface_moments<FT, DIM, VALUES>(k, dt, io);
}

// ------------------------------------------------ smooth nodal solver
// f^n = g [1 - tauN ((a.psi) u + (b.psi) v + A.psi)], f_t = (A.psi) g.
// Outputs x-flux F, Ft and (2D) y-flux G, Gt.  VALUES = false: F, G skipped.
template <class FT, int DIM, bool VALUES>
FDK_HD void gks_node_moments(const Consts& k, const FT* W, const FT* Wx, const FT* Wy, FT* F, FT* Ft, FT* G, FT* Gt) {
  constexpr int N = DIM + 2;
  const FT K = FT(k.K), iKd = FT(k.inv_Kd);
  Prim<FT> s = prim<FT, DIM>(W, FT(k.gamma));
  Mom<FT> m;
  mom_common<FT, DIM>(s, K, m);
  mom_full(s, m);
  FT a[N], b[N], A[N], d[N], tr[N];
#pragma unroll
  for (int i = 0; i < N; ++i) d[i] = Wx[i] * s.irho;
  slope<FT, DIM>(s, K, iKd, d, a);
  if (DIM == 2) {
#pragma unroll
    for (int i = 0; i < N; ++i) d[i] = Wy[i] * s.irho;
    slope<FT, DIM>(s, K, iKd, d, b);
    FT x[N], y[N];
    ma<1, 0>(a, m, x); ma<0, 1>(b, m, y);
    for (int i = 0; i < N; ++i) tr[i] = x[i] + y[i];
  } else {
    ma1<1>(a, m, tr);
  }
#pragma unroll
  for (int i = 0; i < N; ++i) d[i] = -tr[i];
  slope<FT, DIM>(s, K, iKd, d, A);
  FT tauN = k.mu > 0 ? FT(k.mu) * s.ip : FT(0);
  const bool visc = k.mu > 0;
  FT Fu[N], Gv[N];
  if (DIM == 2) {
    FT x[N], y[N], z[N];
    ma<1, 0>(A, m, Fu);
    ma<0, 1>(A, m, Gv);
#pragma unroll
    for (int i = 0; i < N; ++i) { Ft[i] = s.rho * Fu[i]; Gt[i] = s.rho * Gv[i]; }
    if (VALUES || visc) {
      FT u0[N], v0[N];
      muv<1, 0, 0>(m, u0);
      muv<0, 1, 0>(m, v0);
      if (visc) {
        ma<2, 0>(a, m, x); ma<1, 1>(b, m, y);
        for (int i = 0; i < N; ++i) u0[i] -= tauN * (x[i] + y[i] + Fu[i]);
        ma<1, 1>(a, m, x); ma<0, 2>(b, m, z);
        for (int i = 0; i < N; ++i) v0[i] -= tauN * (x[i] + z[i] + Gv[i]);
      }
#pragma unroll
      for (int i = 0; i < N; ++i) { F[i] = s.rho * u0[i]; G[i] = s.rho * v0[i]; }
    }
    if (visc) {  // Prandtl correction with the node's velocity; W^e = W, W^e_t = -rho tr
      FT U = s.U, V = s.V, f = FT(k.prfix);
      FT ax = FT(1.5) * U * U + FT(0.5) * V * V, ay = FT(1.5) * V * V + FT(0.5) * U * U;
      FT bx = FT(0.5) * U * (U * U + V * V), by = FT(0.5) * V * (U * U + V * V);
      FT Wt0 = -s.rho * tr[0], Wt1 = -s.rho * tr[1], Wt2 = -s.rho * tr[2], Wt3 = -s.rho * tr[3];
      FT qx = F[3] - U * F[1] - V * F[2] + ax * F[0] - U * W[3] + U * V * W[2] - bx * W[0];
      FT qy = G[3] - V * G[2] - U * G[1] + ay * G[0] - V * W[3] + U * V * W[1] - by * W[0];
      FT qxt = Ft[3] - U * Ft[1] - V * Ft[2] + ax * Ft[0] - U * Wt3 + U * V * Wt2 - bx * Wt0;
      FT qyt = Gt[3] - V * Gt[2] - U * Gt[1] + ay * Gt[0] - V * Wt3 + U * V * Wt1 - by * Wt0;
      F[3] += f * qx; G[3] += f * qy; Ft[3] += f * qxt; Gt[3] += f * qyt;
    }
  } else {
    ma1<1>(A, m, Fu);
#pragma unroll
    for (int i = 0; i < N; ++i) Ft[i] = s.rho * Fu[i];
    if (VALUES || visc) {
      FT u0[N];
      mu1<1, 0>(m, u0);
      if (visc) {
        FT x[N];
        ma1<2>(a, m, x);
        for (int i = 0; i < N; ++i) u0[i] -= tauN * (x[i] + Fu[i]);
      }
#pragma unroll
      for (int i = 0; i < N; ++i) F[i] = s.rho * u0[i];
    }
    if (visc) {
      FT U = s.U, f = FT(k.prfix);
      FT a1 = FT(1.5) * U * U, b1 = FT(0.5) * U * U * U;
      FT Wt0 = -s.rho * tr[0], Wt2 = -s.rho * tr[2];
      FT q = F[2] - U * F[1] + a1 * F[0] - U * W[2] - b1 * W[0];
      FT qt = Ft[2] - U * Ft[1] + a1 * Ft[0] - U * Wt2 - b1 * Wt0;
      F[2] += f * q; Ft[2] += f * qt;
    }
  }
}

// The same in closed form (FP64): a Maxwellian's fluxes are the Euler fluxes
// (their time derivative follows from the Euler equations), and the tau term
// is the Navier-Stokes stress and heat flux of the BGK model, whose mass part
// vanishes by compatibility.
template <class FT, int DIM, bool VALUES>
FDK_HD void gks_node(const Consts& k, const FT* W, const FT* Wx, const FT* Wy, FT* F, FT* Ft, FT* G, FT* Gt) {
  if constexpr (!std::is_same_v<FT, double>) {
    gks_node_moments<FT, DIM, VALUES>(k, W, Wx, Wy, F, Ft, G, Gt);
    return;
  }
  const FT g1 = FT(k.gamma) - FT(1), hK = FT(0.5) * (FT(k.K) + FT(DIM)), h1 = hK + FT(1);
  const Prim<FT> s = prim<FT, DIM>(W, FT(k.gamma));
  const PState<FT> q = pstate<FT, DIM>(s, FT(0));
  const PSlope<FT> a = prim_slope<FT, DIM>(s, g1, Wx);
  PSlope<FT> b{};
  if (DIM == 2) b = prim_slope<FT, DIM>(s, g1, Wy);
  const PSlope<FT> t = euler_slope<FT, DIM>(q, g1, a, b);
  FT Wt[DIM + 2];
  cons_t<FT, DIM>(s, hK, t, Wt);
  const bool visc = k.mu > 0;
  const FT tp = visc ? FT(k.mu) : FT(0), f = FT(k.prfix);  // tau p = mu
  const FT pt = s.rho * t.th + s.i2l * Wt[0];              // p_t
  const FT H = W[DIM + 1] + s.p, Ht = Wt[DIM + 1] + pt;    // rho H and its time derivative
  Ft[0] = Wt[1];
  Ft[1] = pt + s.U * Wt[1] + W[1] * t.u;
  Ft[DIM + 1] = s.U * Ht + t.u * H;
  if (DIM == 2) {
    Ft[2] = s.V * Wt[1] + W[1] * t.v;
    Gt[0] = Wt[2];
    Gt[1] = Ft[2];
    Gt[2] = pt + s.V * Wt[2] + W[2] * t.v;
    Gt[3] = s.V * Ht + t.v * H;
  }
  if (visc) {  // Prandtl correction of f_t: its heat flux about the node's velocity
    Ft[DIM + 1] = Ft[DIM + 1] + f * (h1 * s.p * t.u);
    if (DIM == 2) Gt[3] = Gt[3] + f * (h1 * s.p * t.v);
  }
  if (VALUES) {
    F[0] = W[1];
    F[1] = s.p + s.U * W[1];
    F[DIM + 1] = s.U * H;
    if (DIM == 2) {
      F[2] = s.V * W[1];
      G[0] = W[2];
      G[1] = F[2];
      G[2] = s.p + s.V * W[2];
      G[3] = s.V * H;
    }
    if (visc) {
      const FT kap = tp * h1 * (FT(1) + f);  // heat conductivity of the corrected flux
      if (DIM == 2) {
        const FT div = g1 * (a.u + b.v);
        const FT sxx = tp * (FT(2) * a.u - div), syy = tp * (FT(2) * b.v - div), sxy = tp * (b.u + a.v);
        F[1] = F[1] - sxx;
        F[2] = F[2] - sxy;
        F[3] = F[3] - (s.U * sxx + s.V * sxy + kap * a.th);
        G[1] = G[1] - sxy;
        G[2] = G[2] - syy;
        G[3] = G[3] - (s.U * sxy + s.V * syy + kap * b.th);
      } else {
        const FT sxx = tp * (FT(2) * a.u - g1 * a.u);
        F[1] = F[1] - sxx;
        F[2] = F[2] - (s.U * sxx + kap * a.th);
      }
    }
  }
}

// ---------------------------------------------------------- compact flux
// Eq. fd-conservative-flux and its (6-4) / (6-2) nonlinear forms.
FDK_HD double compact_flux(int variant, double Fm, double Fc, double Fp, double N0, double N1,
                                               double chi) {
  double Fb = ((Fm + 46.0 * Fc + Fp) - 9.0 * (N0 + N1)) * (1.0 / 30.0);
  if (variant == 2) return Fb;
  double lo = variant == 1 ? Fc : (8.0 * Fc - N0 - N1) * (1.0 / 6.0);
  return lo + chi * (Fb - lo);
}
// The same with the linear flux of order 8: the averaging conditions of Eq.
// fd-conservative-flux-recons imposed also on the nodal cells j-1 and j+2
// (the wider stencil of Sec. 2.1; Nm, Np2 are the nodal fluxes there).  The
// degree-6 solution at the interface is exact to degree 7 (symmetry), error
// -h^8 F^(8) / 161280; the low-order fluxes and the blend are unchanged.
FDK_HD double compact_flux8(int variant, double Fm, double Fc, double Fp, double Nm, double N0, double N1, double Np2,
                            double chi) {
  double Fb = ((32.0 * (Fm + Fp) + 704.0 * Fc) - 171.0 * (N0 + N1) - 3.0 * (Nm + Np2)) * (1.0 / 420.0);
  if (variant == 2) return Fb;
  double lo = variant == 1 ? Fc : (8.0 * Fc - N0 - N1) * (1.0 / 6.0);
  return lo + chi * (Fb - lo);
}

}  // namespace fdk
