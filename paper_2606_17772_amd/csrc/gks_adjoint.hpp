// Reverse-mode (adjoint) arithmetic of the 2D gas-kinetic interface and
// nodal solvers and of the GENO reconstructions, FP64.
//
// Every *_b routine takes the inputs of its forward counterpart in
// gks_device.hpp, recomputes the forward intermediates it needs, and, given
// the adjoint of the forward outputs, ADDS the adjoint of the forward inputs
// into the caller's accumulators (suffix b).  Non-smooth points follow the
// forward code: |x| has derivative 0 at 0, max/min route the adjoint to the
// argument the forward selected (ties: the first), tau = 0 takes the
// tau -> 0+ limit.
#pragma once

#include "gks_device.hpp"

namespace fdk {

// The reverse of the kinetic solvers below lets the compiler fuse any
// multiply and add into one FMA (about 11% fewer FP64 instructions in the
// reverse interface and node sweeps).  Its rounding then differs from the forward
// solver's in the last bits, which no result depends on: it makes no branch
// decision (those use the forward solver's own functions).  The GENO and
// reconstruction reverse further down compares smoothness indicators and keeps
// the forward code's contraction.
#pragma clang fp contract(fast)

// Adjoint of the fields of a Prim<double>.
struct PrimB {
  double rho, irho, U, V, p, i2l;
};
FDK_HD PrimB primb_zero() { return PrimB{0.0, 0.0, 0.0, 0.0, 0.0, 0.0}; }
// prim (2D): W -> (rho, irho, U, V, p, i2l).  Adds the adjoint of W.
FDK_HD void prim_b(const double* W, const Prim<double>& s, double gamma, const PrimB& b, double* Wb) {
  const double pb = b.p + b.i2l * s.irho;              // i2l = p irho
  double irhob = b.irho + b.i2l * s.p;
  const double gm = gamma - 1.0;                       // p = (g-1)(rE - rho (U^2+V^2)/2)
  const double rEb = gm * pb;
  const double rhob = b.rho - gm * 0.5 * (s.U * s.U + s.V * s.V) * pb;
  const double Ub = b.U - gm * s.rho * s.U * pb;
  const double Vb = b.V - gm * s.rho * s.V * pb;
  Wb[1] += Ub * s.irho;                                // U = W1 irho, V = W2 irho
  irhob += Ub * W[1];
  Wb[2] += Vb * s.irho;
  irhob += Vb * W[2];
  Wb[0] += rhob - irhob * s.irho * s.irho;             // irho = 1 / W0, rho = W0
  Wb[3] += rEb;
}

// m[n+2] = U m[n+1] + (n+1) i2l m[n], n = 0..4.  mb is consumed in place.
FDK_HD void mu_rec_b(const double* m, double U, double i2l, double* mb, double& Ub, double& i2lb) {
#pragma unroll
  for (int n = 4; n >= 0; --n) {
    const double g = mb[n + 2];
    mb[n + 1] += U * g;
    Ub += m[n + 1] * g;
    i2lb += double(n + 1) * m[n] * g;
    mb[n] += double(n + 1) * i2l * g;
  }
}

// A value the optimiser may not reuse from an earlier identical computation:
// cheap quantities are recomputed where they are needed instead of held in
// registers through the whole reverse sweep.
FDK_HD double fresh(double x) {
#if defined(__HIP_DEVICE_COMPILE__)
  asm volatile("" : "+v"(x));
#endif
  return x;
}
// A compiler-only memory barrier between the phases of the solver adjoint:
// values the caller keeps in memory (the LDS-resident inputs and output
// adjoints) are reloaded after it instead of being held in registers.
FDK_HD void phase_barrier() {
#if defined(__HIP_DEVICE_COMPILE__)
  asm volatile("" ::: "memory");
#endif
}
// A phase number the compiler cannot see through: the solver adjoint below
// runs its phases as iterations of one loop over it, so that no phase's code
// is peeled, merged or scheduled into another.
FDK_HD int opaque_int(int x) {
#if defined(__HIP_DEVICE_COMPILE__)
  asm volatile("" : "+s"(x));
#endif
  return x;
}

// ------------------------------- reverse of the solvers in primitive slopes
// The reverse follows the forward code's form (see gks_device.hpp): slopes of
// (rho, U, V, theta), polynomials of the normal velocity, one set of 1D
// moments per state.  theta = i2l; 1 / theta and lambda hand their adjoints to it.
typedef PSlope<double> Slope;

// o = prim_slope(s, d) has the adjoint ob: adds those of d (to db) and of s.
FDK_HD void prim_slope_b(const Prim<double>& s, double g1, const double* d, const Slope& o, const Slope& ob, double* db,
                         PrimB& sb) {
  const double k2 = 0.5 * (s.U * s.U + s.V * s.V), eb = g1 * ob.th;
  sb.i2l += -o.r * ob.th;
  sb.U += -(o.u + s.U * o.r) * eb;
  sb.V += -(o.v + s.V * o.r) * eb;
  const double ub = ob.u - s.U * eb, vb = ob.v - s.V * eb;
  sb.U += -o.r * ub;
  sb.V += -o.r * vb;
  const double rb = ob.r - s.i2l * ob.th - k2 * eb - s.U * ub - s.V * vb;
  sb.irho += d[3] * eb + d[2] * vb + d[1] * ub + d[0] * rb;
  db[3] += s.irho * eb;
  db[2] += s.irho * vb;
  db[1] += s.irho * ub;
  db[0] += s.irho * rb;
}
// t = euler_slope(a, b)
FDK_HD void euler_slope_b(const Prim<double>& s, double g1, const Slope& a, const Slope& b, const Slope& tb, Slope& ab,
                          Slope& bb, PrimB& sb) {
  const double U = s.U, V = s.V, th = s.i2l, divb = -tb.r - g1 * th * tb.th;
  ab.r += -U * tb.r - th * tb.u;
  ab.u += divb - U * tb.u;
  ab.v += -U * tb.v;
  ab.th += -tb.u - U * tb.th;
  bb.r += -V * tb.r - th * tb.v;
  bb.u += -V * tb.u;
  bb.v += divb - V * tb.v;
  bb.th += -tb.v - V * tb.th;
  sb.U += -(a.r * tb.r + a.u * tb.u + a.v * tb.v + a.th * tb.th);
  sb.V += -(b.r * tb.r + b.u * tb.u + b.v * tb.v + b.th * tb.th);
  sb.i2l += -(a.r * tb.u + b.r * tb.v + g1 * (a.u + b.v) * tb.th);
}
// o = slope_poly(a)
FDK_HD void slope_poly_b(const PState<double>& q, const Slope& a, const double* o, const double* ob, Slope& ab, PrimB& sb) {
  const double o1b = ob[1] - q.U * ob[0];
  const double o2b = ob[2] - (q.th + q.U * q.U) * ob[0] - 2.0 * q.U * o1b;
  ab.r += ob[0];
  ab.u += q.ith * o1b;
  ab.th += 0.5 * q.ith * q.ith * o2b;
  const double ithb = a.u * o1b + a.th * q.ith * o2b;
  sb.U += -(o[1] + 2.0 * q.U * o[2]) * ob[0] - 2.0 * o[2] * o1b;
  sb.i2l += -o[2] * ob[0] - q.ith * q.ith * ithb;
}
// Wt = cons_t(t); Wt: the forward values
FDK_HD void cons_t_b(const Prim<double>& s, double hK, const Slope& t, const double* Wt, const double* wb, Slope& tb,
                     PrimB& sb) {
  const double rt = Wt[0], c = hK * s.i2l - 0.5 * (s.U * s.U + s.V * s.V);
  const double w1 = wb[1] + s.U * wb[3], w2 = wb[2] + s.V * wb[3];
  const double rtb = wb[0] + c * wb[3] + s.U * w1 + s.V * w2;
  tb.r += s.rho * rtb;
  tb.u += s.rho * w1;
  tb.v += s.rho * w2;
  tb.th += hK * s.rho * wb[3];
  sb.rho += t.r * rtb + t.u * w1 + t.v * w2 + hK * t.th * wb[3];
  sb.U += (Wt[1] - s.U * rt) * wb[3] + rt * w1;
  sb.V += (Wt[2] - s.V * rt) * wb[3] + rt * w2;
  sb.i2l += hK * rt * wb[3];
}

// Half-line moments m0, x of a state (half_moms): the adjoints of U and
// theta.  d x / d z = -2 z x and d m0 / d z = 2 sqrt(lambda) x, z = sqrt(lambda) U.
FDK_HD void half_moms_b(const Prim<double>& s, double x, double m0b, double xb, PrimB& sb) {
  const double ith = 2.0 * s.lam, w = ith * x * (m0b - s.U * xb);
  sb.U += w;
  sb.i2l += 0.5 * ith * (x * xb - s.U * w);
}

// padd: the adjoints WB of W, FB of F (FB[0] is not used: F[0] = W[1]).  Adds
// to the adjoints of p, of the moments, of q's V and hE and of the coefficients
// (kb: k0, kA, kg); dW, dF receive what padd adds forward.
FDK_HD void padd_b(const PState<double>& q, const PTerms<double, 2>& p, const double* mu, double k0, double kA, double kg,
                   const double* WB, const double* FB, PTerms<double, 2>& pb, double* mub, double& Vb, double& hEb,
                   double* kb, double* dW, double* dF) {
  const double pc[4] = {k0 + kA * p.A[0] + kg * p.g[0], kA * p.A[1] + kg * p.g[1], kA * p.A[2] + kg * p.g[2], kg * p.g[3]};
  double M[4];
#pragma unroll
  for (int n = 0; n < 4; ++n) M[n] = pc[0] * mu[n] + pc[1] * mu[n + 1] + pc[2] * mu[n + 2] + pc[3] * mu[n + 3];
  dW[0] = M[0];
  dW[1] = M[1];
  dW[2] = q.V * M[0] + kA * p.vt[0] + kg * p.ng[0];
  dW[3] = 0.5 * M[2] + q.hE * M[0] + kA * p.et[0] + kg * p.eg[0];
  dF[0] = M[1];
  dF[1] = M[2];
  dF[2] = q.V * M[1] + kA * p.vt[1] + kg * p.ng[1];
  dF[3] = 0.5 * M[3] + q.hE * M[1] + kA * p.et[1] + kg * p.eg[1];
  const double Mb[4] = {WB[0] + q.V * WB[2] + q.hE * WB[3], WB[1] + q.V * FB[2] + q.hE * FB[3], FB[1] + 0.5 * WB[3],
                        0.5 * FB[3]};
  Vb += M[0] * WB[2] + M[1] * FB[2];
  hEb += M[0] * WB[3] + M[1] * FB[3];
  kb[1] += p.vt[0] * WB[2] + p.vt[1] * FB[2] + p.et[0] * WB[3] + p.et[1] * FB[3];
  kb[2] += p.ng[0] * WB[2] + p.ng[1] * FB[2] + p.eg[0] * WB[3] + p.eg[1] * FB[3];
  pb.vt[0] += kA * WB[2];
  pb.vt[1] += kA * FB[2];
  pb.et[0] += kA * WB[3];
  pb.et[1] += kA * FB[3];
  pb.ng[0] += kg * WB[2];
  pb.ng[1] += kg * FB[2];
  pb.eg[0] += kg * WB[3];
  pb.eg[1] += kg * FB[3];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    double pj = 0.0;
#pragma unroll
    for (int n = 0; n < 4; ++n) {
      pj += mu[n + j] * Mb[n];
      mub[n + j] += pc[j] * Mb[n];
    }
    if (j == 0) kb[0] += pj;
    if (j < 3) {
      kb[1] += p.A[j] * pj;
      pb.A[j] += kA * pj;
    }
    kb[2] += p.g[j] * pj;
    pb.g[j] += kg * pj;
  }
}

// pterms: from the adjoints pb of its terms to those of the slopes, the
// moments and the state (V through Vb).
FDK_HD void pterms_b(const PState<double>& q, double kappa, const Slope& a, const Slope& b, const Slope& t, const double* mu,
                     const PTerms<double, 2>& p, const PTerms<double, 2>& pb, Slope& ab, Slope& bb, Slope& tb, double* mub,
                     PrimB& sb) {
  double pa[3], pbb[3];
  slope_poly(q, a, pa);
  slope_poly(q, b, pbb);
  const double n0 = b.th + q.V * b.v + q.th * pbb[0], n1 = a.v + q.th * pbb[1], n2 = q.th * pbb[2];
  const double e0 = q.th * b.v + kappa * (q.V * b.th), e1 = kappa * a.th;
  const double ett = kappa * t.th + q.V * t.v;
  double n0b = 0.0, n1b = 0.0, n2b = 0.0, e0b = 0.0, e1b = 0.0, ettb = 0.0, Vb = 0.0;
#pragma unroll
  for (int n = 0; n < 2; ++n) {
    const double gb = pb.ng[n] + q.V * pb.eg[n];
    Vb += p.ng[n] * pb.eg[n];
    e0b += mu[n] * pb.eg[n];
    e1b += mu[n + 1] * pb.eg[n];
    ettb += mu[n] * pb.et[n];
    n0b += mu[n] * gb;
    n1b += mu[n + 1] * gb;
    n2b += mu[n + 2] * gb;
    tb.v += mu[n] * pb.vt[n];
    mub[n] += e0 * pb.eg[n] + ett * pb.et[n] + n0 * gb + t.v * pb.vt[n];
    mub[n + 1] += e1 * pb.eg[n] + n1 * gb;
    mub[n + 2] += n2 * gb;
  }
  tb.th += kappa * ettb;
  tb.v += q.V * ettb;
  ab.th += kappa * e1b;
  ab.v += n1b;
  bb.v += q.th * e0b + q.V * n0b + pb.g[0];
  bb.th += kappa * q.V * e0b + n0b;
  Vb += t.v * ettb + kappa * b.th * e0b + b.v * n0b + pbb[0] * pb.g[0] + pbb[1] * pb.g[1] + pbb[2] * pb.g[2];
  sb.V += Vb;
  sb.i2l += b.v * e0b + pbb[2] * n2b + pbb[1] * n1b + pbb[0] * n0b;
  const double qb[3] = {q.th * n0b + q.V * pb.g[0], q.th * n1b + q.V * pb.g[1], q.th * n2b + q.V * pb.g[2]};
  const double qa[3] = {pb.g[1], pb.g[2], pb.g[3]};
  slope_poly_b(q, b, pbb, qb, bb, sb);
  slope_poly_b(q, a, pa, qa, ab, sb);
  slope_poly_b(q, t, p.A, pb.A, tb, sb);
}

// Inputs of one interface solve and the adjoints of its outputs in slots of
// memory the caller chooses, STRIDE doubles apart (the reverse interface sweep
// keeps them in LDS, a thread's slots a block's threads apart: no two lanes
// meet on a bank).  The solve leaves the adjoints of the inputs in their slots.
enum { IO_WL = 0, IO_WR = 4, IO_NL = 8, IO_NR = 12, IO_WT = 16, IO_F = 20, IO_FT = 24, IO_W = 28, IO_WLT = 32, IO_WRT = 36,
       IO_SLOTS = 40 };
template <int STRIDE> struct SolveIO {
  double* p;
  FDK_HD double& operator()(int slot) const { return p[slot * STRIDE]; }
};

// Adjoint of the 2D interface solver (gks_iface<double, 2, VALUES>).  Slots
// IO_F, IO_FT: adjoints of F, Ft; IO_W: of Wl plus Wr (IO_WL + i, IO_WR + i
// take the e share of each, see below); IO_WLT, IO_WRT: of Wlt, Wrt; wl, wr:
// of Wl, Wr.  VALUES = false: F, Wl, Wr have no adjoint (stage 2).
//
// One pass over the three states (left, right, equilibrium), the iterations
// of one loop: each runs its state's forward terms and their reverse at once.
// That is possible because the adjoints of the moments follow from the outputs'
// and from W0, tau alone; what depends on the moments' values (the adjoint of
// exp(-dt/tau) and, through the Prandtl correction, of U0, V0) is a sum over
// the states.  A last part takes tau and W0 back to the two sides.
// Against the reverse of the moment vectors of psi (seven phases, half of them
// recomputing a side's state) the reverse interface sweep at 1024^2 takes 2.01
// and 1.83 (stage 2) instead of 3.4 ms, the node sweep 0.58 instead of 1.05
// (0.48 since smooth lines skip GENO's reverse).
template <bool VALUES, int STRIDE>
FDK_HD void gks_iface_b(const Consts& k, double dt, const SolveIO<STRIDE>& io, const double* wl, const double* wr) {
  const double K = k.K, gam = k.gamma, g1 = gam - 1.0, kappa = 0.5 * (K + 1.0), hK = 0.5 * (K + 2.0);
  const bool visc = k.mu > 0;
  double W0[4], tau, mS[2], xS[2];
  {
    double wL[4], wR[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) { wL[i] = io(IO_WL + i); wR[i] = io(IO_WR + i); }
    const Prim<double> sL = prim<double, 2>(wL, gam), sR = prim<double, 2>(wR, gam);
    half_moms(sL.lam, sL.i2l, sL.U, 1.0, mS[0], xS[0]);
    half_moms(sR.lam, sR.i2l, sR.U, -1.0, mS[1], xS[1]);
    const double XL = sL.rho * xS[0], XR = sR.rho * xS[1];
#pragma unroll
    for (int i = 0; i < 4; ++i) W0[i] = mS[0] * wL[i] + mS[1] * wR[i];
    W0[1] = W0[1] + (XL + XR);
    W0[3] = W0[3] + 0.5 * (sL.U * XL + sR.U * XR);
    const double p0 = (gam - 1.0) * (W0[3] - 0.5 * (W0[1] * W0[1] + W0[2] * W0[2]) * m_recip(W0[0]));
    tau = (visc ? k.mu * m_recip(p0) : k.tau_c1 * dt) + k.tau_c2 * dt * m_abs(sL.p - sR.p) * m_recip(sL.p + sR.p);
  }
  double Eh = 0.0, o = 1.0;
  if (tau > 1e-290) exp_neg(0.5 * dt * m_recip(tau), Eh, o);
  const double idt = m_recip(dt), oe = o * (2.0 - o);  // 1 - exp(-dt / tau)
  double nm[4], WLb[4], WRb[4], Wtb[4] = {0, 0, 0, 0}, W0b[4] = {0, 0, 0, 0};
  PrimB s0b = primb_zero();
  double c3b = 0.0, c4b = 0.0, ct0b = 0.0, ct1b = 0.0, ct2b = 0.0, taub = 0.0, eb = 0.0;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    nm[i] = 0.5 * (io(IO_NL + i) + io(IO_NR + i));
    WLb[i] = VALUES ? Eh * Eh * wl[i] : 0.0;
    WRb[i] = VALUES ? Eh * Eh * wr[i] : 0.0;
    if (VALUES) eb += io(IO_WL + i) * wl[i] + io(IO_WR + i) * wr[i];
  }
#pragma unroll 1
  for (int ph0 = 0; ph0 < 3; ++ph0) {
    phase_barrier();
    const int ph = opaque_int(ph0);
    const bool eq = ph == 2;
    const int sw = ph == 0 ? IO_WL : IO_WR, sn = ph == 0 ? IO_NL : IO_NR, sx = ph == 0 ? IO_WLT : IO_WRT;
    double W[4], n[4], tg[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      W[i] = eq ? W0[i] : io(sw + i);
      n[i] = eq ? nm[i] : io(sn + i);
      tg[i] = io(IO_WT + i);
    }
    const Prim<double> s = prim<double, 2>(W, gam);
    const double m0 = eq ? 1.0 : (ph == 0 ? mS[0] : mS[1]), x = eq ? 0.0 : (ph == 0 ? xS[0] : xS[1]);
    // forward terms
    const PState<double> q = pstate<double, 2>(s, kappa);
    const Slope a = prim_slope<double, 2>(s, g1, n), b = prim_slope<double, 2>(s, g1, tg);
    const Slope t = euler_slope<double, 2>(q, g1, a, b);
    double mu[7];
    mu[0] = m0;
    mu[1] = s.U * m0 + x;
    mu_rec(mu, s.U, s.i2l);
    const PTerms<double, 2> p = pterms<double, 2>(q, kappa, a, b, t, mu);
    // reverse of the two sums
    PrimB sb = primb_zero();
    PTerms<double, 2> pb{};
    double mub[7] = {0, 0, 0, 0, 0, 0, 0}, Vb = 0.0, hEb = 0.0;
#pragma unroll 1
    for (int set0 = VALUES ? 0 : 1; set0 < 2; ++set0) {
      phase_barrier();
      const int set = opaque_int(set0);
      const double W00 = fresh(W0[0]), iW0 = m_recip(W00), U0 = W0[1] * iW0, V0 = W0[2] * iW0;
      const double ua = 1.5 * U0 * U0 + 0.5 * V0 * V0, ub = 0.5 * U0 * (U0 * U0 + V0 * V0), UV = U0 * V0;
      // time coefficients: c3, c4, t0 = dt ct0, t1 give the ten (see time_coef)
      const double ft = fresh(tau), sd = ft * idt, c3 = sd * o * (2.0 + o), c0 = 1.0 - c3;
      const double c4 = ft * ((1.0 - o * o) - 2.0 * c3);
      const double t0 = 4.0 * sd * (o * o), t1 = 4.0 * sd * (o * (Eh - 2.0 * sd * o)), ct2 = 1.0 - sd * t0;
      const double ca0 = eq ? 0.0 : (set == 0 ? c3 : -(t0 * idt));
      const double ca1 = eq ? (set == 0 ? -ft * c0 : ct2) : -ft * ca0;
      const double ca2 = eq ? (set == 0 ? -ft - c4 : t1) : (set == 0 ? c4 : -t1);
      // adjoints of the sums: of the blend 1 - e, of F[0] = W[1] and of the Prandtl correction
      double raw[4], fo[4], WB[4], FB[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        raw[i] = set == 0 ? io(IO_W + i) : io(IO_WLT + i) + io(IO_WRT + i);
        fo[i] = io((set == 0 ? IO_F : IO_FT) + i);
        WB[i] = oe * raw[i];
        FB[i] = fo[i];
      }
      WB[1] += fo[0];
      const double fb = visc ? k.prfix * fo[3] : 0.0;
      if (visc) {
        FB[3] += fb;
        FB[1] -= U0 * fb;
        FB[2] -= V0 * fb;
        WB[1] += ua * fb;
        WB[3] -= U0 * fb;
        WB[2] += UV * fb;
        WB[0] -= ub * fb;
      }
      double kb[3] = {0, 0, 0}, dW[4], dF[4];
      padd_b(q, p, mu, s.rho * ca0, s.rho * ca1, s.rho * ca2, WB, FB, pb, mub, Vb, hEb, kb, dW, dF);
      sb.rho += ca0 * kb[0] + ca1 * kb[1] + ca2 * kb[2];
      const double k0b = s.rho * kb[0], kAb = s.rho * kb[1], kgb = s.rho * kb[2];
      if (eq) {
        // the leading terms: W0 and its Euler flux with c0 (ct0)
        const double cl = set == 0 ? c0 : t0 * idt, H = W0[3] + s.p;
        const double fe1 = s.p + s.U * W0[1], fe2 = s.V * W0[1], fe3 = s.U * H;
        double clb = fe1 * FB[1] + fe2 * FB[2] + fe3 * FB[3];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          clb += W0[i] * WB[i];
          dW[i] += cl * W0[i];
          W0b[i] += cl * WB[i];
        }
        dF[0] += cl * W0[1];
        dF[1] += cl * fe1;
        dF[2] += cl * fe2;
        dF[3] += cl * fe3;
        const double g1b = cl * FB[1], g2b = cl * FB[2], g3b = cl * FB[3];
        sb.p += g1b + s.U * g3b;
        sb.U += W0[1] * g1b + H * g3b;
        sb.V += W0[1] * g2b;
        W0b[1] += s.U * g1b + s.V * g2b;
        W0b[3] += s.U * g3b;
        if (set == 0) {  // c0 = 1 - c3, c1 = -tau - c4, c2 = -tau c0
          const double c0b = clb - tau * kAb;
          taub += -c0 * kAb - kgb;
          c4b += -kgb;
          c3b += -c0b;
        } else {
          ct0b += clb;
          ct1b += kgb;
          ct2b += kAb;
        }
      } else {
        taub += -ca0 * kAb;
        const double cb = k0b - tau * kAb;
        if (set == 0) {
          c3b += cb;
          c4b += kgb;
        } else {  // ct3 = -ct0, ct4 = -ct1
          ct0b -= cb;
          ct1b -= kgb;
        }
      }
      // the sums' values: shares of the adjoints of e and of U0, V0
#pragma unroll
      for (int i = 0; i < 4; ++i) eb -= raw[i] * dW[i];
      if (visc) {
        s0b.U += fb * (-dF[1] + 3.0 * U0 * dF[0] - dW[3] + V0 * dW[2] - 0.5 * (3.0 * U0 * U0 + V0 * V0) * dW[0]);
        s0b.V += fb * (-dF[2] + V0 * dF[0] + U0 * dW[2] - UV * dW[0]);
      }
    }
    sb.V += Vb + q.V * hEb;  // hE = kappa theta + V^2 / 2
    sb.i2l += kappa * hEb;
    phase_barrier();  // the inputs are read again below
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      if (!eq) {
        W[i] = io(sw + i);
        n[i] = io(sn + i);
      }
      tg[i] = io(IO_WT + i);
    }
    Slope ab{0, 0, 0, 0}, bb{0, 0, 0, 0}, tb{0, 0, 0, 0};
    if (!eq) {  // the side's Euler time derivative in Wlt / Wrt
      double Wt[4], wb[4];
      cons_t<double, 2>(s, hK, t, Wt);
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const double z = io(sx + i);
        eb += Wt[i] * z;
        wb[i] = Eh * Eh * z;
      }
      cons_t_b(s, hK, t, Wt, wb, tb, sb);
    }
    pterms_b(q, kappa, a, b, t, mu, p, pb, ab, bb, tb, mub, sb);
    euler_slope_b(s, g1, a, b, tb, ab, bb, sb);
    double nb[4] = {0, 0, 0, 0};
    prim_slope_b(s, g1, tg, b, bb, Wtb, sb);
    prim_slope_b(s, g1, n, a, ab, nb, sb);
    double Ub = 0.0, i2lb = 0.0;
    mu_rec_b(mu, s.U, s.i2l, mub, Ub, i2lb);
    sb.U += Ub + m0 * mub[1];
    sb.i2l += i2lb;
    if (eq) {
      s0b.rho += sb.rho;
      s0b.irho += sb.irho;
      s0b.U += sb.U;
      s0b.V += sb.V;
      s0b.p += sb.p;
      s0b.i2l += sb.i2l;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        io(IO_NL + i) += 0.5 * nb[i];
        io(IO_NR + i) += 0.5 * nb[i];
      }
    } else {
      half_moms_b(s, x, mub[0] + s.U * mub[1], mub[1], sb);
      if (ph == 0) prim_b(W, s, gam, sb, WLb);
      else prim_b(W, s, gam, sb, WRb);
#pragma unroll
      for (int i = 0; i < 4; ++i) io(sn + i) = nb[i];  // its forward value has done its part
    }
  }
  phase_barrier();
  // ---- time coefficients to tau
  {
    const double sd = tau * idt, c3 = sd * o * (2.0 + o), t0 = 4.0 * sd * (o * o);
    double sb = -t0 * ct2b, ob = -2.0 * Eh * eb;  // exp(-dt / tau) = (1 - o)^2
    const double t0b = ct0b * idt - sd * ct2b;
    taub += ((1.0 - o * o) - 2.0 * c3) * c4b;
    ob += -2.0 * o * tau * c4b;
    const double b3 = c3b - 2.0 * tau * c4b;
    const double z = Eh - 2.0 * sd * o;
    sb += o * (2.0 + o) * b3 + 4.0 * (o * o) * t0b + (4.0 * o * z - 8.0 * sd * (o * o)) * ct1b;
    ob += sd * (2.0 + 2.0 * o) * b3 + 8.0 * sd * o * t0b + 4.0 * sd * (z - o * (1.0 + 2.0 * sd)) * ct1b;
    taub += sb * idt;
    if (Eh > 0.0) {
      const double it = m_recip(tau);
      taub += -ob * Eh * (0.5 * dt * it) * it;
    }
  }
  // ---- tau and W0 to the two sides
  const Prim<double> s0 = prim<double, 2>(W0, gam);
  if (visc) s0b.p += -k.mu * (s0.ip * s0.ip) * taub;
  prim_b(W0, s0, gam, s0b, W0b);
  double wS[2][4];
#pragma unroll
  for (int i = 0; i < 4; ++i) { wS[0][i] = io(IO_WL + i); wS[1][i] = io(IO_WR + i); }
  const Prim<double> sS[2] = {prim<double, 2>(wS[0], gam), prim<double, 2>(wS[1], gam)};
  const double dP = sS[0].p - sS[1].p, iP = m_recip(sS[0].p + sS[1].p);
  const double sg = dP > 0 ? 1.0 : (dP < 0 ? -1.0 : 0.0), gt = k.tau_c2 * dt * iP * taub, ad = m_abs(dP) * iP;
#pragma unroll
  for (int sd2 = 0; sd2 < 2; ++sd2) {
    const Prim<double>& s = sS[sd2];
    double* Wb = sd2 == 0 ? WLb : WRb;
    const double x = xS[sd2], m0 = mS[sd2];
    PrimB sb = primb_zero();
    sb.p = gt * ((sd2 == 0 ? sg : -sg) - ad);
    // W0 = m0 W + rho x (0, 1, 0, U / 2)
    const double Xb = W0b[1] + 0.5 * s.U * W0b[3];
    double m0b = 0.0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      m0b += wS[sd2][i] * W0b[i];
      Wb[i] += m0 * W0b[i];
    }
    sb.U = 0.5 * s.rho * x * W0b[3];
    sb.rho = x * Xb;
    half_moms_b(s, x, m0b, s.rho * Xb, sb);
    prim_b(wS[sd2], s, gam, sb, Wb);
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    io(IO_WL + i) = WLb[i];
    io(IO_WR + i) = WRb[i];
    io(IO_WT + i) = Wtb[i];
  }
}

// Adjoint of the 2D nodal solver (gks_node<double, 2, VALUES>); VALUES =
// false: F, G have no adjoint (stage 2).
template <bool VALUES>
FDK_HD void gks_node_b(const Consts& k, const double* W, const double* Wx, const double* Wy, const double* Fb,
                       const double* Ftb, const double* Gb, const double* Gtb, double* Wb, double* Wxb, double* Wyb) {
  const double g1 = k.gamma - 1.0, hK = 0.5 * (k.K + 2.0), h1 = hK + 1.0, f = k.prfix;
  const bool visc = k.mu > 0;
  const Prim<double> s = prim<double, 2>(W, k.gamma);
  const PState<double> q = pstate<double, 2>(s, 0.0);
  const Slope a = prim_slope<double, 2>(s, g1, Wx), b = prim_slope<double, 2>(s, g1, Wy);
  const Slope t = euler_slope<double, 2>(q, g1, a, b);
  double Wt[4];
  cons_t<double, 2>(s, hK, t, Wt);
  const double pt = s.rho * t.th + s.i2l * Wt[0], H = W[3] + s.p, Ht = Wt[3] + pt;
  const double pc = visc ? f * h1 : 0.0;  // the Prandtl correction of f_t: pc p t.u
  PrimB sb = primb_zero();
  Slope ab{0, 0, 0, 0}, bb{0, 0, 0, 0}, tb{0, 0, 0, 0};
  const double x2 = Ftb[2] + Gtb[1];  // Ft[2] = Gt[1]
  double Wtb[4], Hb = t.u * Ftb[3] + t.v * Gtb[3];
  const double Htb = s.U * Ftb[3] + s.V * Gtb[3];
  const double ptb = Ftb[1] + Gtb[2] + Htb;
  Wtb[0] = s.i2l * ptb;
  Wtb[1] = Ftb[0] + s.U * Ftb[1] + s.V * x2;
  Wtb[2] = Gtb[0] + s.V * Gtb[2];
  Wtb[3] = Htb;
  sb.U = Wt[1] * Ftb[1] + Ht * Ftb[3];
  sb.V = Wt[1] * x2 + Wt[2] * Gtb[2] + Ht * Gtb[3];
  sb.p = pc * Hb;
  sb.rho = t.th * ptb;
  sb.i2l = Wt[0] * ptb;
  tb.u = W[1] * Ftb[1] + (H + pc * s.p) * Ftb[3];
  tb.v = W[1] * x2 + W[2] * Gtb[2] + (H + pc * s.p) * Gtb[3];
  tb.th = s.rho * ptb;
  Wb[1] += t.u * Ftb[1] + t.v * x2;
  Wb[2] += t.v * Gtb[2];
  if (VALUES) {
    const double f2 = Fb[2] + Gb[1];  // F[2] = G[1]
    Wb[1] += Fb[0] + s.U * Fb[1] + s.V * f2;
    Wb[2] += Gb[0] + s.V * Gb[2];
    sb.p += Fb[1] + Gb[2];
    sb.U += W[1] * Fb[1] + H * Fb[3];
    sb.V += W[1] * f2 + W[2] * Gb[2] + H * Gb[3];
    Hb += s.U * Fb[3] + s.V * Gb[3];
    if (visc) {
      const double tp = k.mu, kap = tp * h1 * (1.0 + f), div = g1 * (a.u + b.v);
      const double sxx = tp * (2.0 * a.u - div), syy = tp * (2.0 * b.v - div), sxy = tp * (b.u + a.v);
      const double xxb = -tp * (Fb[1] + s.U * Fb[3]), xyb = -tp * (f2 + s.V * Fb[3] + s.U * Gb[3]);
      const double yyb = -tp * (Gb[2] + s.V * Gb[3]);
      sb.U -= sxx * Fb[3] + sxy * Gb[3];
      sb.V -= sxy * Fb[3] + syy * Gb[3];
      ab.th -= kap * Fb[3];
      bb.th -= kap * Gb[3];
      ab.u += 2.0 * xxb - g1 * (xxb + yyb);
      bb.v += 2.0 * yyb - g1 * (xxb + yyb);
      bb.u += xyb;
      ab.v += xyb;
    }
  }
  Wb[3] += Hb;
  sb.p += Hb;
  cons_t_b(s, hK, t, Wt, Wtb, tb, sb);
  euler_slope_b(s, g1, a, b, tb, ab, bb, sb);
  prim_slope_b(s, g1, Wx, a, ab, Wxb, sb);
  prim_slope_b(s, g1, Wy, b, bb, Wyb, sb);
  prim_b(W, s, k.gamma, sb, Wb);
}

#pragma clang fp contract(on)

// ------------------------------------------------------------------ GENO
struct GenoIn {
  double IS1, IS2, IS3, q1, q2, q3, dq1, dq2, dq3, PH, PHx;
};

// Adjoint of geno() for outputs v, d, chi with adjoints vb, db, chib.
FDK_HD void geno_b(const Consts& k, const GenoIn& g, double d1, double d2, double d3, double vb, double db,
                   double chib, GenoIn& gb) {
  const double X = (g.IS2 + g.IS3) - 2.0 * g.IS1;
  const double tau = 0.5 * fabs(X);
  const double in23 = g.IS3 > g.IS2 ? g.IS3 : g.IS2;
  const int iH = in23 > g.IS1 ? (g.IS3 > g.IS2 ? 3 : 2) : 1;
  const double ISH = in23 > g.IS1 ? in23 : g.IS1;
  const double ln23 = g.IS3 < g.IS2 ? g.IS3 : g.IS2;
  const int iL = ln23 < g.IS1 ? (g.IS3 < g.IS2 ? 3 : 2) : 1;
  const double ISL = ln23 < g.IS1 ? ln23 : g.IS1;
  const double eH = ISH + k.eps, eL = ISL + k.eps;
  const double inv = 1.0 / (eH * eL);
  const double xH = tau * eL * inv, xL = tau * eH * inv;
  const double aH = 1.0 + ipow(xH, k.r), aL = 1.0 + ipow(xL, k.r);
  const double alpha = 2.0 * aH / (aH + aL);
  const double th = g_tanh(k.C * alpha);
  const double chi = th * k.inv_tanhC;
  if (th == 1.0 && chi == 1.0) {  // as in the forward: v = PH, d = PHx, d chi / d alpha = 0
    gb.PH += vb;
    gb.PHx += db;
    return;
  }
  const double t1 = sqr(g.IS1 + k.eps_a), t2 = sqr(g.IS2 + k.eps_a), t3 = sqr(g.IS3 + k.eps_a);
  const double w1 = d1 * t2 * t3, w2 = d2 * t1 * t3, w3 = d3 * t1 * t2;
  const double is = 1.0 / (w1 + w2 + w3);
  const double N = w1 * g.q1 + w2 * g.q2 + w3 * g.q3, Nx = w1 * g.dq1 + w2 * g.dq2 + w3 * g.dq3;
  const double PL = N * is, PLx = Nx * is;
  // v = chi PH + (1-chi) PL, d = chi PHx + (1-chi) PLx
  const double chit = chib + (g.PH - PL) * vb + (g.PHx - PLx) * db;
  gb.PH += chi * vb;
  gb.PHx += chi * db;
  const double PLb = (1.0 - chi) * vb, PLxb = (1.0 - chi) * db;
  gb.q1 += w1 * is * PLb; gb.q2 += w2 * is * PLb; gb.q3 += w3 * is * PLb;
  gb.dq1 += w1 * is * PLxb; gb.dq2 += w2 * is * PLxb; gb.dq3 += w3 * is * PLxb;
  const double isb = N * PLb + Nx * PLxb;
  const double Sb = -is * is * isb;
  const double w1b = (g.q1 * PLb + g.dq1 * PLxb) * is + Sb;
  const double w2b = (g.q2 * PLb + g.dq2 * PLxb) * is + Sb;
  const double w3b = (g.q3 * PLb + g.dq3 * PLxb) * is + Sb;
  const double t1b = d2 * t3 * w2b + d3 * t2 * w3b;
  const double t2b = d1 * t3 * w1b + d3 * t1 * w3b;
  const double t3b = d1 * t2 * w1b + d2 * t1 * w2b;
  gb.IS1 += 2.0 * (g.IS1 + k.eps_a) * t1b;
  gb.IS2 += 2.0 * (g.IS2 + k.eps_a) * t2b;
  gb.IS3 += 2.0 * (g.IS3 + k.eps_a) * t3b;
  // chi = tanh(C alpha) / tanh C
  const double alphab = k.inv_tanhC * k.C * (1.0 - th * th) * chit;
  const double den = aH + aL;
  const double aHb = alphab * 2.0 * aL / (den * den), aLb = -alphab * 2.0 * aH / (den * den);
  const double xHb = aHb * (k.r == 1 ? 1.0 : k.r * ipow(xH, k.r - 1));
  const double xLb = aLb * (k.r == 1 ? 1.0 : k.r * ipow(xL, k.r - 1));
  // xH = tau / eH, xL = tau / eL
  const double taub = xHb * eL * inv + xLb * eH * inv;
  const double ISHb = -xHb * xH / eH, ISLb = -xLb * xL / eL;
  if (iH == 1) gb.IS1 += ISHb; else if (iH == 2) gb.IS2 += ISHb; else gb.IS3 += ISHb;
  if (iL == 1) gb.IS1 += ISLb; else if (iL == 2) gb.IS2 += ISLb; else gb.IS3 += ISLb;
  const double Xb = 0.5 * (X > 0 ? 1.0 : (X < 0 ? -1.0 : 0.0)) * taub;
  gb.IS2 += Xb;
  gb.IS3 += Xb;
  gb.IS1 += -2.0 * Xb;
}

// Adjoint of recon_iface (one component): rb = adjoints of (vl, dl, cl, vr,
// dr, cr).  Adds into qb[4], xb[4].
FDK_HD void recon_iface_b(const Consts& k, const double q[4], const double x[4], double h, double invh,
                          const double rb[6], double qb[4], double xb[4]) {
  double PHlb = 0.0, PHrb = 0.0, PHxb = 0.0;
  const double q0 = q[0], q1 = q[1], q2 = q[2], q3 = q[3];
  if (k.variant == 2) {
    PHlb = rb[0];
    PHrb = rb[3];
    PHxb = rb[1] + rb[4];
  } else {
    const double hx0 = h * x[0], hx3 = h * x[3];
    const double s2 = q0 - 2.0 * q1 + q2, s3 = q1 - 2.0 * q2 + q3;
    const double D2 = s2 * s2, D3 = s3 * s3;
    const double Al = q1 - q0 - hx0, Bl = 2.0 * (q1 - q0) - hx0, El = 3.0 * q1 - 4.0 * q2 + q3;
    const double Ar = q2 - q3 + hx3, Br = 2.0 * (q3 - q2) - hx3, Er = 3.0 * q2 - 4.0 * q1 + q0;
    const double ISl1 = (13.0 / 3.0) * Al * Al + Bl * Bl, ISl2 = (13.0 / 12.0) * D2 + 0.25 * sqr(q2 - q0),
                 ISl3 = (13.0 / 12.0) * D3 + 0.25 * El * El;
    const double ISr1 = (13.0 / 3.0) * Ar * Ar + Br * Br, ISr2 = (13.0 / 12.0) * D3 + 0.25 * sqr(q3 - q1),
                 ISr3 = (13.0 / 12.0) * D2 + 0.25 * Er * Er;
    // smooth lines (chi = 1 on both sides, see geno_smooth) are linear in their values
    if ((int)geno_smooth<double>(k, ISl1, ISl2, ISl3) & (int)geno_smooth<double>(k, ISr1, ISr2, ISr3)) {
      PHlb = rb[0];
      PHrb = rb[3];
      PHxb = rb[1] + rb[4];
    } else {
      const double dmid = (q2 - q1) * invh;
      const double qc = (-q0 + 6.0 * q1 + 3.0 * q2) * 0.125;
      const double PHl = ((7.0 * q0 + 35.0 * q1 + 21.0 * q2 + q3) + (x[0] + 22.0 * x[1] - 7.0 * x[2]) * h) * (1.0 / 64.0);
      const double PHr = ((q0 + 21.0 * q1 + 35.0 * q2 + 7.0 * q3) + (7.0 * x[1] - 22.0 * x[2] - x[3]) * h) * (1.0 / 64.0);
      const double PHx = -((q0 + 45.0 * q1 - 45.0 * q2 - q3) + 9.0 * (x[1] + x[2]) * h) * (invh * (1.0 / 30.0));
      GenoIn L{ISl1, ISl2, ISl3, (-5.0 * q0 + 9.0 * q1 - 3.0 * hx0) * 0.25, qc,
               (3.0 * q1 + 6.0 * q2 - q3) * 0.125, (-3.0 * q0 + 3.0 * q1 - 2.0 * hx0) * invh, dmid, dmid, PHl, PHx};
      GenoIn R{ISr1, ISr2, ISr3, (-5.0 * q3 + 9.0 * q2 + 3.0 * hx3) * 0.25,
               (-q3 + 6.0 * q2 + 3.0 * q1) * 0.125, qc, (-3.0 * q2 + 3.0 * q3 - 2.0 * hx3) * invh, dmid, dmid, PHr, PHx};
      GenoIn Lb{0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0}, Rb{0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
      geno_b(k, L, k.ds, k.dc, k.ds, rb[0], rb[1], rb[2], Lb);
      geno_b(k, R, k.ds, k.dc, k.ds, rb[3], rb[4], rb[5], Rb);
      PHlb = Lb.PH;
      PHrb = Rb.PH;
      PHxb = Lb.PHx + Rb.PHx;
      double hx0b = 0.0, hx3b = 0.0, D2b = 0.0, D3b = 0.0;
      const double qcb = Lb.q2 + Rb.q3, dmidb = Lb.dq2 + Lb.dq3 + Rb.dq2 + Rb.dq3;
      // right side
      qb[2] += -3.0 * invh * Rb.dq1; qb[3] += 3.0 * invh * Rb.dq1; hx3b += -2.0 * invh * Rb.dq1;
      qb[3] += -0.125 * Rb.q2; qb[2] += 0.75 * Rb.q2; qb[1] += 0.375 * Rb.q2;
      qb[3] += -1.25 * Rb.q1; qb[2] += 2.25 * Rb.q1; hx3b += 0.75 * Rb.q1;
      {
        D2b += (13.0 / 12.0) * Rb.IS3;
        const double Eb = 0.5 * Er * Rb.IS3;
        qb[2] += 3.0 * Eb; qb[1] += -4.0 * Eb; qb[0] += Eb;
        D3b += (13.0 / 12.0) * Rb.IS2;
        const double t = 0.5 * (q3 - q1) * Rb.IS2;
        qb[3] += t; qb[1] -= t;
        const double Ab = (26.0 / 3.0) * Ar * Rb.IS1, Bb = 2.0 * Br * Rb.IS1;
        qb[2] += Ab - 2.0 * Bb; qb[3] += -Ab + 2.0 * Bb; hx3b += Ab - Bb;
      }
      // left side
      qb[0] += -3.0 * invh * Lb.dq1; qb[1] += 3.0 * invh * Lb.dq1; hx0b += -2.0 * invh * Lb.dq1;
      qb[1] += 0.375 * Lb.q3; qb[2] += 0.75 * Lb.q3; qb[3] += -0.125 * Lb.q3;
      qb[0] += -1.25 * Lb.q1; qb[1] += 2.25 * Lb.q1; hx0b += -0.75 * Lb.q1;
      {
        D3b += (13.0 / 12.0) * Lb.IS3;
        const double Eb = 0.5 * El * Lb.IS3;
        qb[1] += 3.0 * Eb; qb[2] += -4.0 * Eb; qb[3] += Eb;
        D2b += (13.0 / 12.0) * Lb.IS2;
        const double t = 0.5 * (q2 - q0) * Lb.IS2;
        qb[2] += t; qb[0] -= t;
        const double Ab = (26.0 / 3.0) * Al * Lb.IS1, Bb = 2.0 * Bl * Lb.IS1;
        qb[1] += Ab + 2.0 * Bb; qb[0] += -Ab - 2.0 * Bb; hx0b += -Ab - Bb;
      }
      // shared
      qb[0] += -0.125 * qcb; qb[1] += 0.75 * qcb; qb[2] += 0.375 * qcb;
      qb[2] += invh * dmidb; qb[1] -= invh * dmidb;
      const double s3b = 2.0 * s3 * D3b, s2b = 2.0 * s2 * D2b;
      qb[1] += s3b; qb[2] += -2.0 * s3b; qb[3] += s3b;
      qb[0] += s2b; qb[1] += -2.0 * s2b; qb[2] += s2b;
      xb[0] += h * hx0b;
      xb[3] += h * hx3b;
    }
  }
  const double c = 1.0 / 64.0, kx = -invh * (1.0 / 30.0);
  qb[0] += 7.0 * c * PHlb + c * PHrb + kx * PHxb;
  qb[1] += 35.0 * c * PHlb + 21.0 * c * PHrb + 45.0 * kx * PHxb;
  qb[2] += 21.0 * c * PHlb + 35.0 * c * PHrb - 45.0 * kx * PHxb;
  qb[3] += c * PHlb + 7.0 * c * PHrb - kx * PHxb;
  xb[0] += h * c * PHlb;
  xb[1] += 22.0 * h * c * PHlb + 7.0 * h * c * PHrb + 9.0 * h * kx * PHxb;
  xb[2] += -7.0 * h * c * PHlb - 22.0 * h * c * PHrb + 9.0 * h * kx * PHxb;
  xb[3] += -h * c * PHrb;
}

// Adjoint of recon_node: db is the adjoint of the node derivative.  Adds into
// qb[3], xb[3].
FDK_HD void recon_node_b(const Consts& k, const double q[3], const double x[3], double h, double invh, double db,
                         double qb[3], double xb[3]) {
  double PHxb = db;
  if (k.variant != 2) {
    const double q0 = q[0], q1 = q[1], q2 = q[2];
    const double hx0 = h * x[0], hx2 = h * x[2];
    const double A1 = q1 - q0 - hx0, B1 = 2.0 * (q1 - q0) - hx0;
    const double A2 = q2 - q1 - hx2, B2 = 2.0 * (q2 - q1) - hx2;
    const double s = q0 - 2.0 * q1 + q2, u = q2 - q0;
    const double IS1 = (13.0 / 3.0) * A1 * A1 + B1 * B1;
    const double IS2 = (13.0 / 3.0) * A2 * A2 + B2 * B2;
    const double IS3 = (13.0 / 12.0) * s * s + 0.25 * u * u;
    if (!geno_smooth<double>(k, IS3, IS1, IS2)) {  // smooth lines are linear in their values: PHxb = db
      const double PHx = (9.0 * (q0 - q2) + h * (x[0] + 46.0 * x[1] + x[2])) * (invh * (1.0 / 30.0));
      GenoIn g{IS3, IS1, IS2, q1, q1, q1, (q2 - q0) * (0.5 * invh), (-2.0 * q0 + 2.0 * q1 - hx0) * invh,
               (-2.0 * q1 + 2.0 * q2 - hx2) * invh, q1, PHx};
      GenoIn gb{0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
      geno_b(k, g, k.dc, k.ds, k.ds, 0.0, db, 0.0, gb);
      PHxb = gb.PHx;
      double hx0b = 0.0, hx2b = 0.0;
      qb[1] += gb.q1 + gb.q2 + gb.q3 + gb.PH;
      qb[2] += 0.5 * invh * gb.dq1;
      qb[0] -= 0.5 * invh * gb.dq1;
      qb[0] += -2.0 * invh * gb.dq2; qb[1] += 2.0 * invh * gb.dq2; hx0b += -invh * gb.dq2;
      qb[1] += -2.0 * invh * gb.dq3; qb[2] += 2.0 * invh * gb.dq3; hx2b += -invh * gb.dq3;
      {
        const double sb = (13.0 / 6.0) * s * gb.IS1, ub = 0.5 * u * gb.IS1;
        qb[0] += sb - ub; qb[1] += -2.0 * sb; qb[2] += sb + ub;
        const double Ab2 = (26.0 / 3.0) * A2 * gb.IS3, Bb2 = 2.0 * B2 * gb.IS3;
        qb[2] += Ab2 + 2.0 * Bb2; qb[1] += -Ab2 - 2.0 * Bb2; hx2b += -Ab2 - Bb2;
        const double Ab1 = (26.0 / 3.0) * A1 * gb.IS2, Bb1 = 2.0 * B1 * gb.IS2;
        qb[1] += Ab1 + 2.0 * Bb1; qb[0] += -Ab1 - 2.0 * Bb1; hx0b += -Ab1 - Bb1;
      }
      xb[0] += h * hx0b;
      xb[2] += h * hx2b;
    }
  }
  const double kx = invh * (1.0 / 30.0);
  qb[0] += 9.0 * kx * PHxb;
  qb[2] += -9.0 * kx * PHxb;
  xb[0] += h * kx * PHxb;
  xb[1] += 46.0 * h * kx * PHxb;
  xb[2] += h * kx * PHxb;
}

// ---------------------------------------------- characteristic variables
// Reverse of the 2D characteristic reconstructions (recon_iface_char<2>,
// recon_node_char<2> in gks_device.hpp): the frame (eigenvectors at the mean
// interface state, or at the node) depends on the line's values, so its
// adjoint flows back into them as well.
struct FrameB {
  double u, v, c, ic, H, b1, b2, k2;
};
FDK_HD FrameB frameb_zero() { return FrameB{0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0}; }

// q = L(f) w: adds L^T qb to wb and the frame's adjoint to fb.
FDK_HD void to_char_b(const CharFrame& f, const double* w, const double* qb, double* wb, FrameB& fb) {
  const double ab = 0.5 * (qb[0] + qb[3]) - qb[1];  // a = b2 w0 + s
  const double mb = 0.5 * (qb[3] - qb[0]);           // m = ic w1 - u ic w0
  const double sb = ab;                               // s = b1 (w3 - u w1 - v w2)
  wb[0] += qb[1] - f.v * qb[2] + f.b2 * ab - f.u * f.ic * mb;
  wb[1] += f.ic * mb - f.u * f.b1 * sb;
  wb[2] += qb[2] - f.v * f.b1 * sb;
  wb[3] += f.b1 * sb;
  fb.b2 += w[0] * ab;
  fb.b1 += (w[3] - f.u * w[1] - f.v * w[2]) * sb;
  fb.ic += (w[1] - f.u * w[0]) * mb;
  fb.u += -f.ic * w[0] * mb - f.b1 * w[1] * sb;
  fb.v += -w[0] * qb[2] - f.b1 * w[2] * sb;
}

// w = R(f) q: adds R^T wb to qb and the frame's adjoint to fb.
FDK_HD void from_char_b(const CharFrame& f, const double* q, const double* wb, double* qb, FrameB& fb) {
  const double lo = q[0], en = q[1], sh = q[2], hi = q[3], sum = lo + en + hi, d = hi - lo;
  const double sb = wb[0] + f.u * wb[1] + f.v * wb[2];
  qb[0] += sb - f.c * wb[1] + (f.H - f.u * f.c) * wb[3];
  qb[1] += sb + f.k2 * wb[3];
  qb[2] += wb[2] + f.v * wb[3];
  qb[3] += sb + f.c * wb[1] + (f.H + f.u * f.c) * wb[3];
  fb.u += sum * wb[1] + f.c * d * wb[3];
  fb.v += sum * wb[2] + sh * wb[3];
  fb.c += d * wb[1] + f.u * d * wb[3];
  fb.H += (lo + hi) * wb[3];
  fb.k2 += en * wb[3];
}

// The frame from the state W: adds the adjoint of W.
FDK_HD void char_frame_b(double gamma, const double* W, const CharFrame& f, FrameB fb, double* Wb) {
  const double ir = 1.0 / W[0], gm = gamma - 1.0;
  const double p = gm * (W[3] - W[0] * f.k2), c2 = f.c * f.c;
  fb.b1 += f.k2 * fb.b2;  // b2 = b1 k2
  fb.k2 += f.b1 * fb.b2;
  double c2b = -gm / (c2 * c2) * fb.b1;                 // b1 = (gamma - 1) / c2
  fb.c += -fb.ic / c2;                                  // ic = 1 / c
  c2b += fb.c / (2.0 * f.c);                            // c = sqrt(c2)
  double pb = ir * fb.H + gamma * ir * c2b;             // H = (W3 + p) ir, c2 = gamma p ir
  double irb = (W[3] + p) * fb.H + gamma * p * c2b;
  Wb[3] += ir * fb.H + gm * pb;                         // p = (gamma - 1)(W3 - W0 k2)
  Wb[0] += -gm * f.k2 * pb;
  fb.k2 += -gm * W[0] * pb;
  fb.u += f.u * fb.k2;                                  // k2 = (u^2 + v^2) / 2
  fb.v += f.v * fb.k2;
  Wb[1] += ir * fb.u;                                   // u = W1 ir, v = W2 ir
  Wb[2] += ir * fb.v;
  irb += W[1] * fb.u + W[2] * fb.v;
  Wb[0] += -ir * ir * irb;                              // ir = 1 / W0
}

// Reverse of recon_iface_char<2>.  rb[c]: adjoints of rec[c].vl, dl, vr, dr
// (local frame); chib: adjoint of chi.  Adds into Qb, Xb.  chi's adjoint goes
// to the first of chi^l(u-c), chi^r(u-c), chi^l(u+c), chi^r(u+c) that attains
// the minimum.
FDK_HD void recon_iface_char_b(const Consts& k, const double (&Q)[4][4], const double (&X)[4][4], double h,
                               double invh, const double (&rb)[4][4], double chib, double (&Qb)[4][4],
                               double (&Xb)[4][4]) {
  double Wm[4];
#pragma unroll
  for (int c = 0; c < 4; ++c) Wm[c] = 0.5 * (Q[c][1] + Q[c][2]);
  const CharFrame f = char_frame<2>(k.gamma, Wm);
  double qc[4][4], xc[4][4];
#pragma unroll
  for (int m = 0; m < 4; ++m) {
    double a[4], b[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) a[c] = Q[c][m];
    to_char<2>(f, a, b);
#pragma unroll
    for (int c = 0; c < 4; ++c) { qc[c][m] = b[c]; a[c] = X[c][m]; }
    to_char<2>(f, a, b);
#pragma unroll
    for (int c = 0; c < 4; ++c) xc[c][m] = b[c];
  }
  IfaceRec cr[4];
#pragma unroll
  for (int c = 0; c < 4; ++c)
    cr[c] = recon_iface<double>(k, qc[c][0], qc[c][1], qc[c][2], qc[c][3], xc[c][0], xc[c][1], xc[c][2], xc[c][3],
                                h, invh);
  // adjoints of the characteristic results (vl, dl, cl, vr, dr, cr per field)
  double crb[4][6];
#pragma unroll
  for (int c = 0; c < 4; ++c)
#pragma unroll
    for (int t = 0; t < 6; ++t) crb[c][t] = 0.0;
  FrameB fb = frameb_zero();
#pragma unroll
  for (int slot = 0; slot < 4; ++slot) {  // vl, dl, vr, dr
    const int t = slot < 2 ? slot : slot + 1;
    double a[4], wb[4], ab[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      a[c] = t == 0 ? cr[c].vl : (t == 1 ? cr[c].dl : (t == 3 ? cr[c].vr : cr[c].dr));
      wb[c] = rb[c][slot];
    }
    from_char_b(f, a, wb, ab, fb);
#pragma unroll
    for (int c = 0; c < 4; ++c) crb[c][t] += ab[c];
  }
  {
    const double cand[4] = {cr[0].cl, cr[0].cr, cr[3].cl, cr[3].cr};
    int sel = 0;
#pragma unroll
    for (int a = 1; a < 4; ++a)
      if (cand[a] < cand[sel]) sel = a;
    crb[sel < 2 ? 0 : 3][sel % 2 == 0 ? 2 : 5] += chib;
  }
  double qcb[4][4], xcb[4][4];
#pragma unroll
  for (int c = 0; c < 4; ++c) {
#pragma unroll
    for (int m = 0; m < 4; ++m) { qcb[c][m] = 0.0; xcb[c][m] = 0.0; }
    recon_iface_b(k, qc[c], xc[c], h, invh, crb[c], qcb[c], xcb[c]);
  }
#pragma unroll
  for (int m = 0; m < 4; ++m) {
    double a[4], b[4], wb[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int c = 0; c < 4; ++c) { a[c] = Q[c][m]; b[c] = qcb[c][m]; }
    to_char_b(f, a, b, wb, fb);
#pragma unroll
    for (int c = 0; c < 4; ++c) { Qb[c][m] += wb[c]; wb[c] = 0.0; a[c] = X[c][m]; b[c] = xcb[c][m]; }
    to_char_b(f, a, b, wb, fb);
#pragma unroll
    for (int c = 0; c < 4; ++c) Xb[c][m] += wb[c];
  }
  double Wmb[4] = {0.0, 0.0, 0.0, 0.0};
  char_frame_b(k.gamma, Wm, f, fb, Wmb);
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    Qb[c][1] += 0.5 * Wmb[c];
    Qb[c][2] += 0.5 * Wmb[c];
  }
}

// Reverse of recon_node_char<2>: db = adjoint of the node derivative d (local
// frame).  Adds into Qb, Xb.
FDK_HD void recon_node_char_b(const Consts& k, const double (&Q)[4][3], const double (&X)[4][3], double h,
                              double invh, const double (&db)[4], double (&Qb)[4][3], double (&Xb)[4][3]) {
  double Wc[4];
#pragma unroll
  for (int c = 0; c < 4; ++c) Wc[c] = Q[c][1];
  const CharFrame f = char_frame<2>(k.gamma, Wc);
  double qc[4][3], xc[4][3];
#pragma unroll
  for (int m = 0; m < 3; ++m) {
    double a[4], b[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) a[c] = Q[c][m];
    to_char<2>(f, a, b);
#pragma unroll
    for (int c = 0; c < 4; ++c) { qc[c][m] = b[c]; a[c] = X[c][m]; }
    to_char<2>(f, a, b);
#pragma unroll
    for (int c = 0; c < 4; ++c) xc[c][m] = b[c];
  }
  double dc[4];
#pragma unroll
  for (int c = 0; c < 4; ++c)
    dc[c] = recon_node<double>(k, qc[c][0], qc[c][1], qc[c][2], xc[c][0], xc[c][1], xc[c][2], h, invh);
  FrameB fb = frameb_zero();
  double dcb[4] = {0.0, 0.0, 0.0, 0.0};
  from_char_b(f, dc, db, dcb, fb);
  double qcb[4][3], xcb[4][3];
#pragma unroll
  for (int c = 0; c < 4; ++c) {
#pragma unroll
    for (int m = 0; m < 3; ++m) { qcb[c][m] = 0.0; xcb[c][m] = 0.0; }
    recon_node_b(k, qc[c], xc[c], h, invh, dcb[c], qcb[c], xcb[c]);
  }
#pragma unroll
  for (int m = 0; m < 3; ++m) {
    double a[4], b[4], wb[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int c = 0; c < 4; ++c) { a[c] = Q[c][m]; b[c] = qcb[c][m]; }
    to_char_b(f, a, b, wb, fb);
#pragma unroll
    for (int c = 0; c < 4; ++c) { Qb[c][m] += wb[c]; wb[c] = 0.0; a[c] = X[c][m]; b[c] = xcb[c][m]; }
    to_char_b(f, a, b, wb, fb);
#pragma unroll
    for (int c = 0; c < 4; ++c) Xb[c][m] += wb[c];
  }
  double Wcb[4] = {0.0, 0.0, 0.0, 0.0};
  char_frame_b(k.gamma, Wc, f, fb, Wcb);
#pragma unroll
  for (int c = 0; c < 4; ++c) Qb[c][1] += Wcb[c];
}

}  // namespace fdk
