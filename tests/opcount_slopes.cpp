// Source-level operation count of one stage-1 interface point in the form that
// FP64 runs (the solver in primitive slopes), with the counting scalar of
// opcount_iface.cpp; its entry counts the form from moment vectors.  exp, erf
// and the square root count as one operation each, as there.
#define main opcount_moments
#include "opcount_iface.cpp"
#undef main

namespace fdk {

inline void exp_neg(Cnt x, Cnt& E, Cnt& o) {
  ++C.exp;
  E = Cnt(std::exp(-x.v));
  o = Cnt(-std::expm1(-x.v));
}
inline void half_moms(Cnt lam, Cnt i2l, Cnt U, double sgn, Cnt& m0, Cnt& x) {
  const Cnt sl = m_sqrt(lam), z = sl * U;
  m0 = Cnt(0.5) * m_erfc(Cnt(-sgn * z.v));
  Cnt E, o;
  exp_neg(z * z, E, o);
  x = sgn * E * (i2l * sl) * 0.56418958354775628695;
}
// time_coef's FP64 branch, operation for operation
inline TimeCoef<Cnt> time_coef(Cnt dt, Cnt tau) {
  TimeCoef<Cnt> r;
  Cnt Eh, o;
  exp_neg(0.5 * dt * m_recip(tau), Eh, o);
  const Cnt idt = m_recip(dt), s = tau * idt;
  r.e1 = Eh * Eh;
  const Cnt c3 = s * o * (2.0 + o);
  const Cnt c4 = tau * ((1.0 - o * o) - 2.0 * c3);
  const Cnt t0 = 4.0 * s * (o * o), t1 = 4.0 * s * (o * (Eh - 2.0 * s * o));
  r.c[0] = 1.0 - c3;
  r.c[1] = -tau - c4;
  r.c[2] = -tau * r.c[0];
  r.c[3] = c3;
  r.c[4] = c4;
  r.ct[0] = t0 * idt;
  r.ct[1] = t1;
  r.ct[2] = 1.0 - s * t0;
  r.ct[3] = -r.ct[0];
  r.ct[4] = -t1;
  return r;
}

}  // namespace fdk

int main() {
  const fdk::Consts k = consts();
  const double h = 1.0 / 2048.0;
  const double base[4] = {1.0, 0.3, -0.05, 1.0 / (1.4 * 0.15 * 0.15) / 0.4 + 0.5 * 0.09};
  fdk::C = fdk::Counts();
  for (int G = 0; G < 2; ++G) {
    fdk::GksIO<Cnt, 2> io;
    for (int c = 0; c < 4; ++c) {
      Cnt q[4], x[4];
      for (int m = 0; m < 4; ++m) {
        q[m] = Cnt(base[c] * (1.0 + 1e-3 * (m - 1.5)));
        x[m] = Cnt(base[c] * 1e-3 / h);
      }
      fdk::IfaceRecT<Cnt> r = fdk::recon_iface<Cnt>(k, q[0], q[1], q[2], q[3], x[0], x[1], x[2], x[3], h, 1.0 / h);
      io.WL[c] = r.vl;
      io.WR[c] = r.vr;
      io.nL[c] = r.dl;
      io.nR[c] = r.dr;
      io.Wt[c] = 0.5 * (r.dl + r.dr);
    }
    fdk::gks_iface_slopes<Cnt, 2, true>(k, Cnt(1e-5), io);
  }
  // partner exchange and blend, as in opcount_iface.cpp
  fdk::C.add += 2 * 4 * (2 + 4);
  fdk::C.mul += 2 * 4 * 8;
  const fdk::Counts& c = fdk::C;
  std::printf("{\"add\": %ld, \"mul\": %ld, \"div\": %ld, \"sqrt\": %ld, \"exp\": %ld, \"erfc\": %ld, \"arith\": %ld}\n",
              c.add, c.mul, c.div, c.sqrt, c.exp, c.erfc, c.add + c.mul + c.div + c.sqrt);
  return 0;
}
