// The reverse gas-kinetic solvers of gks_adjoint.hpp against central
// differences, in long double, of the forward moment form (gks_iface_moments,
// gks_node_moments of gks_device.hpp) on seeded states and output adjoints.
// Reads lines "mu mach jump dt count seed"; prints the largest error per line
// of an input's adjoint, relative to the largest adjoint of its solve.
// Host only (--cuda-host-only).
#include <cmath>

typedef long double LD;
namespace fdk {
inline LD m_erfc(LD x) { return erfcl(x); }
inline LD m_exp(LD x) { return expl(x); }
inline LD m_sqrt(LD x) { return sqrtl(x); }
inline LD m_abs(LD x) { return fabsl(x); }
inline LD val(LD x) { return x; }
}  // namespace fdk

#include <cstdio>
#include <random>

#include "../paper_2606_17772_amd/csrc/gks_adjoint.hpp"

// Largest difference of g (n adjoints) from central differences of f at x.
template <class F> static double check(const F& f, const double* x, const double* g, int n) {
  // four-point differences: the moment form's time coefficients lose (tau / dt)^2 units of
  // their last digit, which a step of 1e-6 would raise above the bound at tau / dt = 1000
  const LD h = 5e-5L;
  double big = 0.0, err = 0.0;
  LD y[32];
  for (int i = 0; i < n; ++i) y[i] = x[i];
  for (int i = 0; i < n; ++i) {
    auto at = [&](LD m) {
      y[i] = (LD)x[i] + m * h;
      return f(y);
    };
    const double d = (double)((8 * (at(1) - at(-1)) - (at(2) - at(-2))) / (12 * h));
    y[i] = x[i];
    big = std::fmax(big, std::fabs(d));
    err = std::fmax(err, std::fabs(g[i] - d));
  }
  return err / big;
}

template <bool VALUES> static double worst(double mu, double mach, double jump, double dt, int count, int seed) {
  std::mt19937_64 rng(seed);
  auto U = [&](double a, double b) { return std::uniform_real_distribution<double>(a, b)(rng); };
  fdk::Consts k{};
  // gamma = 1.5: gamma - 1, K and their products are exact, so both forms solve the same equations
  k.gamma = 1.5;
  k.K = 2.0;
  k.inv_Kd = 0.25;
  k.mu = mu;
  k.prfix = mu > 0 ? 0.375 : 0.0;
  k.tau_c1 = 0.05;
  k.tau_c2 = 1.0;
  double w = 0.0;
  for (int it = 0; it < count; ++it) {
    double x[20], ob[6][4];  // WL, WR, nL, nR, Wt; adjoints of F, Ft, Wl, Wr, Wlt, Wrt
    auto state = [&](double* W, double r, double u, double v, double p) {
      W[0] = r;
      W[1] = r * u;
      W[2] = r * v;
      W[3] = p / 0.5 + 0.5 * r * (u * u + v * v);
    };
    const double r = U(0.5, 1.5), u = mach * U(-1, 1), v = mach * U(-1, 1), p = U(0.5, 1.5);
    state(x, r, u, v, p);
    // the pressures differ by more than the difference step: |p_l - p_r| is smooth around the point
    state(x + 4, r * (1 + jump * U(-1, 1)), u + jump * U(-1, 1), v + jump * U(-1, 1), p * (1 + jump * U(0.2, 1)));
    for (int c = 8; c < 20; ++c) x[c] = U(-1, 1);
    for (auto& o : ob)
      for (double& q : o) q = U(-1, 1);
    if (!VALUES)
      for (int c = 0; c < 4; ++c) ob[0][c] = ob[2][c] = ob[3][c] = 0.0;
    double slots[fdk::IO_SLOTS];
    for (int c = 0; c < 20; ++c) slots[c] = x[c];
    for (int c = 0; c < 4; ++c) {
      slots[fdk::IO_F + c] = ob[0][c];
      slots[fdk::IO_FT + c] = ob[1][c];
      slots[fdk::IO_W + c] = ob[2][c] + ob[3][c];
      slots[fdk::IO_WLT + c] = ob[4][c];
      slots[fdk::IO_WRT + c] = ob[5][c];
    }
    fdk::gks_iface_b<VALUES>(k, dt, fdk::SolveIO<1>{slots}, ob[2], ob[3]);
    auto f = [&](const LD* y) {
      fdk::GksIO<LD, 2> a;
      for (int c = 0; c < 4; ++c) {
        a.WL[c] = y[c];
        a.WR[c] = y[4 + c];
        a.nL[c] = y[8 + c];
        a.nR[c] = y[12 + c];
        a.Wt[c] = y[16 + c];
      }
      fdk::gks_iface_moments<LD, 2, true>(k, (LD)dt, a);
      LD s = 0;
      for (int c = 0; c < 4; ++c)
        s += ob[0][c] * a.F[c] + ob[1][c] * a.Ft[c] + ob[2][c] * a.Wl[c] + ob[3][c] * a.Wr[c] + ob[4][c] * a.Wlt[c] +
             ob[5][c] * a.Wrt[c];
      return s;
    };
    w = std::fmax(w, check(f, x, slots, 20));
    // the nodal solver at the left state with slopes nL, nR; adjoints of F, Ft, G, Gt
    double g[12] = {0}, zero[4] = {0, 0, 0, 0};
    const double *Fb = VALUES ? ob[1] : zero, *Gb = VALUES ? ob[4] : zero;
    fdk::gks_node_b<VALUES>(k, x, x + 8, x + 12, Fb, ob[5], Gb, slots, g, g + 4, g + 8);
    auto fn = [&](const LD* y) {
      LD F[4], Ft[4], G[4], Gt[4], s = 0;
      fdk::gks_node_moments<LD, 2, true>(k, y, y + 4, y + 8, F, Ft, G, Gt);
      for (int c = 0; c < 4; ++c) s += Fb[c] * F[c] + ob[5][c] * Ft[c] + Gb[c] * G[c] + slots[c] * Gt[c];
      return s;
    };
    double xn[12];
    for (int c = 0; c < 4; ++c) { xn[c] = x[c]; xn[4 + c] = x[8 + c]; xn[8 + c] = x[12 + c]; }
    w = std::fmax(w, check(fn, xn, g, 12));
  }
  return w;
}

int main() {
  double mu, mach, jump, dt;
  int count, seed;
  while (scanf("%lf %lf %lf %lf %d %d", &mu, &mach, &jump, &dt, &count, &seed) == 6)
    printf("%.3e %.3e\n", worst<true>(mu, mach, jump, dt, count, seed), worst<false>(mu, mach, jump, dt, count, seed));
  return 0;
}
