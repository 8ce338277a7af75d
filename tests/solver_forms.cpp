// The FP64 gas-kinetic solvers (gks_iface, gks_node of gks_device.hpp, in
// primitive slopes and closed form) against their moment form in long double,
// on seeded states.  Reads lines "dim mu mach jump dt count seed"; prints the
// largest error per line in units of its bound: values 64 eps S, their time
// derivatives 64 eps S / dt (differences of the dt / 2 and dt time integrals
// over dt^2), nodal quantities 64 eps S, with S the size of the terms summed.
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

#include "../paper_2606_17772_amd/csrc/gks_device.hpp"

template <int DIM>
static double worst(double mu, double mach, double jump, double dt, int count, int seed) {
  constexpr int N = DIM + 2;
  std::mt19937_64 rng(seed);
  auto U = [&](double a, double b) { return std::uniform_real_distribution<double>(a, b)(rng); };
  fdk::Consts k{};
  // gamma = 1.5: gamma - 1, K and their products are exact, so both forms solve the same equations
  k.gamma = 1.5;
  k.K = DIM == 2 ? 2.0 : 3.0;
  k.inv_Kd = 1.0 / (k.K + DIM);
  k.mu = mu;
  k.prfix = mu > 0 ? 0.375 : 0.0;
  k.tau_c2 = 1.0;
  const double eps = 2.3e-16;
  double w = 0.0;
  for (int it = 0; it < count; ++it) {
    fdk::GksIO<double, DIM> a;
    fdk::GksIO<LD, DIM> x;
    auto state = [&](double* W, double r, double u, double v, double p) {
      W[0] = r;
      W[1] = r * u;
      if (DIM == 2) W[2] = r * v;
      W[N - 1] = p / 0.5 + 0.5 * r * (u * u + (DIM == 2 ? v * v : 0.0));
    };
    const double r = U(0.5, 1.5), u = mach * U(-1, 1), v = mach * U(-1, 1), p = U(0.5, 1.5);
    state(a.WL, r, u, v, p);
    state(a.WR, r * (1 + jump * U(-1, 1)), u + jump * U(-1, 1), v + jump * U(-1, 1), p * (1 + jump * U(-1, 1)));
    for (int c = 0; c < N; ++c) {
      a.nL[c] = U(-1, 1);
      a.nR[c] = a.nL[c] + jump * U(-1, 1);
      a.Wt[c] = U(-1, 1);
      x.WL[c] = a.WL[c]; x.WR[c] = a.WR[c]; x.nL[c] = a.nL[c]; x.nR[c] = a.nR[c]; x.Wt[c] = a.Wt[c];
    }
    fdk::gks_iface<double, DIM, true>(k, dt, a);
    fdk::gks_iface_moments<LD, DIM, true>(k, (LD)dt, x);
    const double m = 1.0 + mach, S = 8.0 * m * m * m * m * (1.0 + mu);
    for (int c = 0; c < N; ++c) {
      const double dv[3] = {(double)(a.F[c] - x.F[c]), (double)(a.Wl[c] - x.Wl[c]), (double)(a.Wr[c] - x.Wr[c])};
      const double dd[3] = {(double)(a.Ft[c] - x.Ft[c]), (double)(a.Wlt[c] - x.Wlt[c]), (double)(a.Wrt[c] - x.Wrt[c])};
      for (int q = 0; q < 3; ++q) {
        w = std::fmax(w, std::fabs(dv[q]) / (64 * eps * S));
        w = std::fmax(w, std::fabs(dd[q]) / (64 * eps * S / dt));
      }
    }
    double f[4][4] = {};
    LD g[4][4] = {};
    fdk::gks_node<double, DIM, true>(k, a.WL, a.nL, a.Wt, f[0], f[1], f[2], f[3]);
    fdk::gks_node_moments<LD, DIM, true>(k, x.WL, x.nL, x.Wt, g[0], g[1], g[2], g[3]);
    for (int q = 0; q < 2 * DIM; ++q)
      for (int c = 0; c < N; ++c) w = std::fmax(w, std::fabs((double)(f[q][c] - g[q][c])) / (64 * eps * 8 * S));
    if (!(w == w)) return 1e300;
  }
  return w;
}

int main() {
  int dim, count, seed;
  double mu, mach, jump, dt;
  while (std::scanf("%d %lf %lf %lf %lf %d %d", &dim, &mu, &mach, &jump, &dt, &count, &seed) == 7)
    std::printf("%.3g\n", dim == 2 ? worst<2>(mu, mach, jump, dt, count, seed) : worst<1>(mu, mach, jump, dt, count, seed));
  return 0;
}
