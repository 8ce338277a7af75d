// The gas-kinetic solvers with and without values (stage 1 and stage 2, which
// takes time derivatives only), on seeded states in one, two and three
// dimensions: prints the number of time derivatives that differ in any bit.
// Host only (--cuda-host-only).
#include <cstdio>
#include <cstring>
#include <random>

#include "../paper_2606_17772_amd/csrc/gks3d_device.hpp"

static std::mt19937_64 rng(3);
static double U(double a, double b) { return std::uniform_real_distribution<double>(a, b)(rng); }

static fdk::Consts consts(int dim, double mu) {
  fdk::Consts k{};
  k.gamma = 1.4;
  k.K = (dim == 1 ? 3.0 - 1.4 : (dim == 2 ? 4.0 - 2.8 : 5.0 - 4.2)) / 0.4;
  k.inv_Kd = 1.0 / (k.K + dim);
  k.mu = mu;
  k.prfix = mu > 0 ? 1.0 / 0.72 - 1.0 : 0.0;
  k.tau_c2 = 1.0;
  return k;
}
static void state(int dim, double* W) {
  const double r = U(0.5, 1.5), p = U(0.5, 1.5);
  double q = 0.0;
  W[0] = r;
  for (int a = 0; a < dim; ++a) {
    const double u = U(-2, 2);
    W[1 + a] = r * u;
    q += u * u;
  }
  W[dim + 1] = p / 0.4 + 0.5 * r * q;
}
static int differ(const double* a, const double* b, int n) { return std::memcmp(a, b, n * sizeof *a) != 0; }

template <int DIM> static int planar(double mu) {
  constexpr int N = DIM + 2;
  const fdk::Consts k = consts(DIM, mu);
  fdk::GksIO<double, DIM> a;
  state(DIM, a.WL);
  state(DIM, a.WR);
  for (int c = 0; c < N; ++c) a.nL[c] = U(-1, 1), a.nR[c] = U(-1, 1), a.Wt[c] = U(-1, 1);
  fdk::GksIO<double, DIM> b = a;
  const double dt = U(1e-4, 1e-2);
  fdk::gks_iface<double, DIM, true>(k, dt, a);
  fdk::gks_iface<double, DIM, false>(k, dt, b);
  double F[4], Ft[4], G[4], Gt[4], f[4], ft[4], g[4], gt[4];
  fdk::gks_node<double, DIM, true>(k, a.WL, a.nL, a.Wt, F, Ft, G, Gt);
  fdk::gks_node<double, DIM, false>(k, a.WL, a.nL, a.Wt, f, ft, g, gt);
  return differ(a.Ft, b.Ft, N) + differ(a.Wlt, b.Wlt, N) + differ(a.Wrt, b.Wrt, N) + differ(Ft, ft, N) +
         (DIM == 2 ? differ(Gt, gt, N) : 0);
}
static int volume(double mu) {
  const fdk::Consts k = consts(3, mu);
  fdk3::GksIO3 a;
  state(3, a.WL);
  state(3, a.WR);
  for (int c = 0; c < 5; ++c) a.nL[c] = U(-1, 1), a.nR[c] = U(-1, 1), a.Wt[c] = U(-1, 1), a.Wt2[c] = U(-1, 1);
  fdk3::GksIO3 b = a;
  const double dt = U(1e-4, 1e-2);
  fdk3::gks_iface<true>(k, dt, a);
  fdk3::gks_iface<false>(k, dt, b);
  double F[3][5], Ft[3][5], f[3][5], ft[3][5];
  fdk3::gks_node<true>(k, a.WL, a.nL, a.Wt, a.Wt2, F, Ft);
  fdk3::gks_node<false>(k, a.WL, a.nL, a.Wt, a.Wt2, f, ft);
  return differ(a.Ft, b.Ft, 5) + differ(a.Wlt, b.Wlt, 5) + differ(a.Wrt, b.Wrt, 5) + differ(Ft[0], ft[0], 15);
}

int main() {
  int n[3] = {};
  for (int it = 0; it < 2000; ++it)
    for (double mu : {0.0, 1e-3}) {
      n[0] += planar<1>(mu);
      n[1] += planar<2>(mu);
      n[2] += volume(mu);
    }
  std::printf("%d %d %d\n", n[0], n[1], n[2]);
  return 0;
}
