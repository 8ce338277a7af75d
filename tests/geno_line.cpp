// The line routines that decide smooth components from one ratio
// (recon_line, recon_node_line of gks_device.hpp) against the general routine
// of each component, bit for bit: smooth lines, near ties, jumps, noise, zeros
// and extreme magnitudes, for several r, C and eps.  Also the indicators
// themselves: wherever the one-ratio test holds, geno() takes its shortcut.
// Prints one JSON line; host only (--cuda-host-only).
#include <cmath>
#include <cstdio>
#include <cstring>
#include <random>

#include "../paper_2606_17772_amd/csrc/gks_device.hpp"

using fdk::Consts;

int main() {
  std::mt19937_64 rng(7);
  std::uniform_real_distribution<double> U(-1.0, 1.0);
  long total = 0, quick = 0, differ = 0, fired = 0, wrong = 0;
  const double Cs[] = {20.0, 40.0, 10.0}, epss[] = {1e-15, 1e-6, 1e-40, 1e-120, 0.0};
  for (int r = 1; r <= 8; ++r)
    for (double C : Cs)
      for (double eps : epss)
        for (int variant = 0; variant < 3; ++variant) {
          Consts k{};
          k.C = C;
          k.inv_tanhC = 1.0 / std::tanh(C);
          k.eps = eps;
          k.eps_a = 1e-6;
          k.dc = 8.0;
          k.ds = 1.0;
          k.r = r;
          k.variant = variant;
          k.geno_ratio = fdk::geno_smooth_ratio(k.C, k.inv_tanhC, k.r, k.eps);
          const double h = 0.01, invh = 1.0 / h;
          for (int n = 0; n < 1500; ++n) {
            double Q[4][4], X[4][4], Q3[4][3], X3[4][3];
            for (int c = 0; c < 4; ++c) {
              const int mode = (n + c) % 6;
              const double big = mode == 5 ? std::pow(10.0, 150.0 * U(rng)) : 1.0, a = U(rng), s = U(rng), cu = U(rng);
              for (int m = 0; m < 4; ++m) {
                const double x = (m - 1.5) * h;
                Q[c][m] = big * (1.0 + 0.1 * a + s * x + cu * x * x);
                X[c][m] = big * (s + 2.0 * cu * x);
                if (mode == 1) Q[c][m] += 1e-9 * U(rng);
                if (mode == 2 && m >= 2) Q[c][m] += 0.3 * U(rng);
                if (mode == 3) { Q[c][m] = U(rng); X[c][m] = U(rng) / h; }
                if (mode == 4) { Q[c][m] = 0.5; X[c][m] = 0.0; }
              }
              for (int m = 0; m < 3; ++m) { Q3[c][m] = Q[c][m]; X3[c][m] = X[c][m]; }
            }
            fdk::IfaceRec a[4], b[4];
            double da[4], db[4];
            fdk::recon_line<4>(k, Q, X, h, invh, a);
            fdk::recon_node_line<4>(k, Q3, X3, h, invh, da);
            for (int c = 0; c < 4; ++c) {
              b[c] = fdk::recon_iface<double>(k, Q[c][0], Q[c][1], Q[c][2], Q[c][3], X[c][0], X[c][1], X[c][2],
                                              X[c][3], h, invh);
              db[c] = fdk::recon_node<double>(k, Q3[c][0], Q3[c][1], Q3[c][2], X3[c][0], X3[c][1], X3[c][2], h, invh);
              fdk::IfaceRec q;
              quick += fdk::recon_iface_smooth(k, Q[c][0], Q[c][1], Q[c][2], Q[c][3], X[c][0], X[c][1], X[c][2],
                                               X[c][3], h, invh, q);
              ++total;
            }
            differ += std::memcmp(a, b, sizeof a) != 0;
            differ += std::memcmp(da, db, sizeof da) != 0;
            // the forms that read the line again and evaluate both sides in one run
            fdk::recon_line_compact<4>(
                k, Q, X,
                [&](int c, double (&q)[4], double (&x)[4]) {
                  for (int m = 0; m < 4; ++m) { q[m] = Q[c][m]; x[m] = X[c][m]; }
                },
                h, invh, a);
            fdk::recon_node_compact<4>(
                k, Q3, X3,
                [&](int c, double (&q)[3], double (&x)[3]) {
                  for (int m = 0; m < 3; ++m) { q[m] = Q3[c][m]; x[m] = X3[c][m]; }
                },
                h, invh, da);
            auto same = [](double u, double v) { return std::memcmp(&u, &v, sizeof u) == 0 || (u != u && v != v); };
            for (int c = 0; c < 4; ++c)
              differ += !(same(a[c].vl, b[c].vl) && same(a[c].dl, b[c].dl) && same(a[c].cl, b[c].cl) &&
                          same(a[c].vr, b[c].vr) && same(a[c].dr, b[c].dr) && same(a[c].cr, b[c].cr) &&
                          same(da[c], db[c]));
            // indicator triples over the whole double range
            double IS[3];
            for (int t = 0; t < 3; ++t) {
              IS[t] = std::pow(10.0, n % 2 ? -20.0 + 12.0 * U(rng) : 300.0 * U(rng));
              if (n % 3 == 1 && t > 0) IS[t] = IS[0] * (1.0 + 0.5 * U(rng));
              if (n % 5 == 4 && t == 2) IS[t] = 2.0 * IS[0] - IS[1] > 0.0 ? 2.0 * IS[0] - IS[1] : 0.0;
            }
            if (fdk::geno_smooth<double>(k, IS[0], IS[1], IS[2])) {
              ++fired;
              const auto o = fdk::geno<double>(k, IS[0], IS[1], IS[2], 0.1, 0.8, 0.1, 1.1, 2.3, 3.7, 4.1, 5.3, 6.7,
                                               7.0, 8.0);
              wrong += !(o.v == 7.0 && o.d == 8.0 && o.chi == 1.0);
            }
          }
        }
  std::printf("{\"total\": %ld, \"quick\": %ld, \"differ\": %ld, \"fired\": %ld, \"wrong\": %ld}\n", total, quick,
              differ, fired, wrong);
  return 0;
}
