// The secular equation's roots (secular.h, one thread for a wave's lanes) against long double: each lies in its
// interval, and there f vanishes to the rounding of its own evaluation, (k + 10) eps (1 + |psi| + |phi|), or
// changes sign within four units of the offset's last place.
#include <algorithm>
#include <cmath>
#include <cstdio>
#include <random>
#include <vector>

#include "secular.h"

namespace {
int g_fail = 0;

struct OneLane {
  int first() const { return 0; }
  int stride() const { return 1; }
  double sum(double v) const { return v; }
};

// f at d[org] + tau, and 1 + |psi| + |phi|
long double f_at(const std::vector<double> &d, const std::vector<double> &z, double rho, int org, long double tau,
                 long double *size = nullptr) {
  long double s = 0, a = 0;
  for (size_t i = 0; i < d.size(); ++i) {
    const long double t = static_cast<long double>(z[i]) * z[i] / ((static_cast<long double>(d[i]) - d[org]) - tau);
    s += t;
    a += std::fabs(t);
  }
  if (size) *size = 1 + rho * a;
  return 1 + rho * s;
}

void problem(const char *what, const std::vector<double> &d, std::vector<double> z, double rho) {
  const int k = static_cast<int>(d.size());
  long double zz = 0;
  for (double x : z) zz += static_cast<long double>(x) * x;
  for (int j = 0; j < k; ++j) {
    int org = -1;
    double tau = NAN;
    dacp::secular_root(d.data(), z.data(), k, rho, j, OneLane(), org, tau);
    const long double lam = static_cast<long double>(d[std::max(org, 0)]) + tau;
    const long double end = j + 1 < k ? static_cast<long double>(d[j + 1]) : d[j] + rho * zz * (1 + 1e-15L);
    bool ok = (org == j || (org == j + 1 && j + 1 < k)) && lam >= d[j] && lam <= end && tau != 0.0 &&
              (org == j ? tau > 0 : tau < 0);
    if (ok) {
      long double size = 0;
      const long double eps = 2.220446049250313e-16L, f = f_at(d, z, rho, org, tau, &size), t = tau;
      const long double lo = f_at(d, z, rho, org, t - 4 * eps * std::fabs(t)), hi = f_at(d, z, rho, org, t + 4 * eps * std::fabs(t));
      ok = std::fabs(f) <= (k + 10) * eps * size || (lo <= 0 && hi >= 0);
    }
    if (!ok && g_fail++ < 20)
      std::fprintf(stderr, "FAIL: %s, k %d root %d: origin %d offset %.17g\n", what, k, j, org, tau);
  }
}
}  // namespace

int main() {
  std::mt19937_64 rng(7);
  std::uniform_real_distribution<double> u(0.0, 1.0);
  for (double rho : {1e-12, 0.3, 1.0, 40.0, 1e12}) {
    problem("one pole", {0.7}, {1.0}, rho);
    problem("two poles", {-1.0, 1.0}, {0.6, 0.8}, rho);
    problem("a tiny z", {-1.0, 0.0, 1.0}, {0.6, 1e-9, 0.8}, rho);
    problem("two tiny z", {0.0, 1.0, 2.0, 3.0}, {1e-8, 1.0, 1e-8, 1e-8}, rho);
  }
  for (int t = 0; t < 400; ++t) {
    const int k = 2 + static_cast<int>(rng() % 60);
    std::vector<double> d(k), z(k);
    for (double &x : d) x = 2 * u(rng) - 1;
    if (t % 4 == 1)  // clusters a few hundred eps apart, as deflation leaves them
      for (int i = 1; i < k; ++i) d[i] = (i % 7) ? d[i - 1] + 1e-13 * (1 + u(rng)) : u(rng) * 2 - 1;
    if (t % 4 == 2)  // graded over 12 decades
      for (double &x : d) x = std::pow(10.0, -12 * u(rng));
    std::sort(d.begin(), d.end());
    for (int i = 1; i < k; ++i)
      if (!(d[i] > d[i - 1] + 1e-14 * std::fabs(d[i]))) d[i] = d[i - 1] + 1e-13 * (1 + std::fabs(d[i - 1]));
    double n = 0;
    for (double &x : z) {
      x = (t % 3 == 2) ? std::pow(10.0, -7 * u(rng)) : 2 * u(rng) - 1;
      n += x * x;
    }
    for (double &x : z) x /= std::sqrt(n);
    problem("random", d, z, t % 5 == 4 ? std::pow(10.0, 12 * u(rng) - 6) : 0.1 + u(rng));
  }
  std::printf("%d failures\n", g_fail);
  return g_fail != 0;
}
