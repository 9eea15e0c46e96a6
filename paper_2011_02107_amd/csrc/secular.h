// Roots of the secular equation of a symmetric rank-one update, for a group of lanes that share
// the sums (one wave on the GPU, one thread on the host).
#pragma once

#include <cmath>

#if defined(__HIPCC__)
#define DACP_HD __host__ __device__ __forceinline__
#else
#define DACP_HD inline
#endif

namespace dacp {

// Root j of f(lam) = 1 + rho sum_i z_i^2 / (d_i - lam) in (d_j, d_{j+1}), or in
// (d_{k-1}, d_{k-1} + rho |z|^2] for the last one; d ascending, rho > 0.  The root is returned as an
// origin org (the nearer of the two poles) and the offset tau = lam - d_org, so that
// d_i - lam = (d_i - d_org) - tau keeps full relative accuracy near the pole.
//
// Every step writes f = 1 + psi + phi, psi the terms left of the root (negative) and phi those right
// of it, interpolates each by a pole of its own, r + s / (d_j - x) and R + S / (d_{j+1} - x), through
// its value and derivative, and takes the root of the sum (a quadratic): the "middle way" of
// R.-C. Li, Solving secular equations stably and efficiently (LAPACK Working Note 89, 1994).  Five
// evaluations on average reach the rounding of f (4.7 to 5.1 on merges of random and Laplacian
// tridiagonals of 64 to 700 rows), where bisection takes over fifty.  A step that leaves
// the bracket is replaced by its midpoint; after twelve steps every other one is a bisection, so
// the bracket collapses whatever f's rounding does.  The search ends when |f| is within its
// rounding error or the offset no longer changes.
//
// Lanes: first() and stride() split the sums' index range, sum(x) adds x over the group and returns
// the same value to every lane.
template <class Lanes>
DACP_HD void secular_root(const double *d, const double *z, int k, double rho, int j, const Lanes &ln, int &org,
                          double &tau) {
  const double eps = 2.220446049250313e-16;
  const bool last = j + 1 >= k;
  double gap;
  if (last) {
    double zz = 0.0;
    for (int i = ln.first(); i < k; i += ln.stride()) zz += z[i] * z[i];
    gap = rho * ln.sum(zz);
  } else {
    gap = d[j + 1] - d[j];
  }
  int o = j;
  double t = 0.5 * gap, lo = 0.0, hi = gap;
  for (int it = 0; it < 100; ++it) {
    const double dorg = d[o];
    double psi = 0.0, phi = 0.0, dpsi = 0.0, dphi = 0.0;
    for (int i = ln.first(); i < k; i += ln.stride()) {
      const double zi = z[i];
      const double q = zi / ((d[i] - dorg) - t);
      const double w = zi * q, dw = q * q;
      if (i <= j) {
        psi += w;
        dpsi += dw;
      } else {
        phi += w;
        dphi += dw;
      }
    }
    psi = rho * ln.sum(psi);
    dpsi = rho * ln.sum(dpsi);
    if (!last) {
      phi = rho * ln.sum(phi);
      dphi = rho * ln.sum(dphi);
    }
    const double f = 1.0 + psi + phi;
    if (it == 0 && !last) {
      // f at the middle of the interval decides the nearer pole, the origin of the offset
      if (f <= 0.0) {
        o = j + 1;
        lo = -t;
        hi = 0.0;
        t = -t;
      } else {
        hi = t;
      }
    } else if (f > 0.0) {
      hi = t;
    } else {
      lo = t;
    }
    if (fabs(f) <= 2.0 * eps * (1.0 + phi - psi)) break;
    // the step: d1 < 0 < d2 are the two poles' distances from the current point
    const double d1 = (d[j] - d[o]) - t;
    double eta;
    if (last) {
      const double c = f - d1 * dpsi;
      eta = (c != 0.0) ? d1 + d1 * d1 * dpsi / c : 0.0;
    } else {
      const double d2 = (d[j + 1] - d[o]) - t;
      const double c = f - d1 * dpsi - d2 * dphi;
      const double a = (d1 + d2) * f - d1 * d2 * (dpsi + dphi);
      const double b = d1 * d2 * f;
      const double disc = sqrt(fmax(a * a - 4.0 * b * c, 0.0));
      if (a <= 0.0) eta = (c != 0.0) ? (a - disc) / (2.0 * c) : b / a;
      else eta = 2.0 * b / (a + disc);
    }
    double tn = t + eta;
    if (!(tn > lo && tn < hi) || (it >= 12 && (it & 1))) tn = 0.5 * (lo + hi);
    if (tn == t || !(tn > lo && tn < hi)) break;
    t = tn;
  }
  org = o;
  tau = t;
}

}  // namespace dacp
