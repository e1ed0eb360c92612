// When a growing Krylov space is worth a test of its error estimate (Lanczos and Arnoldi).
#pragma once

#include <algorithm>
#include <cmath>

namespace rsv {

// The a-priori course of the estimate |x| h_{k+1,k} |[exp(tau H_k) e_1]_k|, in log2: at most
// lead_k = |x| h_{k+1,k} prod_{i<k} tau h_{i+1,i} / (k-1)!, and for a spectrum of half-width a /
// tau below that by about exp(-a^2 / 4k) (J_k(a) against (a/2)^k / k!).  The first test, at 2^10
// times the tolerance, takes the Gershgorin half-width (up to twice the true one), later ones
// half of it, relative to the last value found.  A function of the matrix alone: the dimension
// found does not depend on how the iterations were queued.
struct KrylovCourse {
  double tau = 0.0, lead = 0.0, lo = 1e300, hi = -1e300, below = 0.0, off = -10.0;
  bool tested = false;
  int k = 0;
  void start(double t, double nx) {
    *this = KrylovCourse{};
    tau = t;
    lead = std::log2(nx);
  }
  // row k - 1 of H_k: its place on the spectrum's axis and the entry below it
  void add(double diag, double beta) {
    ++k;
    lo = std::min(lo, diag - below - beta);
    hi = std::max(hi, diag + below + beta);
    if (k > 1) lead += std::log2(std::max(tau * below / (k - 1), 1e-300));
    below = beta;
  }
  double value(bool tight, int at, double l) const {
    const double a = 0.5 * tau * (hi - lo) * (tight ? 0.5 : 1.0);
    return l + std::log2(std::max(below, 1e-300)) - 0.3607 * a * a / at;
  }
  bool due(double log2_tol) const { return !(value(tested, k, lead) + off > log2_tol); }
  void found(double est) {
    off = std::log2(std::max(est, 1e-300)) - value(true, k, lead) - 2.0;
    tested = true;
  }
  // iterations until a test is due, were the couplings to stay as they are
  int ahead(double log2_tol, int most) const {
    double l = lead;
    for (int n = 1; n < most; ++n) {
      l += std::log2(std::max(tau * below / (k + n - 1), 1e-300));
      if (!(value(tested, k + n, l) + off > log2_tol)) return n;
    }
    return std::max(1, most);
  }
};

}  // namespace rsv
