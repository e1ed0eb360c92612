// When a growing Krylov space is worth a test of its error estimate, and how many iterations to
// queue before the next one (Lanczos and Arnoldi).
#pragma once

#include <algorithm>
#include <cmath>

namespace rsv {

// The a-priori course of the estimate |x| h_{k+1,k} |[exp(tau H_k) e_1]_k|, in log2: at most
// lead_k = |x| h_{k+1,k} prod_{i<k} tau h_{i+1,i} / (k-1)!, and for a spectrum of half-width a /
// tau below that by about exp(-a^2 / 4k) (J_k(a) against (a/2)^k / k!).  The first test, at 2^10
// times the tolerance, takes the Gershgorin half-width (up to twice the true one), later ones
// half of it, relative to the last value found.
//
// That slope is too flat where the interactions set the width (a^2 / k falls with k, but few
// amplitudes feel the far end of the spectrum): over a sweep of 18 to 21 atoms in 30 x 30 um it
// alone queued 2 to 5 % too many iterations, at 27 atoms every step to kmax = 48 for 43 needed.  So
// a test is also due where the decay found so far (its mean from |x| on, or between the last two
// tests, whichever is faster) meets the tolerance when it speeds up by `quicken`: 1.25 where an
// iteration costs about as much as a test and its round trip, 3 (the decay of all dimensions
// together never gained more between two tests) for costly vectors, whose iterations are then
// queued one at a time towards the end; at least 1 and 2 bits per iteration, for tests so early that
// there is no decay yet (27 atoms complex64).  Replayed on 284 steps of 13 to 21 atoms: 5298 iterations
// needed, 5298 queued (costly) and 5306; 5333 and 5335 by the slope alone.  On one MI355X steps 5 to
// 24 of the 27-atom sweep went from 48 iterations and 180 ms each to 43.35 and 160 (complex128), from 48
// and 93.9 ms to 39.35 and 80 (complex64); 22 atoms complex64 2.12 -> 1.88 ms.
//
// Which dimensions are tested is a function of the matrix alone, and with it the dimension found:
// neither depends on how the iterations were queued.
struct KrylovCourse {
  double tau = 0.0, lead = 0.0, lo = 1e300, hi = -1e300, below = 0.0, off = -10.0;
  double first_log = 0.0, last_log = 0.0;  // |x|, and the estimate last found
  bool costly = false, tested = false;
  int k = 0, last = 0, next = 0;           // dimensions: now, last tested, tested next at the latest

  // Iterations to queue before anything is known of the matrix; hint: the dimension of the
  // comparable previous run (0: none).  One too many costs a long vector more than a round trip.
  static int first(int hint, bool costly) { return hint <= 0 ? 6 : std::max(1, costly ? hint - 1 : hint); }

  void start(double t, double nx, bool costly_vectors) {
    *this = KrylovCourse{};
    tau = t;
    costly = costly_vectors;
    lead = first_log = last_log = std::log2(nx);
  }
  // row k - 1 of H_k: its place on the spectrum's axis and the entry below it
  void add(double diag, double beta) {
    ++k;
    lo = std::min(lo, diag - below - beta);
    hi = std::max(hi, diag + below + beta);
    if (k > 1) lead += std::log2(std::max(tau * below / (k - 1), 1e-300));
    below = beta;
  }
  double value(int at, double l) const {
    const double a = 0.5 * tau * (hi - lo) * (tested ? 0.5 : 1.0);
    return l + std::log2(std::max(below, 1e-300)) - 0.3607 * a * a / at;
  }
  bool due_at(int at, double l, double log2_tol) const {
    return (tested && at >= next) || !(value(at, l) + off > log2_tol);
  }
  bool due(double log2_tol) const { return due_at(k, lead, log2_tol); }
  // a test of dimension k that missed the tolerance
  void found(double est, double log2_tol) {
    const double l = std::log2(std::max(est, 1e-300)), quicken = costly ? 3.0 : 1.25;
    const double found_decay = std::max((first_log - l) / k, (last_log - l) / (k - last));
    const double decay = std::max(quicken * found_decay, costly ? 2.0 : 1.0);
    next = k + (int)std::min(64.0, std::max(1.0, (l - log2_tol) / decay));
    last = k;
    last_log = l;
    tested = true;
    off = l - value(k, lead) - 2.0;
  }
  // iterations until a test is due, were the couplings to stay as they are (at most `most`)
  int ahead(double log2_tol, int most) const {
    double l = lead;
    int n = 1;
    for (; n < most; ++n) {
      l += std::log2(std::max(tau * below / (k + n - 1), 1e-300));
      if (due_at(k + n, l, log2_tol)) break;
    }
    n = std::min(n, most);
    return std::max(1, costly && !tested ? n - 2 : n);
  }
};

}  // namespace rsv
