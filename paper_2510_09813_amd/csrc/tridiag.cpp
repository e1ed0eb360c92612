// Host FP64 part of the Krylov exponential (Sec. III.A): exp(-i tau T) e_1 for the Lanczos
// tridiagonal T.
//
// T is diagonalised by implicit symmetric QR steps with a Wilkinson shift, chasing the bulge
// with Givens rotations (Golub & Van Loan, "Matrix Computations", Sec. 8.3).  T stays small
// (at most 64 x 64), so the active block is kept as a dense matrix and every rotation
// updates only the rows and columns it touches inside the band.  With T = Q diag(l) Q^T:
//   y = Q exp(-i tau diag(l)) Q^T e_1,  y_j = sum_k Q[j][k] exp(-i tau l_k) Q[0][k].
// The Lanczos driver takes y from tridiag_expm_series; the eigenvectors serve spectra too wide for it
// and the public call.  tridiag_expm_last (rows 0 and m-1 of Q only) is kept as a check of both: it
// gives |y_{m-1}| by another path.
#include <cfloat>
#include <cmath>

#include "rsv_internal.h"

namespace rsv {

size_t tridiag_work_doubles(int m) { return (size_t)2 * m * m + 2 * (size_t)m; }

namespace {

// c, s with  c*x - s*z = r  and  s*x + c*z = 0.
inline void givens(double x, double z, double& c, double& s) {
  if (z == 0.0) {
    c = 1.0;
    s = 0.0;
  } else if (std::fabs(z) > std::fabs(x)) {
    const double t = -x / z;
    s = 1.0 / std::sqrt(1.0 + t * t);
    c = s * t;
  } else {
    const double t = -z / x;
    c = 1.0 / std::sqrt(1.0 + t * t);
    s = c * t;
  }
}

inline bool negligible(double off, double d0, double d1) {
  return std::fabs(off) <= DBL_EPSILON * (std::fabs(d0) + std::fabs(d1)) ||
         std::fabs(off) < DBL_MIN;
}

// Eigenvalues into the diagonal of t (m x m), eigenvectors into the columns of q.  With
// all_rows false only rows 0 and m-1 of q are kept up to date.
int tridiag_eig(int m, const double* alpha, const double* beta, double* t, double* q,
                bool all_rows) {
  for (int i = 0; i < m * m; ++i) t[i] = q[i] = 0.0;
  for (int i = 0; i < m; ++i) {
    t[i * m + i] = alpha[i];
    q[i * m + i] = 1.0;
    if (i + 1 < m) t[i * m + i + 1] = t[(i + 1) * m + i] = beta[i];
  }
  auto T = [&](int i, int j) -> double& { return t[i * m + j]; };
  auto rotate_q = [&](int i, int k, double c, double s) {
    const double a0 = q[i * m + k], a1 = q[i * m + k + 1];
    q[i * m + k] = c * a0 - s * a1;
    q[i * m + k + 1] = s * a0 + c * a1;
  };

  int hi = m - 1, iter = 0;
  while (hi > 0) {
    if (negligible(T(hi, hi - 1), T(hi - 1, hi - 1), T(hi, hi))) {
      T(hi, hi - 1) = T(hi - 1, hi) = 0.0;
      --hi;
      iter = 0;
      continue;
    }
    int lo = hi - 1;
    while (lo > 0 && !negligible(T(lo, lo - 1), T(lo - 1, lo - 1), T(lo, lo))) --lo;
    if (lo > 0) T(lo, lo - 1) = T(lo - 1, lo) = 0.0;
    if (++iter > 100) return -2;

    // Wilkinson shift: eigenvalue of the trailing 2x2 block closer to T(hi, hi)
    const double d = 0.5 * (T(hi - 1, hi - 1) - T(hi, hi));
    const double b = T(hi, hi - 1);
    const double den = d + std::copysign(std::hypot(d, b), d == 0.0 ? 1.0 : d);
    const double mu = T(hi, hi) - b * b / den;

    double x = T(lo, lo) - mu, z = T(lo + 1, lo);
    for (int k = lo; k < hi; ++k) {
      double c, s;
      givens(x, z, c, s);
      const int j0 = k > lo ? k - 1 : lo;
      const int j1 = k + 2 < hi ? k + 2 : hi;
      for (int j = j0; j <= j1; ++j) {  // rows k, k+1 of G^T T
        const double a0 = T(k, j), a1 = T(k + 1, j);
        T(k, j) = c * a0 - s * a1;
        T(k + 1, j) = s * a0 + c * a1;
      }
      for (int i = j0; i <= j1; ++i) {  // columns k, k+1 of (G^T T) G
        const double a0 = T(i, k), a1 = T(i, k + 1);
        T(i, k) = c * a0 - s * a1;
        T(i, k + 1) = s * a0 + c * a1;
      }
      if (all_rows) {
        for (int i = 0; i < m; ++i) rotate_q(i, k, c, s);  // Q <- Q G
      } else {
        rotate_q(0, k, c, s);
        if (m > 1) rotate_q(m - 1, k, c, s);
      }
      if (k + 1 < hi) {
        x = T(k + 1, k);
        z = T(k + 2, k);
      }
    }
  }
  return 0;
}

}  // namespace

// work: 2*m*m + 2*m doubles.
int tridiag_expm(int m, const double* alpha, const double* beta, double tau, double* y_re,
                 double* y_im, double* work) {
  if (m <= 0 || m > kMaxKrylov) return -1;
  double* t = work;
  double* q = work + m * m;
  const int rc = tridiag_eig(m, alpha, beta, t, q, true);
  if (rc) return rc;
  double* er = work + 2 * m * m;  // Q[0][k] exp(-i tau l_k)
  double* ei = er + m;
  for (int k = 0; k < m; ++k) {
    const double ph = -tau * t[k * m + k];
    er[k] = q[k] * std::cos(ph);
    ei[k] = q[k] * std::sin(ph);
  }
  for (int j = 0; j < m; ++j) {
    double sr = 0.0, si = 0.0;
    for (int k = 0; k < m; ++k) {
      sr += q[j * m + k] * er[k];
      si += q[j * m + k] * ei[k];
    }
    y_re[j] = sr;
    y_im[j] = si;
  }
  return 0;
}

int tridiag_expm_last(int m, const double* alpha, const double* beta, double tau,
                      double* last_abs, double* work) {
  if (m <= 0 || m > kMaxKrylov) return -1;
  double* t = work;
  double* q = work + m * m;
  const int rc = tridiag_eig(m, alpha, beta, t, q, false);
  if (rc) return rc;
  double sr = 0.0, si = 0.0;
  for (int k = 0; k < m; ++k) {
    const double ph = -tau * t[k * m + k];
    const double w = q[(m - 1) * m + k] * q[k];
    sr += w * std::cos(ph);
    si += w * std::sin(ph);
  }
  *last_abs = std::hypot(sr, si);
  return 0;
}

// The same y by the Chebyshev series of the exponential: a + 8 a^(1/3) + 20 products with T for a
// spectrum of half-width a / tau (28 rows, a = 16: 4 us, where the eigenvectors take 40), as exact
// (J_k by Miller's recurrence, Gershgorin bounds).  Wider spectra take the eigenvectors.
int tridiag_expm_series(int m, const double* alpha, const double* beta, double tau, double* y_re,
                        double* y_im, double* work) {
  if (m <= 0 || m > kMaxKrylov) return -1;
  double lo = DBL_MAX, hi = -DBL_MAX;
  for (int i = 0; i < m; ++i) {
    const double w = (i > 0 ? std::fabs(beta[i - 1]) : 0.0) + (i + 1 < m ? std::fabs(beta[i]) : 0.0);
    lo = std::fmin(lo, alpha[i] - w);
    hi = std::fmax(hi, alpha[i] + w);
  }
  const double c = 0.5 * (hi + lo), a = std::fmax(0.5 * std::fabs(tau) * (hi - lo), 0.5);
  const double terms = a + 8.0 * std::cbrt(a) + 20.0;
  constexpr int kMost = 256;
  if (!(terms < kMost)) return tridiag_expm(m, alpha, beta, tau, y_re, y_im, work);
  const int K = (int)terms, M = K + 16;
  double bes[kMost + 18];
  bes[M + 1] = 0.0;
  bes[M] = 1e-250;
  for (int k = M; k >= 1; --k) {
    bes[k - 1] = 2.0 * k / a * bes[k] - bes[k + 1];
    if (std::fabs(bes[k - 1]) > 1e250)
      for (int q = k - 1; q <= M; ++q) bes[q] *= 1e-250;
  }
  double norm = bes[0];
  for (int k = 2; k <= M; k += 2) norm += 2.0 * bes[k];
  // 2 X = 2 (T - c) |tau| / a, padded by a zero row at both ends
  const double s = 2.0 * std::fabs(tau) / a, sign = tau < 0.0 ? -1.0 : 1.0;
  double d[kMaxKrylov + 2] = {}, o[kMaxKrylov + 2] = {}, t0[kMaxKrylov + 2] = {}, t1[kMaxKrylov + 2] = {},
         yr[kMaxKrylov + 2] = {}, yi[kMaxKrylov + 2] = {};
  for (int i = 0; i < m; ++i) {
    d[i + 1] = (alpha[i] - c) * s;
    if (i + 1 < m) o[i + 1] = beta[i] * s;  // couples rows i and i + 1
  }
  t0[1] = 1.0;
  t1[1] = 0.5 * d[1];
  if (m > 1) t1[2] = 0.5 * o[1];
  yr[1] = bes[0] / norm;
  for (int k = 1; k <= K; ++k) {
    const double b = 2.0 * bes[k] / norm;
    double* y = (k & 1) ? yi : yr;
    const double w = (k & 2) ? ((k & 1) ? b : -b) : ((k & 1) ? -b : b);  // (-i)^k
    for (int i = 1; i <= m; ++i) y[i] += w * t1[i];
    for (int i = 1; i <= m; ++i)
      t0[i] = d[i] * t1[i] + o[i - 1] * t1[i - 1] + o[i] * t1[i + 1] - t0[i];
    for (int i = 1; i <= m; ++i) {
      const double v = t0[i];
      t0[i] = t1[i];
      t1[i] = v;
    }
  }
  const double pr = std::cos(tau * c), pi = -std::sin(tau * c);
  for (int i = 0; i < m; ++i) {
    const double re = yr[i + 1], im = sign * yi[i + 1];
    y_re[i] = pr * re - pi * im;
    y_im[i] = pr * im + pi * re;
  }
  return 0;
}

}  // namespace rsv
