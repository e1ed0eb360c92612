// exp(A) of a small dense complex matrix, host FP64: scaling and squaring with the diagonal
// [6/6] Pade approximant (Golub & Van Loan, "Matrix Computations", Sec. 11.3, Algorithm
// 11.3.1): A is scaled by 2^-j with j = max(0, 1 + floor(log2 |A|_inf)), so |A/2^j|_inf <= 1/2,
// where the [6/6] approximant's relative backward error is below 1e-16; N(A) and D(A) are
// summed term by term, D F = N is solved by Gaussian elimination with partial pivoting, and F
// is squared j times.
//
// hess_expm_e1 is what the Arnoldi exponential of the Lindblad and gradient paths needs of its
// upper Hessenberg matrix (m <= 63): the first column only.  Where the matrix is nearly
// skew-Hermitian (unitary dynamics with weak dissipation, the usual case) that column comes from
// the Chebyshev series of the exponential, some a + 25 products with the Hessenberg matrix for a
// spectrum of half-width a (28 vectors: about 0.1 ms against 1 ms for the whole exponential),
// else from dense_expm.
#include <algorithm>
#include <cmath>
#include <complex>
#include <vector>

#include "arnoldi.h"

namespace rsv {

using cd = std::complex<double>;

namespace {

void matmul(int m, const cd* a, const cd* b, cd* c) {
  for (int i = 0; i < m; ++i)
    for (int j = 0; j < m; ++j) {
      cd s = 0.0;
      for (int k = 0; k < m; ++k) s += a[i * m + k] * b[k * m + j];
      c[i * m + j] = s;
    }
}

// Solves D X = B for X (both m x m, row-major) in place in B; D is destroyed.
int solve(int m, cd* d, cd* b) {
  for (int col = 0; col < m; ++col) {
    int piv = col;
    for (int r = col + 1; r < m; ++r)
      if (std::abs(d[r * m + col]) > std::abs(d[piv * m + col])) piv = r;
    if (std::abs(d[piv * m + col]) == 0.0) return -1;
    if (piv != col)
      for (int k = 0; k < m; ++k) {
        std::swap(d[piv * m + k], d[col * m + k]);
        std::swap(b[piv * m + k], b[col * m + k]);
      }
    for (int r = col + 1; r < m; ++r) {
      const cd f = d[r * m + col] / d[col * m + col];
      if (f == 0.0) continue;
      for (int k = col; k < m; ++k) d[r * m + k] -= f * d[col * m + k];
      for (int k = 0; k < m; ++k) b[r * m + k] -= f * b[col * m + k];
    }
  }
  for (int col = m - 1; col >= 0; --col) {
    for (int k = 0; k < m; ++k) b[col * m + k] /= d[col * m + col];
    for (int r = 0; r < col; ++r) {
      const cd f = d[r * m + col];
      if (f == 0.0) continue;
      for (int k = 0; k < m; ++k) b[r * m + k] -= f * b[col * m + k];
    }
  }
  return 0;
}

}  // namespace

int dense_expm(int m, const cd* a, cd* out) {
  if (m < 1) return -1;
  double norm = 0.0;  // infinity norm
  for (int i = 0; i < m; ++i) {
    double s = 0.0;
    for (int j = 0; j < m; ++j) s += std::abs(a[i * m + j]);
    norm = std::max(norm, s);
  }
  if (!std::isfinite(norm)) return -1;
  int j = 0;
  if (norm > 0.0) j = std::max(0, 1 + (int)std::floor(std::log2(norm)));
  const double scale = std::ldexp(1.0, -j);
  const size_t mm = (size_t)m * m;
  std::vector<cd> as(mm), x(mm), t(mm), num(mm), den(mm);
  for (size_t i = 0; i < mm; ++i) as[i] = a[i] * scale;
  for (int i = 0; i < m; ++i)
    for (int k = 0; k < m; ++k) {
      const cd e = (i == k) ? 1.0 : 0.0;
      x[i * m + k] = e;
      num[i * m + k] = e;
      den[i * m + k] = e;
    }
  const int q = 6;
  double c = 1.0;
  for (int k = 1; k <= q; ++k) {
    c = c * (q - k + 1) / ((2.0 * q - k + 1) * k);
    matmul(m, as.data(), x.data(), t.data());
    x.swap(t);
    const double sgn = (k % 2) ? -1.0 : 1.0;
    for (size_t i = 0; i < mm; ++i) {
      num[i] += c * x[i];
      den[i] += sgn * c * x[i];
    }
  }
  if (solve(m, den.data(), num.data()) != 0) return -1;
  for (int s = 0; s < j; ++s) {
    matmul(m, num.data(), num.data(), t.data());
    num.swap(t);
  }
  for (size_t i = 0; i < mm; ++i) out[i] = num[i];
  return 0;
}

// A = tau a = c + i r X with X's spectrum in [-1, 1] up to a non-Hermitian part of norm delta:
// exp(A) = e^c (J_0(r) + 2 sum_k i^k J_k(r) T_k(X)).  |T_k(X)| is at most about exp(k
// asinh(delta / r)); the series is used while that stays below e^2 over its terms.
int hess_expm_e1(int m, const cd* a, int ld, double tau, cd* y) {
  if (m < 1) return -1;
  double slo = 1e300, shi = -1e300, dlo = 1e300, dhi = -1e300;  // Gershgorin, skew and Hermitian part
  for (int i = 0; i < m; ++i) {
    double s = 0.0, d = 0.0;
    for (int j = 0; j < m; ++j) {
      if (j == i) continue;
      const cd u = j >= i - 1 ? a[i * ld + j] : 0.0, l = i >= j - 1 ? std::conj(a[j * ld + i]) : 0.0;
      s += 0.5 * std::hypot(u.real() - l.real(), u.imag() - l.imag());
      d += 0.5 * std::hypot(u.real() + l.real(), u.imag() + l.imag());
    }
    const cd g = a[i * ld + i];
    slo = std::min(slo, g.imag() - s);
    shi = std::max(shi, g.imag() + s);
    dlo = std::min(dlo, g.real() - d);
    dhi = std::max(dhi, g.real() + d);
  }
  const double r = std::max(0.5 * tau * (shi - slo), 0.5);
  const cd c(0.5 * tau * (dlo + dhi), 0.5 * tau * (slo + shi));
  if (!std::isfinite(r) || !std::isfinite(c.real()) || !std::isfinite(c.imag())) return -1;
  const double kd = r + 8.0 * std::cbrt(r) + 20.0, delta = 0.5 * tau * (dhi - dlo);
  if (kd > 600.0 || kd * std::asinh(delta / r) > 2.0) {
    std::vector<cd> full((size_t)m * m), e((size_t)m * m);
    for (int i = 0; i < m; ++i)
      for (int j = 0; j < m; ++j) full[i * m + j] = tau * a[i * ld + j];
    if (dense_expm(m, full.data(), e.data()) != 0) return -1;
    for (int i = 0; i < m; ++i) y[i] = e[i * m];
    return 0;
  }
  // J_k(r) by Miller's backward recurrence
  const int K = (int)kd, M = K + 24;
  std::vector<double> bes(M + 2, 0.0);
  double norm = 0.0;
  bes[M] = 1e-250;
  for (int k = M; k >= 1; --k) {
    bes[k - 1] = 2.0 * k / r * bes[k] - bes[k + 1];
    if (std::fabs(bes[k - 1]) > 1e250)
      for (int q = k - 1; q <= M; ++q) bes[q] *= 1e-250;
  }
  for (int k = 2; k <= M; k += 2) norm += 2.0 * bes[k];
  norm += bes[0];
  // columns of 2 X = 2 (tau a - c) / (i r), real and imaginary parts apart
  std::vector<double> xr((size_t)m * m, 0.0), xi((size_t)m * m, 0.0), v((size_t)8 * m, 0.0);
  for (int j = 0; j < m; ++j)
    for (int i = 0; i <= std::min(j + 1, m - 1); ++i) {
      const cd z = (tau * a[i * ld + j] - (i == j ? c : 0.0)) * cd(0.0, -2.0 / r);
      xr[(size_t)j * m + i] = z.real();
      xi[(size_t)j * m + i] = z.imag();
    }
  double *t0r = v.data(), *t0i = t0r + m, *t1r = t0i + m, *t1i = t1r + m, *t2r = t1i + m, *t2i = t2r + m,
         *yr = t2i + m, *yi = yr + m;
  t0r[0] = 1.0;
  for (int i = 0; i < std::min(2, m); ++i) {  // T_1 e_1 = X e_1
    t1r[i] = 0.5 * xr[i];
    t1i[i] = 0.5 * xi[i];
  }
  yr[0] = bes[0] / norm;
  int top = std::min(2, m);  // entries of t1 that are not zero
  for (int k = 1; k <= K; ++k) {
    const double b = 2.0 * bes[k] / norm;
    const double br = (k & 3) == 0 ? b : (k & 3) == 2 ? -b : 0.0, bi = (k & 3) == 1 ? b : (k & 3) == 3 ? -b : 0.0;
    for (int i = 0; i < top; ++i) {
      yr[i] += br * t1r[i] - bi * t1i[i];
      yi[i] += br * t1i[i] + bi * t1r[i];
    }
    const int n2 = std::min(top + 1, m);
    for (int i = 0; i < n2; ++i) {
      t2r[i] = -t0r[i];
      t2i[i] = -t0i[i];
    }
    for (int j = 0; j < top; ++j) {
      const double p = t1r[j], q = t1i[j];
      const double *cr = &xr[(size_t)j * m], *ci = &xi[(size_t)j * m];
      const int len = std::min(j + 2, m);
      for (int i = 0; i < len; ++i) {
        t2r[i] += cr[i] * p - ci[i] * q;
        t2i[i] += cr[i] * q + ci[i] * p;
      }
    }
    std::swap(t0r, t1r);
    std::swap(t0i, t1i);
    std::swap(t1r, t2r);
    std::swap(t1i, t2i);
    top = n2;
  }
  const cd ec = std::exp(c);
  for (int i = 0; i < m; ++i) y[i] = ec * cd(yr[i], yi[i]);
  return 0;
}

}  // namespace rsv
