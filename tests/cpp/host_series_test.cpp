// The series forms of the host exponentials (csrc/tridiag.cpp: tridiag_expm_series,
// csrc/dense_expm.cpp: hess_expm_e1), built with the sanitizers and checked against the forms they stand
// in for: eigenvectors of the tridiagonal matrix, Pade approximant of the whole Hessenberg matrix.
// Widths on both sides of the number of terms where the series give way, both signs of the time, rows
// 1..64, leading dimensions above the size.  Prints "host_series ok" when every check holds.
#include <cmath>
#include <complex>
#include <cstdio>
#include <random>
#include <vector>

namespace rsv {
int tridiag_expm(int m, const double* alpha, const double* beta, double tau, double* y_re,
                 double* y_im, double* work);
int tridiag_expm_series(int m, const double* alpha, const double* beta, double tau, double* y_re,
                        double* y_im, double* work);
size_t tridiag_work_doubles(int m);
int dense_expm(int m, const std::complex<double>* a, std::complex<double>* out);
int hess_expm_e1(int m, const std::complex<double>* a, int ld, double tau, std::complex<double>* y);
}  // namespace rsv

int main() {
  using cd = std::complex<double>;
  std::mt19937_64 gen(9813);
  std::uniform_real_distribution<double> u(-1.0, 1.0);
  int failures = 0;
  auto check = [&](bool ok, const char* what, int m, double v) {
    if (!ok) {
      std::printf("FAIL %s m=%d value=%.3e\n", what, m, v);
      ++failures;
    }
  };
  // widest arguments a with a + 8 a^(1/3) + 20 below 256 (tridiagonal) and 600 (Hessenberg)
  auto widest = [](double terms) {
    double a = terms;
    for (int i = 0; i < 200; ++i) a = terms - 20.0 - 8.0 * std::cbrt(a);
    return a;
  };
  for (int m = 1; m <= 64; ++m) {
    for (const double a : {1e-3, 0.4, 5.0, 60.0, widest(256.0) * (1 - 1e-9), widest(256.0) * (1 + 1e-9), 400.0}) {
      std::vector<double> al(m), be(m), yr(m), yi(m), zr(m), zi(m), work(rsv::tridiag_work_doubles(m));
      double lo = 1e300, hi = -1e300;
      for (int i = 0; i < m; ++i) {
        al[i] = u(gen) + 3.0;
        be[i] = 0.05 + std::fabs(u(gen));
      }
      if (m == 1) al[0] = 0.7;  // no width at all
      for (int i = 0; i < m; ++i) {
        const double w = (i > 0 ? be[i - 1] : 0.0) + (i + 1 < m ? be[i] : 0.0);
        lo = std::fmin(lo, al[i] - w);
        hi = std::fmax(hi, al[i] + w);
      }
      const double tau = m == 1 ? a : 2.0 * a / (hi - lo);  // the series' argument is a
      for (const double t : {tau, -tau}) {
        check(rsv::tridiag_expm_series(m, al.data(), be.data(), t, yr.data(), yi.data(), work.data()) == 0,
              "series status", m, a);
        check(rsv::tridiag_expm(m, al.data(), be.data(), t, zr.data(), zi.data(), work.data()) == 0,
              "eigenvectors status", m, a);
        double err = 0.0;
        for (int i = 0; i < m; ++i) err = std::fmax(err, std::hypot(yr[i] - zr[i], yi[i] - zi[i]));
        // phases tau lambda of up to 5 a radians and their eigenvalues' rounding, 256 terms
        check(err <= 1e-13 * (1.0 + a), "series against eigenvectors", m, err);
      }
    }
  }
  for (const int m : {1, 2, 3, 12, 28, 62, 63}) {
    for (const double a : {1e-3, 2.0, 40.0, widest(600.0) * 0.999, widest(600.0) * 1.001}) {
      for (const double loss : {0.0, 0.01, 3.0}) {
        const int ld = m + 3;
        std::vector<cd> h((size_t)ld * m, cd(0.0)), full((size_t)m * m), e((size_t)m * m), y(m);
        double lo = 1e300, hi = -1e300;
        for (int i = 0; i < m; ++i) {
          h[(size_t)i * ld + i] = cd(-loss * std::fabs(u(gen)), u(gen));
          if (i + 1 < m) {
            const double b = 0.1 + std::fabs(u(gen));
            h[(size_t)(i + 1) * ld + i] = b;
            h[(size_t)i * ld + i + 1] = -b;
          }
        }
        for (int i = 0; i < m; ++i) {
          const double w = (i > 0 ? std::abs(h[(size_t)i * ld + i - 1]) : 0.0) +
                           (i + 1 < m ? std::abs(h[(size_t)i * ld + i + 1]) : 0.0);
          lo = std::fmin(lo, h[(size_t)i * ld + i].imag() - w);
          hi = std::fmax(hi, h[(size_t)i * ld + i].imag() + w);
        }
        const double tau = m == 1 ? a : 2.0 * a / (hi - lo);
        for (int i = 0; i < m; ++i)
          for (int j = 0; j < m; ++j) full[(size_t)i * m + j] = tau * h[(size_t)i * ld + j];
        check(rsv::hess_expm_e1(m, h.data(), ld, tau, y.data()) == 0, "hess status", m, a);
        check(rsv::dense_expm(m, full.data(), e.data()) == 0, "dense status", m, a);
        double err = 0.0;
        for (int i = 0; i < m; ++i) err = std::fmax(err, std::abs(y[i] - e[(size_t)i * m]));
        // the squared Pade approximant's rounding grows with the norm it squares away (2 a at most
        // here, times the loss); the series sums 600 terms of size e^2 at most
        check(err <= 1e-12 + 1e-14 * a * (1.0 + loss), "hess column", m, err);
      }
    }
  }
  if (failures == 0) std::printf("host_series ok\n");
  return failures != 0;
}
