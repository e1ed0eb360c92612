// Replays of csrc/krylov_course.h on stored Lanczos coefficients, with the estimate from
// csrc/tridiag.cpp: the dimensions found and the iterations queued, for costly and cheap vectors,
// where the length of the first queue comes from the run before (hint) or is 1 or kmax.
// Input (argv[1]): the number of runs, then per run a line "series run norm tau tol kmax need" and
// the kmax alphas and betas.  Prints one line per run: "series run need", and for (costly, cheap) x
// (hint, 1, kmax) "dimension queued".
#include <cmath>
#include <cstdio>
#include <map>
#include <vector>

#include "krylov_course.h"

namespace rsv {
int tridiag_expm_series(int m, const double* alpha, const double* beta, double tau, double* y_re,
                        double* y_im, double* work);
size_t tridiag_work_doubles(int m);
}  // namespace rsv

int main(int argc, char** argv) {
  std::FILE* f = argc > 1 ? std::fopen(argv[1], "r") : nullptr;
  int runs = 0;
  if (!f || std::fscanf(f, "%d", &runs) != 1) return 1;
  std::map<std::pair<int, std::pair<int, int>>, int> hints;  // (policy, (series, run)) -> dimension
  for (int i = 0; i < runs; ++i) {
    int series, run, kmax, need;
    double norm, tau, tol;
    if (std::fscanf(f, "%d %d %lf %lf %lf %d %d", &series, &run, &norm, &tau, &tol, &kmax, &need) != 7)
      return 1;
    std::vector<double> al(kmax), be(kmax), yr(kmax), yi(kmax), work(rsv::tridiag_work_doubles(kmax));
    for (double& x : al)
      if (std::fscanf(f, "%lf", &x) != 1) return 1;
    for (double& x : be)
      if (std::fscanf(f, "%lf", &x) != 1) return 1;
    std::printf("%d %d %d", series, run, need);
    const double log2_tol = std::log2(tol);
    for (int policy = 0; policy < 6; ++policy) {
      const bool costly = policy < 3;
      int& hint = hints[{policy, {series, run}}];
      auto meets = [&](int m, double* est) {
        if (rsv::tridiag_expm_series(m, al.data(), be.data(), tau, yr.data(), yi.data(), work.data()) != 0)
          return false;
        *est = be[m - 1] * std::hypot(yr[m - 1], yi[m - 1]) * norm;
        return *est <= tol;
      };
      rsv::KrylovCourse course;
      course.start(tau, norm, costly);
      int m = 0, upto = 0, found = 0;
      int next = policy % 3 == 0 ? rsv::KrylovCourse::first(hint, costly) : policy % 3 == 1 ? 1 : kmax;
      while (!found) {
        if (next < 1) return 2;
        upto = m + next < kmax ? m + next : kmax;
        for (int k = m + 1; k <= upto && !found; ++k) {
          m = k;
          course.add(al[k - 1], be[k - 1]);
          if (k < kmax && !course.due(log2_tol)) continue;
          double est = 0.0;
          if (meets(k, &est)) {
            while (m > 1 && meets(m - 1, &est)) --m;
            found = m;
          } else {
            course.found(est, log2_tol);
            if (k == kmax) found = kmax;
          }
        }
        if (!found) next = course.ahead(log2_tol, kmax - m);
      }
      hint = found;
      std::printf(" %d %d", found, upto);
    }
    std::printf("\n");
  }
  std::fclose(f);
  std::printf("replay ok\n");
  return 0;
}
