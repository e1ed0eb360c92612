// Arnoldi Krylov exponential on device vectors, driven from the host (see arnoldi.h).
//
// Iterations are queued several at a time (as many as the previous run took, or as the decay of
// the a-priori estimate suggests) and their Hessenberg columns fetched together; the host then
// goes through them in order.  What it decides (a second Gram-Schmidt pass, the dimension that
// meets the tolerance) depends on the columns alone, not on how they were queued: columns after a
// vector that needs a second pass are computed again, columns beyond the final dimension ignored.
#include "arnoldi.h"

#include <algorithm>
#include <cmath>
#include <cstring>

namespace rsv {

namespace {

using cd = std::complex<double>;
size_t up256(size_t b) { return (b + 255) / 256 * 256; }

// dscal: |u_i|^2, the diagonal of H as the device has it, the second pass's inner products, then
// column j's 2 (j + 2) values.
constexpr size_t kNorms = kMaxKrylov + 2, kDiag = kNorms, kAgain = kDiag + 2 * (kMaxKrylov + 2),
                 kCols = kAgain + 2 * (kMaxKrylov + 2);
inline size_t col_off(int j) { return kCols + (size_t)j * j + 3 * (size_t)j; }

struct Run {
  const OpFn& op;
  ArnoldiSpace& sp;
  void* d_x;
  hipStream_t s;
  rsv_stats* st;
  size_t count;
  bool small;
  int parts;

  void* vec(int i) const { return i == 0 ? d_x : (void*)(sp.base + (size_t)i * sp.vb); }

  ArnoldiStep step(int j, bool again) const {
    ArnoldiStep a{};
    a.j = j;
    a.again = again;
    a.v0 = d_x;
    a.base = sp.base;
    a.stride = sp.vb / amp_bytes(sp.prec);
    a.count = count;
    a.w = again ? vec(j + 1) : (void*)sp.base;
    a.herm = sp.herm;
    a.shift = sp.shift ? 1 : 0;
    a.nrm2 = sp.dscal;
    a.diag = sp.dscal + kDiag;
    a.npart = sp.npart;
    a.nparts = !again && small && j > 0 ? parts : 0;
    a.part = sp.part;
    a.dparts = small ? parts : 0;
    a.dots = sp.dscal + (again ? kAgain : col_off(j));
    a.npart_out = sp.npart;
    return a;
  }
  // One Gram-Schmidt pass; long vectors sum their partials in launches of their own.
  int orthogonalise(int j, bool again) {
    const ArnoldiStep a = step(j, again);
    HIP_TRY(arnoldi_dots(sp.prec, a, s));
    if (!small) HIP_TRY(finalize_rows(sp.part, parts, (sp.herm ? 1 : 2) * (j + 2), a.dots, s));
    HIP_TRY(arnoldi_update(sp.prec, a, s));
    if (!small) HIP_TRY(finalize_sum(sp.npart, parts, sp.dscal + j + 1, s));
    return RSV_OK;
  }
  int iterate(int j) {
    RSV_TRY(op(vec(j), sp.base, s));
    st->krylov_iters += 1;
    return orthogonalise(j, false);
  }
  // |u_upto|^2 and everything up to column upto - 1 (or the second pass's inner products).
  int fetch(int upto) {
    if (small) HIP_TRY(arnoldi_norm(sp.npart, parts, sp.dscal + upto, s));
    HIP_TRY(hipMemcpyAsync(sp.h_scal, sp.dscal, col_off(upto) * sizeof(double),
                           hipMemcpyDeviceToHost, s));
    HIP_TRY(hipStreamSynchronize(s));
    return RSV_OK;
  }
};

// x <- exp(sub Op) x for the largest sub <= tau found that kmax vectors resolve.
int expm_part(const OpFn& op, ArnoldiSpace& sp, ArnoldiSpace::Last& last, void* d_x, double tau, double tol,
              int max_depth, hipStream_t s, rsv_stats* st, double* sub) {
  const int kmax = sp.kmax;
  const size_t count = size_t(1) << sp.nb;
  Run run{op, sp, d_x, s, st, count, count <= (size_t(1) << kSmallBits), arnoldi_parts(count)};
  *sub = tau;
  HIP_TRY(norm2_partial(sp.prec, sp.nb, d_x, sp.part, s));
  HIP_TRY(finalize_sum(sp.part, vec_num_partials(sp.prec, sp.nb), sp.dscal, s));
  std::vector<cd> h((size_t)(kmax + 1) * kmax, 0.0), y(kmax);  // h[i * kmax + j], i <= j + 1
  auto H = [&](int i, int j) -> cd& { return h[(size_t)i * kmax + j]; };
  std::vector<double> scale(kmax + 1, 0.0);
  const double* sc = sp.h_scal;
  const double log2_tol = std::log2(tol);
  KrylovCourse course;
  double nx = 0.0;
  // What is queued behind a vector that needs a second pass is computed again.  The same columns need
  // one step after step (the gradients' second, whose diagonal entry is far from the first's; every
  // one under strong dissipation), so a queue ends with the next column that did in the comparable
  // run before.  After a surprise it goes on, after a second one a column at a time.
  const int hint = last.dim, first = KrylovCourse::first(hint, !run.small);
  const uint64_t expected = last.again;
  last.again = 0;
  int surprises = 0;
  int m = 0;  // columns gone through
  int next = first;
  auto finish = [&](int dim, double part) -> int {
    last.dim = dim;
    st->krylov_max = std::max<int64_t>(st->krylov_max, dim);
    CombineCoef cc;
    std::memset(&cc, 0, sizeof cc);
    cc.m = dim;
    for (int l = 0; l < dim; ++l) {
      const cd c = nx * scale[l] * y[l];
      cc.re[l] = c.real();
      cc.im[l] = sp.herm ? 0.0 : c.imag();  // (real there up to rounding)
      cc.x[l] = run.vec(l);
    }
    *sub = part;
    HIP_TRY(krylov_combine(sp.prec, sp.nb, cc, d_x, sp.part, s));
    return RSV_OK;
  };
  for (;;) {
    if (surprises > 1) next = 1;
    int upto = std::min(kmax, m + std::max(1, next));
    for (int j = m; j < upto; ++j)
      if ((expected >> j) & 1u) upto = j + 1;
    for (int j = m; j < upto; ++j) RSV_TRY(run.iterate(j));
    RSV_TRY(run.fetch(upto));
    if (m == 0) {
      nx = std::sqrt(sc[0]);
      if (!std::isfinite(nx)) return fail(RSV_ENUMERIC, "state norm is not finite");
      if (nx == 0.0) return RSV_OK;
      scale[0] = 1.0 / nx;
      course.start(tau, nx, !run.small);
    }
    for (int j = m; j < upto; ++j) {
      // inner product i as fetched at d (real ones for Hermitian matrices)
      auto value = [&](const double* d, int i) {
        return sp.herm ? cd(d[i], 0.0) : cd(d[2 * i], d[2 * i + 1]);
      };
      const double* d = sc + col_off(j);
      const double y2 = value(d, j + 1).real();
      double beta2 = sc[j + 1];
      for (int i = 0; i <= j; ++i) {
        const cd di = value(d, i);
        if (!std::isfinite(di.real()) || !std::isfinite(di.imag()))
          return fail(RSV_ENUMERIC, "Arnoldi inner product not finite");
        H(i, j) = scale[i] * di;  // <v_i, y1>
      }
      // y = y1 - beta_{j-1} v_{j-1} (+ h_{j-1,j-1} v_j)
      if (j > 0) H(j - 1, j) -= 1.0 / scale[j];
      if (j > 0 && sp.shift) H(j, j) += cd(sc[kDiag + 2 * j - 2], sc[kDiag + 2 * j - 1]);
      if (!std::isfinite(beta2)) return fail(RSV_ENUMERIC, "Arnoldi residual not finite");
      bool again = false;
      if (!(beta2 >= 0.5 * y2)) {
        // the first pass removed most of the vector (|y'| < |y1| / sqrt(2), the criterion of
        // Daniel, Gragg, Kaufman and Stewart, 1976): rounding in what is left is no longer small
        // against it, so orthogonalise it once more
        again = true;
        last.again |= uint64_t(1) << j;
        surprises += !((expected >> j) & 1u);
        RSV_TRY(run.orthogonalise(j, true));
        RSV_TRY(run.fetch(j + 1));
        for (int i = 0; i <= j; ++i) {
          const cd d2 = value(sc + kAgain, i);
          if (!std::isfinite(d2.real()) || !std::isfinite(d2.imag()))
            return fail(RSV_ENUMERIC, "Arnoldi inner product not finite");
          H(i, j) += scale[i] * d2;
        }
        beta2 = sc[j + 1];
        if (!std::isfinite(beta2)) return fail(RSV_ENUMERIC, "Arnoldi residual not finite");
      }
      const double beta = std::sqrt(std::max(beta2, 0.0));
      H(j + 1, j) = beta;  // h_{j+1,j} = |y - sum_i v_i <v_i, y>|
      m = j + 1;
      scale[m] = 1.0 / beta;
      course.add(H(j, j).imag(), beta);
      if (m == kmax || beta == 0.0 || course.due(log2_tol)) {
        auto estimate = [&](double t, double* est) -> int {
          if (hess_expm_e1(m, h.data(), kmax, t, y.data()) != 0)
            return fail(RSV_ENUMERIC, "Hessenberg exponential failed (m = %d)", m);
          *est = nx * beta * std::abs(y[m - 1]);
          return RSV_OK;
        };
        double est = 0.0;
        RSV_TRY(estimate(tau, &est));
        if (!(est > tol) || beta == 0.0) return finish(m, tau);
        course.found(est, log2_tol);
        if (m == kmax) {
          // the longest part of the step this basis resolves (same operator, so the split is
          // exact): the estimate grows like the m-th power of the time
          const double least = std::ldexp(tau, -max_depth);
          double t = tau;
          while (est > tol) {
            if (!(t > least))
              return fail(RSV_ENOTCONV, "Arnoldi exponential not converged with kmax = %d", kmax);
            const double r = std::pow(0.5 * tol / est, 1.0 / m);
            t = std::max(least, t * std::min(0.95, std::max(0.5, r)));
            RSV_TRY(estimate(t, &est));
          }
          st->substeps += 1;
          return finish(m, t);
        }
      }
      if (again) break;  // what was queued after this vector used its first form
    }
    next = hint > 0 && m < first ? first - m : course.ahead(log2_tol, kmax - m);
  }
}

}  // namespace

size_t arnoldi_host_doubles() { return col_off(kMaxKrylov); }

int arnoldi_host(rsv_register* reg, double** out) {
  if (!reg->h_arnoldi) {
    const hipError_t e = hipHostMalloc((void**)&reg->h_arnoldi, arnoldi_host_doubles() * sizeof(double),
                                       hipHostMallocDefault);
    if (e != hipSuccess) {
      reg->h_arnoldi = nullptr;
      return fail(RSV_EDEVICE, "hipHostMalloc failed: %s", hipGetErrorString(e));
    }
  }
  *out = reg->h_arnoldi;
  return RSV_OK;
}

static size_t part_doubles(int prec, int nb, int kmax) {
  const size_t rows = (size_t)2 * (kmax + 2) * arnoldi_parts(size_t(1) << nb);
  return std::max(rows, (size_t)vec_num_partials(prec, nb));
}

size_t arnoldi_device_bytes(int prec, int nb, int kmax) {
  const size_t vb = up256((size_t(1) << nb) * amp_bytes(prec));
  return (size_t)(kmax + 1) * vb + up256(part_doubles(prec, nb, kmax) * sizeof(double)) +
         up256(arnoldi_parts(size_t(1) << nb) * sizeof(double)) +
         up256(arnoldi_host_doubles() * sizeof(double));
}

void arnoldi_carve(void* block, double* h_scal, int prec, int nb, int kmax, ArnoldiSpace* sp) {
  sp->prec = prec;
  sp->nb = nb;
  sp->kmax = kmax;
  sp->vb = up256((size_t(1) << nb) * amp_bytes(prec));
  sp->base = (char*)block;
  char* p = (char*)block + (size_t)(kmax + 1) * sp->vb;
  sp->part = (double*)p;
  p += up256(part_doubles(prec, nb, kmax) * sizeof(double));
  sp->npart = (double*)p;
  p += up256(arnoldi_parts(size_t(1) << nb) * sizeof(double));
  sp->dscal = (double*)p;
  sp->h_scal = h_scal;
}

int arnoldi_expm(const OpFn& op, ArnoldiSpace& sp, void* d_x, double tau, double tol,
                 int max_depth, hipStream_t s, rsv_stats* st) {
  if (sp.kmax < 2 || sp.kmax > kMaxKrylov - 1) return fail(RSV_EINVAL, "kmax must be in 2..%d", kMaxKrylov - 1);
  int part = 0;
  for (double remaining = tau; remaining > 0.0;) {
    double sub = 0.0;
    RSV_TRY(expm_part(op, sp, sp.last[part], d_x, remaining, tol, max_depth, s, st, &sub));
    part = std::min(part + 1, ArnoldiSpace::kParts - 1);
    remaining = sub >= remaining ? 0.0 : remaining - sub;
  }
  return RSV_OK;
}

}  // namespace rsv
