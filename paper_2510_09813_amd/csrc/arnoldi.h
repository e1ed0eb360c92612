// Arnoldi Krylov exponential x <- exp(tau Op) x for non-Hermitian operators on device vectors
// (the Lindblad equation's Liouvillian, the augmented operator of the pulse gradients), and
// the exponential of its small Hessenberg matrix.
#pragma once

#include <hip/hip_runtime.h>

#include <complex>
#include <cstdint>
#include <functional>
#include <vector>

#include "engine.h"
#include "krylov_course.h"

namespace rsv {

// exp(a) of an m x m complex matrix (row-major), host FP64; 0 on success.
int dense_expm(int m, const std::complex<double>* a, std::complex<double>* out);
// y = exp(tau a) e_1 of an m x m upper Hessenberg matrix (row-major, leading dimension ld), host
// FP64; 0 on success.
int hess_expm_e1(int m, const std::complex<double>* a, int ld, double tau, std::complex<double>* y);

// ------------------------------------------------------------------------------- kernels
constexpr int kArnoldiGroup = 8;  // vectors per pass over y in the inner products
constexpr int kHermGroup = 16;    // the same of Hermitian matrices, whose inner products are real
constexpr int kSmallBits = 18;    // vectors up to 2^18 elements: partial sums summed by their reader
constexpr int kSmallParts = 256;  // at most
// One Gram-Schmidt pass of iteration j.  u_0 = v0, u_i = base + i stride (elements); w = Op u_j
// (again: w = u_{j+1}, the second pass, which orthogonalises u_{j+1} once more in place).
struct ArnoldiStep {
  int j, again;
  const void* v0;
  void* base;
  size_t stride, count;
  const void* w;
  int herm;             // > 0: vectors are Hermitian 2^herm x 2^herm matrices (long vectors only);
                        // dots then holds j + 2 real values
  int shift;            // take out h_{j-1,j-1} along u_j (see gram_schmidt.hip)
  double* nrm2;         // |u_i|^2, i <= j
  double* diag;         // shift: h_ii re, im, i < j; h_jj is added
  const double* npart;  // nparts > 0: the partials of |u_j|^2, to be summed into nrm2[j]
  int nparts;
  double* part;         // 2 (j + 2) x arnoldi_parts partial inner products
  int dparts;           // > 0: the update sums them (into dots); 0: dots holds the sums
  double* dots;         // <u_i, y1> re, im for i <= j, then <y1, y1>, 0
  double* npart_out;    // arnoldi_parts partials of |u_{j+1}|^2
};
int arnoldi_parts(size_t count);
hipError_t arnoldi_dots(int prec, const ArnoldiStep& a, hipStream_t s);
hipError_t arnoldi_update(int prec, const ArnoldiStep& a, hipStream_t s);
// |u_{j+1}|^2 from a small vector's partial sums.
hipError_t arnoldi_norm(const double* npart, int parts, double* out, hipStream_t s);
// Partials of |x - x^+|^2, then of |x|^2 (arnoldi_parts(4^n) each), of a 2^n x 2^n matrix; with
// write, x <- (x + x^+) / 2 instead.  n >= 5.
hipError_t hermitise(int prec, int n, void* x, bool write, double* part, hipStream_t s);

// ------------------------------------------------------------------------------- process
// Device vectors of 2^nb amplitudes (storage precision prec): the Krylov basis (kmax vectors
// after the state itself, kept unnormalised), the operator's result, partial sums and device
// scalars.
struct ArnoldiSpace {
  int prec = 0, nb = 0, kmax = 0;
  char* base = nullptr;  // slot i >= 1 holds u_i; slot 0 the operator's result
  size_t vb = 0;
  double* part = nullptr;   // partial inner products
  double* npart = nullptr;  // partials of the newest norm
  double* dscal = nullptr;  // the norms, the Hessenberg diagonal, the second pass's inner products
                            // (kMaxKrylov + 2 of each), then the columns
  double* h_scal = nullptr;  // pinned host copy of dscal
  int herm = 0;              // the vectors are Hermitian 2^herm x 2^herm matrices and op keeps them so
  bool shift = false;        // the operator's diagonal in the basis is far from zero (-i H)
  // of the step before, by sub-step: its dimension (how many iterations to queue first) and the columns
  // that needed a second Gram-Schmidt pass
  struct Last {
    int dim = 0;
    uint64_t again = 0;
  };
  static constexpr int kParts = 8;
  Last last[kParts];
};
size_t arnoldi_device_bytes(int prec, int nb, int kmax);
// Lays out the device block (arnoldi_device_bytes); h_scal: arnoldi_host_doubles() pinned doubles.
void arnoldi_carve(void* block, double* h_scal, int prec, int nb, int kmax, ArnoldiSpace* sp);
size_t arnoldi_host_doubles();
// The register's pinned block of that size, allocated on first use and kept.
int arnoldi_host(rsv_register* reg, double** out);

using OpFn = std::function<int(const void* in, void* out, hipStream_t s)>;

// x <- exp(tau Op) x with the Arnoldi process (classical Gram-Schmidt, a second pass when the
// first removes most of the new vector, FP64 inner products), y = exp(tau H_m) e_1 from the
// Hessenberg matrix, converged when
// |x| h_{m+1,m} |y_m| <= tol (the estimate of Saad 1992 used by the Lanczos path), x = |x| V_m y.
// Without convergence in kmax vectors the part of the step that the basis resolves is taken and
// the rest follows (exact for a constant operator); RSV_ENOTCONV where that is less than
// 2^-max_depth of it.
int arnoldi_expm(const OpFn& op, ArnoldiSpace& sp, void* d_x, double tau, double tol,
                 int max_depth, hipStream_t s, rsv_stats* st);

}  // namespace rsv
