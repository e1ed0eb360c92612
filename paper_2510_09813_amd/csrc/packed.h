// Small-register evolution: one workgroup runs one job's whole evolution (see packed.hip).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "rsv.h"
#include "rsv_internal.h"

namespace rsv {

constexpr int kMaxPackBits = 13;     // largest n in either precision
constexpr int kPackOccOffset = 8;    // out[8 + p]: sum |psi_b|^2 b_p

// One job; every pointer is device memory.  Each step's midpoint values (Sec. III) are formed
// on the host: omega, delta and phi hold n_steps values for a global drive, [n][n_steps] by
// atom for a per-site one.
struct PackedJob {
  int n, kmax, max_depth, per_site;
  int real;       // 1: global drive without phase (one real coupling)
  int direct;     // 1: omega and phi hold 2 Re and 2 Im of <1|h|0> instead (one step's StepCoef)
  int resume;     // 1: out holds a previous launch's results: go on from its state and counters
  double dir;     // -1: exp(+i tau H), the step backwards in time
  int64_t n_steps;
  double tau, tol;  // step in us
  const double* omega;
  const double* delta;
  const double* phi;   // may be null
  const double* ub;    // 32 x 32 interactions by bit position
  double* diag;        // scratch: the interaction energies E_b (2^n)
  const double2* psi0;  // initial state in complex128, or
  const void* psi_in;   // in the storage precision; neither: |0...0>
  void* psi_out;        // optional: final state in the storage precision,
  double2* state;       // optional: and in complex128; written when every step succeeded
  void* basis;        // kmax vectors
  double* out;        // [0] status, [1] H applications, [2] largest Krylov dimension,
                      // [3] sub-steps, [4] |psi|^2, [8 + p] occupation numerators
  double* obs;        // optional: |psi|^2 and the n occupation numerators after every obs_every-th
  int64_t obs_every, obs_first;  // step of the call, obs_first steps of which were done before
};

int packed_max_atoms(int prec);
// Whether the exponentials of a step this wide fit the device's series: half_width bounds the
// half-width of H_k's spectrum (rad/us).
bool packed_resolves(double tau, double half_width);

// Jobs of a batch in device memory, the n_small of up to kPackSmallBits atoms first, then the n_large
// others: one launch each, on their own streams.
constexpr int kPackSmallBits = 10;
hipError_t packed_evolve(int prec, const PackedJob* d_jobs, int n_small, int n_large,
                         hipStream_t s_small, hipStream_t s_large);

// One job whose descriptor and step values travel as kernel arguments (job.omega, delta and phi
// are ignored: mid holds omega, delta and, when with_phi, phi, each job.n_steps x (per_site ? n
// : 1) values).
constexpr int kMidValues = 440;
hipError_t small_evolve(int prec, const PackedJob& job, const double* mid, bool with_phi,
                        hipStream_t s);

}  // namespace rsv
