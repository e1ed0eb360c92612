// The block operator of the pulse gradients (see augmented.hip).
#pragma once

#include <hip/hip_runtime.h>

#include "rsv_internal.h"

namespace rsv {

// From 19 atoms on the vectors leave the L2 and the H psi passes, which read each amplitude a
// few times instead of n, take over.
constexpr int kMaxAugmentedAtoms = 18;

// A step's global drive (<1|h|0> and detuning) and the derivative taken: which = 0, by Omega (v =
// <1|dh/dOmega|0>); 1, by delta.
struct AugmentedCoef {
  int n, which;
  double up_re, up_im, delta, v_re, v_im;
};

// out = -i (H a + V b, H b) of in = [a | b], 2^n amplitudes each; e: the 2^n interaction energies.
hipError_t augmented_apply(int prec, const AugmentedCoef& c, const double* e, const void* in, void* out,
                           hipStream_t s);

}  // namespace rsv
