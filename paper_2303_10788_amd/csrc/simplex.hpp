// The shift tau that projects values onto the probability simplex
// (max(v - tau, 0) sums to one) by Michelot's iteration: tau = (sum of the
// active values - 1) / their count, active = the values above the previous tau.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace ccut {

struct SimplexShift {
  double tau;      // the values above it are active
  uint64_t count;  // of them the last time
  // One round: the sum and number of the active values.  False: tau is the shift.
  // The active set shrinks from round to round, but tau is rounded: values within
  // its rounding (the zero eigenvalues of a state are such values, tau being a
  // rounding residue there) would come back and go again for ever.  A set that
  // does not shrink ends it: at most one round per value.
  __host__ __device__ bool round(double sum, uint64_t active) {
    if (active >= count || active == 0) return false;
    tau = (sum - 1.0) / (double)active;
    count = active;
    return true;
  }
};

}  // namespace ccut
