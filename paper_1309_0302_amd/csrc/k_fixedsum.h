// Sums of squares whose terms come in any order, shared by the selection's
// compaction and its final step (and compiled for the host by its test).
#pragma once

#include <hip/hip_runtime.h>
#include <math.h>

namespace godec {

// Sum that does not depend on the order of its terms: each term relative to a
// bound of the whole sum in two limbs of 40 bits (what is cut off is 2^-80 of
// the bound per term), added as integers.  A low limb holds 2^23 terms: an
// adder carries it into the high limb at least that often, and once more after
// adding up lanes, so it hands on less than 2^40 and 2^24 adders fit in 64
// bits, whatever the number of terms.  Bounds outside the range of the scale
// factor leave it to plain FP64 sums.
struct FixedSum {
  double up, down;
  bool on;
  __host__ __device__ explicit FixedSum(double bound) {
    on = bound > 1e-280 && bound < 1e280;
    int ex = 0;
    if (on) frexp(bound, &ex);
    up = on ? ldexp(1.0, 40 - ex) : 0.0;
    down = on ? ldexp(1.0, ex - 40) : 0.0;
  }
  static __host__ __device__ void carry(unsigned long long& hi, unsigned long long& lo) {
    hi += lo >> 40;
    lo &= (1ull << 40) - 1ull;
  }
  __host__ __device__ void add(double q, unsigned long long& hi, unsigned long long& lo) const {
    const double s = q * up, f = floor(s);
    hi += (unsigned long long)f;
    lo += (unsigned long long)((s - f) * 0x1p40);
  }
  __host__ __device__ double value(unsigned long long hi, unsigned long long lo) const {
    return ((double)hi + (double)lo * 0x1p-40) * down;
  }
};

}  // namespace godec
