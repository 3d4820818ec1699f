// hpic_divide.h -- exact integer division from an approximate quotient.  No GPU
// headers unless hipcc compiles it, so that a test can compile it for the host.
#pragma once

#ifdef __HIPCC__
#include <hip/hip_runtime.h>
#define HPIC_HD __host__ __device__ __forceinline__
#else
#define HPIC_HD inline
#endif

namespace hp {

// a / b and its remainder for 0 <= a < 2^30, b > 0 from a guess q of the quotient.
// The guess is a float product with a hardware reciprocal: right or one off below
// 2^23, and off by up to a / b * 2^-22 + 1 above (a row number of a grid of 8 x 2^27
// cells no longer fits a float), so the correction goes on until the remainder is one.
HPIC_HD int settle_quotient(int a, int b, int q, int &rem) {
  int m = a - q * b;
  while (m < 0) {
    --q;
    m += b;
  }
  while (m >= b) {
    ++q;
    m -= b;
  }
  rem = m;
  return q;
}

}  // namespace hp
