// The 2D median of the median entropy filter (section 4), shared by the step
// kernel and the several-steps kernel.
#pragma once

#include "lbm_device.h"

namespace lbm {

template <class R>
__device__ __forceinline__ void sort_net9(R a[9]) {
#pragma unroll
  for (int pass = 0; pass < 9; ++pass) {
#pragma unroll
    for (int j = pass & 1; j + 1 < 9; j += 2) {
      const R lo = fmin(a[j], a[j + 1]), hi = fmax(a[j], a[j + 1]);
      a[j] = lo;
      a[j + 1] = hi;
    }
  }
}

// The ceil(n/2)-th smallest of the n values among nb(0..8) that are not NaN
// (NaN marks a position outside the lattice).
template <class R, class F>
__device__ __forceinline__ R median_of_9(F nb) {
  R a[9];
  int n = 0;
#pragma unroll
  for (int k = 0; k < 9; ++k) {
    const R val = nb(k);
    const bool in = !(val != val);
    n += in ? 1 : 0;
    a[k] = in ? val : r_inf<R>();
  }
  sort_net9<R>(a);
  const int rank = (n + 1) / 2 - 1;
  R med = a[0];
#pragma unroll
  for (int k = 1; k < 9; ++k) med = rank == k ? a[k] : med;
  return med;
}

}  // namespace lbm
