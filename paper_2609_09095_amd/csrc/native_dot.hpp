// The native FP64 re-issue of one output (the range check that ends Alg. 1).
#pragma once

#include <hip/hip_runtime.h>
#include <cstdint>

namespace oz {

// Alg. 1's last step, the native FP64 re-issue: an output whose row of A or
// column of B holds a NaN or an infinity (exponent INT32_MIN) has no
// emulated value, and becomes the dot product of that row and column in
// index order from +0, each product rounded and then added (the library is
// built with -ffp-contract=off; contraction is also switched off here).
// Such a value is always an infinity or a NaN.
__device__ __forceinline__ double native_dot(const double* __restrict__ a, const double* __restrict__ b,
                                             int64_t ldb, int64_t k) {
#pragma clang fp contract(off)
  double s = 0.0;
  for (int64_t l = 0; l < k; ++l) {
    const double p = a[l] * b[l * ldb];
    s = s + p;
  }
  return s;
}

// N such outputs at once, each as above: the dots' chains run side by side,
// since one is bound by the latency of its loads and additions.
template <int N>
__device__ __forceinline__ void native_dots(const double* const (&a)[N], const double* const (&b)[N], int64_t ldb,
                                            int64_t k, double (&s)[N]) {
#pragma clang fp contract(off)
#pragma unroll
  for (int j = 0; j < N; ++j) s[j] = 0.0;
  for (int64_t l = 0; l < k; ++l) {
#pragma unroll
    for (int j = 0; j < N; ++j) {
      const double p = a[j][l] * b[j][l * ldb];
      s[j] = s[j] + p;
    }
  }
}

}  // namespace oz
