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
// N outputs of one row a at once, in columns col[j] < 2^28 of B, their chains
// side by side, with the loads of U terms in flight: the additions keep their
// order, and with one term's loads at a time every addition waited for memory
// (a flagged row of 256 columns at k = 4096 added 1.0 ms to its call, now 0.2).
template <int N, int U>
__device__ __forceinline__ void native_dots(const double* __restrict__ a, const double* __restrict__ B,
                                            const uint32_t (&col)[N], int64_t ldb, int64_t k, double (&s)[N]) {
#pragma clang fp contract(off)
  // through a buffer resource at the row of B: one 32-bit offset per output
  // where global loads took a 64-bit address per load, and the reconstruction's
  // occupancy with them
  const auto b = [&](int64_t l, int j) __attribute__((always_inline)) {
    const uint64_t v = (uint64_t)(B + l * ldb);
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v);
    const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
    const __amdgpu_buffer_rsrc_t row = __builtin_amdgcn_make_buffer_rsrc((void*)(((uint64_t)hi << 32) | lo), (short)0,
                                                                         0x7FFFFFFF, 0x00020000);
    return __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(row, (int)(col[j] * 8u), 0, 0));
  };
#pragma unroll
  for (int j = 0; j < N; ++j) s[j] = 0.0;
  int64_t l = 0;
#pragma unroll 1
  for (; l + U <= k; l += U) {
    double x[U], y[U][N];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      x[u] = a[l + u];
#pragma unroll
      for (int j = 0; j < N; ++j) y[u][j] = b(l + u, j);
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int j = 0; j < N; ++j) {
        const double p = x[u] * y[u][j];
        s[j] = s[j] + p;
      }
  }
#pragma unroll 1
  for (; l < k; ++l)
#pragma unroll
    for (int j = 0; j < N; ++j) {
      const double p = a[l] * b(l, j);
      s[j] = s[j] + p;
    }
}

__device__ __forceinline__ double native_dot(const double* a, const double* B, uint32_t col, int64_t ldb, int64_t k) {
  const uint32_t cols[1] = {col};
  double s[1];
  native_dots<1, 8>(a, B, cols, ldb, k, s);
  return s[0];
}

}  // namespace oz
