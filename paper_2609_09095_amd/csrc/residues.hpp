// Quantiser and centred residues of Alg. 2 (Eq. (scale), Eq. (residueprod)),
// shared by the deconstruction and the one-kernel product.
#pragma once

#include <hip/hip_runtime.h>
#include <cstdint>

#include "moduli.hpp"

namespace oz {

// Integer-valued doubles y with |y| <= 2^51 sit in the low mantissa bits of
// y + kMagic (every such sum lies in [2^52, 2^53], where the spacing is 1),
// so the low word of that sum is y mod 2^32.
constexpr double kMagic = 6755399441055744.0;  // 1.5 * 2^52
__device__ __forceinline__ uint32_t low_word(double v) {
  return (uint32_t)__builtin_bit_cast(uint64_t, v);
}
constexpr int log2_exact(int m) { return m <= 1 ? 0 : 1 + log2_exact(m / 2); }

// Residue modes (the template parameter RM below), by the range of the
// scaled integers y = RN(x 2^sigma), |y| <= 2^t:
//  1: ylo = y mod 2^32 from y + kMagic                        (|y| <= 2^51)
//  2: ylo split off by one exact FMA                          (|y| <= 2^52,
//     the odd byte moduli only)
//  3: y first reduced modulo the product N of a group of moduli, which keeps
//     every residue of the group and brings it into mode 1's range
//                                                             (|y| <= 2^58)
// 2^58 bounds every scale the library uses (t(k) <= 58 for both sets, and
// the accurate mode's shifts are capped there).  One reduction per group of
// four (published) or five (byte) moduli costs four FP64 instructions per
// element; correcting each modulus's quotient instead cost seven each
// (whole calls: 1537 x 2049 x 1031 on the byte moduli at t = 53 167 -> 157 us,
// accurate mode at 4096^3 1331 -> 1301 us).
//
// y - q M modulo 2^24 for the FMA quotient q (ylo = y mod 2^32).  For odd M
// the FMA rounds y RN(1/M) + kMagic once, to kMagic + the integer nearest
// y RN(1/M) (|y / M| < 2^51, so the sum lies in [2^52, 2^53), where the
// spacing is 1); that product is within |y| ulp(1/M) / 2 of y / M.  For
// |y| <= 2^51 that is at most 1/(4M), while y / M is at least 1/(2M) away
// from a half integer, so the integer is the nearest quotient q and the low
// word of the sum is q mod 2^32.  For the odd byte moduli (M <= 255,
// ulp(1/M) / 2 = 2^-61) this holds up to |y| <= 2^52: the error is at most
// 2^-9 < 1/510.  The 24-bit multiply-add gives y - q M mod 2^24.  For a
// power of two M, y itself (mod 2^24) serves: its low log2(M) bits are the
// residue.
template <int M>
__device__ __forceinline__ int residue_low(double y, uint32_t ylo) {
  if constexpr ((M & (M - 1)) == 0) {
    return (int)ylo;
  } else {
    const double t = __builtin_fma(y, 1.0 / M, kMagic);
    // spelled out: left to itself the compiler widens this into a 64-bit
    // multiply-add once it sees that only the low bits are used
    int r;
    asm("v_mad_i32_i24 %0, %1, %2, %3" : "=v"(r) : "v"(low_word(t)), "s"(-M), "v"(ylo));
    return r;
  }
}

// Centred residue of the integer-valued y modulo M, in [-(M/2), (M-1)/2]
// (an int, |residue| <= 544): the low bits of residue_low, sign-extended --
// log2(M) bits for a power of two (the two's complement field is
// [-M/2, M/2) by itself), 24 bits for odd M, centred as q is the nearest
// quotient.
template <int M>
__device__ __forceinline__ int centred_residue(double y, uint32_t ylo) {
  if constexpr ((M & (M - 1)) == 0) {
    constexpr int sh = 32 - log2_exact(M);
    return (int)(ylo << sh) >> sh;
  } else {
    return (int)((uint32_t)residue_low<M>(y, ylo) << 8) >> 8;
  }
}

// Four byte residues at once, the first in the low byte: only y - q M modulo
// 2^8 is wanted, so pairs of quotients and of y (ypair: their low halves)
// share one packed 16-bit multiply-add -- nine instructions per four
// residues where separate 24-bit multiply-adds and their byte packing take
// eleven.
typedef uint16_t u16x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t low_halves(uint32_t a, uint32_t b) {  // a low, b high
  return __builtin_amdgcn_perm(b, a, 0x05040100u);
}
// minus M = -M in both halves, qinv = RN(1/M)
__device__ __forceinline__ uint32_t residue_bytes(double y0, double y1, double y2, double y3, uint32_t y01,
                                                  uint32_t y23, u16x2 minus_m, double qinv) {
  const uint32_t q01 = low_halves(low_word(__builtin_fma(y0, qinv, kMagic)), low_word(__builtin_fma(y1, qinv, kMagic)));
  const uint32_t q23 = low_halves(low_word(__builtin_fma(y2, qinv, kMagic)), low_word(__builtin_fma(y3, qinv, kMagic)));
  const u16x2 r01 = __builtin_bit_cast(u16x2, q01) * minus_m + __builtin_bit_cast(u16x2, y01);
  const u16x2 r23 = __builtin_bit_cast(u16x2, q23) * minus_m + __builtin_bit_cast(u16x2, y23);
  return __builtin_amdgcn_perm(__builtin_bit_cast(uint32_t, r23), __builtin_bit_cast(uint32_t, r01), 0x06040200u);
}
template <int M>
__device__ __forceinline__ uint32_t residue_bytes(double y0, double y1, double y2, double y3, uint32_t y01,
                                                  uint32_t y23) {
  if constexpr (M == 256)
    return __builtin_amdgcn_perm(y23, y01, 0x06040200u);
  else
    return residue_bytes(y0, y1, y2, y3, y01, y23, u16x2{(uint16_t)-M, (uint16_t)-M}, 1.0 / M);
}

// Mode 3: y modulo N, |result| <= N (1/2 + 2^-12), and its low word.  The
// quotient's error is at most |y| 2^-52 / N; y - q N is an integer below
// 2^48, so the one FMA gives it exactly.
template <int E>
__device__ __forceinline__ void reduce_group(const double (&y)[E], double N, double ninv, double (&z)[E],
                                             uint32_t (&zlo)[E]) {
#pragma unroll
  for (int c = 0; c < E; ++c) {
    const double q = __builtin_rint(y[c] * ninv);
    z[c] = __builtin_fma(-q, N, y[c]);
    zlo[c] = low_word(z[c] + kMagic);
  }
}
// the product of moduli i .. i + count - 1, below 2^48 and at least 2^18
// (at |y| <= 2^58 the quotient then errs by at most 2^-12, so that |y - q N| is
// at most N (1/2 + 2^-12))
template <int R>
constexpr int64_t group_product(const int (&m)[R], int i, int count) {
  int64_t p = 1;
  for (int j = i; j < i + count; ++j) p *= m[j];
  return p;
}
constexpr int kGroup = 4, kGroupA = 5;  // moduli per group, published / byte set
template <int R>
constexpr bool groups_in_range(const int (&m)[R], int count) {
  if (R % count) return false;
  for (int i = 0; i < R; i += count) {
    const int64_t p = group_product(m, i, count);
    if (p >= (int64_t)1 << 48 || p < (int64_t)1 << 18) return false;
  }
  return true;
}
static_assert(groups_in_range(kModulus, kGroup) && groups_in_range(kModulusA, kGroupA), "mode 3 groups");

// |x 2^sigma| < 2^t: the scaling is exact, and the quantiser of Eq. (scale)
// is the one rounding: to nearest even (RN), or toward zero (TZ).  Then
// ylo = y mod 2^32: from y + kMagic (RM 1, |y| <= 2^51), or (RM 2: past
// 2^51 that sum is no longer exact) as y - h 2^32 with h = floor(y 2^-32),
// one exact FMA; RM 3 forms it per group (reduce_group).
template <bool TZ, int RM, int E>
__device__ __forceinline__ void scale_round(const double (&x)[E], int sigma, double (&y)[E],
                                            uint32_t (&ylo)[E]) {
#pragma unroll
  for (int c = 0; c < E; ++c) {
    const double v = __builtin_ldexp(x[c], sigma);
    y[c] = TZ ? __builtin_trunc(v) : __builtin_rint(v);
    if constexpr (RM == 1)
      ylo[c] = low_word(y[c] + kMagic);
    else if constexpr (RM == 2)
      ylo[c] = (uint32_t)__builtin_fma(-__builtin_floor(y[c] * 0x1p-32), 0x1p32, y[c]);
  }
}

// four residues in [-128, 127] as bytes, the first in the low byte
// (v_perm_b32 selectors: 0-3 bytes of the second operand, 4-7 of the first,
// 12 gives 0)
__device__ __forceinline__ uint32_t pack_bytes(int a, int b, int c, int d) {
  const uint32_t ab = __builtin_amdgcn_perm((uint32_t)b, (uint32_t)a, 0x0c0c0400u);
  const uint32_t cd = __builtin_amdgcn_perm((uint32_t)d, (uint32_t)c, 0x0c0c0400u);
  return __builtin_amdgcn_perm(cd, ab, 0x05040100u);
}

}  // namespace oz
