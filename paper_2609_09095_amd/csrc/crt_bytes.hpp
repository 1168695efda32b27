// Reconstruction modulo the fifteen byte moduli (Alg. 3) as one weighted sum:
// X = sum_q c_q W_q mod M with W_q = (M / m_q) w_q, w_q the centred inverse of
// M / m_q modulo m_q (the CRT that Eq. (garner) evaluates digit by digit), in
// FP64 limbs, and RN(X 2^e).  About 100 VALU instructions per output, nearly
// all of them FP64 FMAs, where Garner's digits and their halves take 171.
// Plain arithmetic only, so it also compiles for the host.
//
// Limbs base 2^40, balanced and scaled to units of 2^40 (w2 2^40, w1, w0
// 2^-40, all exact): the sums are integers below 2^51 times the limb's unit,
// so every FMA of a sum is exact.
//  - k = rint(S / M), |k| < 2^11, from the upper two limbs: the quotient errs
//    by less than 2^-40, so X = S - k M lies in [-M/2, M/2) unless the
//    quotient is within 2^-40 of a half integer (declined).
//  - R_j = S_j - k M_j exactly (|k M_j| < 2^51 units).
//  - p + ep = R_2 + R_1 and t + te = ep + R_0 exactly (two-sums), and
//    r = RN(p + t).  Where te = 0 (ep = 0, or X has few significant bits, as
//    the products of integers and of FP32 values do), X 2^-40 = p + t and r is
//    the rounding itself, of ties and powers of two too.  Otherwise |p| >= 2^53,
//    |t| < 2^26, res = p + t - r exactly (Fast2Sum), and X 2^-40 - r = res + d
//    with |d| <= |t| 2^-53: r is RN of it when |res| + |d| < ulp(r)/2 (with a
//    factor-2 margin) and r is no power of two.
//  - a subnormal result is r rounded once more, by the scaling: the rounding of
//    X 2^e unless r lies on a tie of the subnormal grid (the ties are FP64
//    numbers: any other is at least a whole step from r on its side, X 2^-40 at
//    most half of one), where the sign of X 2^-40 - r decides.
// Returns false where that does not go through.
#pragma once

#include <cstdint>

#include "moduli.hpp"

namespace oz {

struct CrtLimbs {
  double w[kRA][3];  // W_q, lowest limb first
  double m[3];       // M
  double minv;       // 2^40 / M
};
constexpr void crt_split(__int128 v, double (&out)[3]) {
  constexpr __int128 B = (__int128)1 << 40;
  for (int i = 0; i < 2; ++i) {
    __int128 d = v % B;
    if (d >= B / 2) d -= B;
    if (d < -B / 2) d += B;
    out[i] = (double)(int64_t)d;
    v = (v - d) / B;
  }
  out[2] = (double)(int64_t)v;
  out[0] *= 0x1p-40;
  out[2] *= 0x1p40;
}
constexpr CrtLimbs make_crt() {
  CrtLimbs r{};
  __int128 M = 1;
  for (int q = 0; q < kRA; ++q) M *= kModulusA[q];
  for (int q = 0; q < kRA; ++q) {
    const int m = kModulusA[q];
    const __int128 rest = M / m;
    int64_t w = inverse_mod((int64_t)(rest % m), m);
    if (w > m / 2) w -= m;
    crt_split(rest * w, r.w[q]);
  }
  crt_split(M, r.m);
  r.minv = 1.0 / (r.m[2] + r.m[1]);
  return r;
}
inline constexpr CrtLimbs kCrt = make_crt();
// the sums stay exact: 15 terms of |c| <= 128, and k M
constexpr bool crt_limbs_fit() {
  for (int j = 0; j < 3; ++j) {
    const double unit = j == 0 ? 0x1p-40 : (j == 1 ? 1.0 : 0x1p40);
    double s = 0.0;
    for (int q = 0; q < kRA; ++q) s += 128.0 * (kCrt.w[q][j] < 0 ? -kCrt.w[q][j] : kCrt.w[q][j]);
    const double km = 2048.0 * (kCrt.m[j] < 0 ? -kCrt.m[j] : kCrt.m[j]);
    if (s / unit >= 0x1p51 || km / unit >= 0x1p51) return false;
  }
  return true;
}
static_assert(crt_limbs_fit(), "limb sums below 2^51 units");

__device__ __forceinline__ bool crt_bytes(const int (&c)[kRA], int e, double& out) {
  double s0 = 0.0, s1 = 0.0, s2 = 0.0;
#pragma unroll
  for (int q = 0; q < kRA; ++q) {
    const double d = (double)c[q];
    s0 = __builtin_fma(d, kCrt.w[q][0], s0);
    s1 = __builtin_fma(d, kCrt.w[q][1], s1);
    s2 = __builtin_fma(d, kCrt.w[q][2], s2);
  }
  const double quo = (s2 + s1) * kCrt.minv;
  const double k = __builtin_rint(quo);
  const bool inside = __builtin_fabs(quo - k) < 0.5 - 0x1p-39;
  const double r0 = __builtin_fma(-k, kCrt.m[0], s0);
  const double r1 = __builtin_fma(-k, kCrt.m[1], s1);
  const double r2 = __builtin_fma(-k, kCrt.m[2], s2);
  const double p = r2 + r1, b = p - r2;
  const double ep = (r2 - (p - b)) + (r1 - b);
  const double t = ep + r0;
  const double r = p + t;
  const double res = t - (r - p);
  const uint64_t rb = __builtin_bit_cast(uint64_t, r);
  const int eb = (int)(rb >> 52) & 0x7FF;
  const double halfu = __builtin_bit_cast(double, (uint64_t)(eb - 53) << 52);
  const double bound = __builtin_fma(__builtin_fabs(t), 0x1p-51, __builtin_fabs(res));
  const bool proven = ep == 0.0 || (bound < halfu && (rb << 12) != 0);
  out = __builtin_ldexp(r, e + 40);
  const bool normal = eb + e + 40 >= 1 || eb == 0;
  if (inside && proven && normal) [[likely]]
    return true;
  // apart from the common path, whose chain it would lengthen (201 x 333 x 157
  // 11.4 -> 11.5 us)
  const double tb = t - ep;
  const double te = (ep - (t - tb)) + (r0 - tb);
  if (!inside || !(proven || te == 0.0)) return false;
  if (normal) return true;
  const double half = __builtin_ldexp(1.0, -1115 - e);  // of the subnormal grid's step
  // res + te: X 2^-40 - r exactly (where |p| < |t|, p + t needs no rounding)
  if (__builtin_fabs(r - __builtin_ldexp(out, -e - 40)) == half && res + te != 0.0)
    out = __builtin_copysign(__builtin_ldexp(r + __builtin_copysign(half, res + te), e + 40), r);
  return true;
}

}  // namespace oz
