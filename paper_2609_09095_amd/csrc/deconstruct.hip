// Deconstruction (Alg. 2): scale by 2^sigma, quantise (round to nearest even,
// or toward zero for the truncating variant), twelve
// centred residues, limb split, packed e4m3 plane stores (every limb is an
// e4m3-exact integer, Lemma 1, so the conversion is exact).  For the
// all-byte set (Sec. 5.1, candidate A) fifteen centred residues stored as
// int8, one plane per modulus.
//
// Each thread owns one vector (row of A / column of B) and 16 consecutive k,
// so every plane store is one 16-byte write.  VALU work and HBM traffic (8
// bytes read and 30 bytes written per element) are close: the nonsquare
// limb split comes from a small LDS table to keep the VALU side short.
// A wavefront covers 8 vectors x 128 k on both sides (group_of), so each of
// its plane stores is one contiguous KiB of the k-block-major layout:
//  - A (side 0): eight lanes read 1 KiB of one row;
//  - B (side 1): every FP64 load reads 64 contiguous bytes of 8 rows of B.
#include <utility>

#include "exponent_key.hpp"
#include "kernels.hpp"
#include "moduli.hpp"
#include "residues.hpp"

namespace oz {
namespace {

constexpr int kElems = 16;  // k values per thread

// 16 plane bytes: a streaming store (the planes are read back by the
// residue GEMM long after, from HBM)
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
template <bool NT = true>
__device__ __forceinline__ void put16(int8_t* p, uint4 w) {
  const u32x4 v{w.x, w.y, w.z, w.w};
  if constexpr (NT)
    __builtin_nontemporal_store(v, reinterpret_cast<u32x4*>(p));
  else
    *reinterpret_cast<u32x4*>(p) = v;
}

// four limbs as e4m3 bytes (OCP E4M3FN), the first in the low byte
__device__ __forceinline__ uint32_t pack4(float a, float b, float c, float d) {
  const int lo = __builtin_amdgcn_cvt_pk_fp8_f32(a, b, 0, false);
  return (uint32_t)__builtin_amdgcn_cvt_pk_fp8_f32(c, d, lo, true);
}

__device__ __forceinline__ void store16(int8_t* p, const float (&b)[kElems]) {
  uint4 w;
  w.x = pack4(b[0], b[1], b[2], b[3]);
  w.y = pack4(b[4], b[5], b[6], b[7]);
  w.z = pack4(b[8], b[9], b[10], b[11]);
  w.w = pack4(b[12], b[13], b[14], b[15]);
  put16(p, w);
}

// Square modulus s^2 (Eq. (pieces) with base s): d0 = centred d mod s (the
// balanced digit, [-16, 15] for s = 32), d1 = (d - d0) / s.  |d| <= 544, so
// every step is exact in FP32 and the digits come out as the floats the
// e4m3 conversion takes.
template <int S>
__device__ __forceinline__ void split_square(float d, float& d0, float& d1) {
  // d1 = floor(d / s + 1/2): for even s exactly the balanced digit with d0 in
  // [-s/2, s/2); for odd s, d / s is never within 1/(2s) of a half integer,
  // far above the FP32 error of the FMA, so this is the nearest digit.  floor
  // never returns -0 here, so a zero digit gets the e4m3 code 0x00.
  d1 = __builtin_floorf(__builtin_fmaf(d, 1.0f / S, 0.5f));
  d0 = __builtin_fmaf(-(float)S, d1, d);
}

// Nonsquare modulus (Lemma 1): canonical balanced base-16 split (d0 in
// [-8, 7]), then one carry when d0 + d1 is odd with |d0 + d1| >= 17 --
// exactly the sums +-17, +-19, +-21, +-23 that e4m3 cannot hold.  d0 != 0
// whenever it fires.  All in FP32 on small integers, so exact; no -0 can
// arise (x - x and x + (-x) give +0 under round to nearest).
__device__ __forceinline__ void split_16(float d, float& d0, float& d1, float& d2) {
  float h = __builtin_floorf(__builtin_fmaf(d, 1.0f / 16, 0.5f));
  float l = __builtin_fmaf(-16.0f, h, d);
  const float s = l + h;
  const bool carry = __builtin_fabsf(s) > 16.0f && __builtin_amdgcn_fractf(s * 0.5f) != 0.0f;
  const float sg = l > 0.0f ? 1.0f : -1.0f;
  l = carry ? __builtin_fmaf(-16.0f, sg, l) : l;
  h = carry ? h + sg : h;
  d0 = l;
  d1 = h;
  d2 = l + h;
}

// The split depends on the residue alone, not on the modulus, and every
// nonsquare residue lies in [-255, 255]: a block tabulates it once in LDS
// as the three e4m3 codes (d0, d1, d0 + d1) in bytes 0-2 of entry d + 256.
constexpr int kSplitTable = 512;

__device__ __forceinline__ uint32_t split_16_codes(int d) {
  float d0, d1, d2;
  split_16((float)d, d0, d1, d2);
  const int lo = __builtin_amdgcn_cvt_pk_fp8_f32(d0, d1, 0, false);
  return (uint32_t)__builtin_amdgcn_cvt_pk_fp8_f32(d2, 0.0f, lo, true);
}

// Byte k of four table entries into one dword per plane (v_perm_b32 picks
// bytes of {hi, lo}: 0-3 from lo, 4-7 from hi, 12 gives 0).
__device__ __forceinline__ void gather_planes(uint32_t x0, uint32_t x1, uint32_t x2, uint32_t x3,
                                              uint32_t& p0, uint32_t& p1, uint32_t& p2) {
  const uint32_t t01 = __builtin_amdgcn_perm(x1, x0, 0x05010400u);  // x0.b0 x1.b0 x0.b1 x1.b1
  const uint32_t t23 = __builtin_amdgcn_perm(x3, x2, 0x05010400u);
  const uint32_t u01 = __builtin_amdgcn_perm(x1, x0, 0x0c0c0602u);  // x0.b2 x1.b2 0 0
  const uint32_t u23 = __builtin_amdgcn_perm(x3, x2, 0x0c0c0602u);
  p0 = __builtin_amdgcn_perm(t23, t01, 0x05040100u);
  p1 = __builtin_amdgcn_perm(t23, t01, 0x07060302u);
  p2 = __builtin_amdgcn_perm(u23, u01, 0x05040100u);
}

template <int I>
__device__ __forceinline__ void emit_modulus(const double (&y)[kElems], const uint32_t (&ylo)[kElems],
                                             int8_t* planes,
                                             int64_t plane_stride, int64_t off,
                                             const uint32_t* lut) {
  constexpr int M = kModulus[I];
  constexpr int S = root_of(I);
  constexpr int Q = plane_base(I);
  int8_t* base = planes + (int64_t)Q * plane_stride + off;
  if constexpr (S != 0) {
    float l0[kElems], l1[kElems];
#pragma unroll
    for (int c = 0; c < kElems; ++c)
      split_square<S>((float)centred_residue<M>(y[c], ylo[c]), l0[c], l1[c]);
    store16(base, l0);
    store16(base + plane_stride, l1);
  } else {
    uint32_t x[kElems];
#pragma unroll
    for (int c = 0; c < kElems; ++c) x[c] = lut[centred_residue<M>(y[c], ylo[c]) + 256];
    uint4 w0, w1, w2;
    gather_planes(x[0], x[1], x[2], x[3], w0.x, w1.x, w2.x);
    gather_planes(x[4], x[5], x[6], x[7], w0.y, w1.y, w2.y);
    gather_planes(x[8], x[9], x[10], x[11], w0.z, w1.z, w2.z);
    gather_planes(x[12], x[13], x[14], x[15], w0.w, w1.w, w2.w);
    put16(base, w0);
    put16(base + plane_stride, w1);
    put16(base + 2 * plane_stride, w2);
  }
}

// moduli FIRST + I...
template <int FIRST, int... I>
__device__ __forceinline__ void emit_some(std::integer_sequence<int, I...>, const double (&y)[kElems],
                                          const uint32_t (&ylo)[kElems], int8_t* planes,
                                          int64_t plane_stride, int64_t off, const uint32_t* lut) {
  (emit_modulus<FIRST + I>(y, ylo, planes, plane_stride, off, lut), ...);
}
template <int RM>
__device__ __forceinline__ void emit_all(const double (&y)[kElems], const uint32_t (&ylo)[kElems],
                                         int8_t* planes, int64_t plane_stride, int64_t off,
                                         const uint32_t* lut) {
  if constexpr (RM != 3) {
    emit_some<0>(std::make_integer_sequence<int, kR>{}, y, ylo, planes, plane_stride, off, lut);
  } else {
    [&]<int... G>(std::integer_sequence<int, G...>) {
      ([&] {
        constexpr double N = (double)group_product(kModulus, G * kGroup, kGroup);
        double z[kElems];
        uint32_t zlo[kElems];
        reduce_group(y, N, 1.0 / N, z, zlo);
        emit_some<G * kGroup>(std::make_integer_sequence<int, kGroup>{}, z, zlo, planes, plane_stride, off, lut);
      }(),
       ...);
    }(std::make_integer_sequence<int, kR / kGroup>{});
  }
}

// Thread -> (vector, 16-k group), both sides: a block covers 32 vectors x
// 128 k -- one k-block of the plane layout -- and a wavefront 8 vectors, so
// every plane store of a wavefront fills 1 KiB of contiguous plane bytes and
// consecutive blocks continue the same k-block: the stores sweep each plane
// region linearly.  Lane l takes vector l%8 and k group l/8 (for B, eight
// consecutive columns: each FP64 load reads 64 contiguous bytes of 8 rows).
__device__ __forceinline__ void group_of(int64_t block, int64_t vecs, int64_t& v, int64_t& g) {
  const int64_t vb = (vecs + 31) / 32;
  const int lane = threadIdx.x & 63;
  v = (block % vb) * 32 + (threadIdx.x >> 6) * 8 + (lane & 7);
  g = (block / vb) * 8 + (lane >> 3);
}

// Byte offset of a thread's 16 plane bytes within plane 0, in the layout
// [k_pad/128][planes][vecs][128]: plane q adds q * vecs * 128.
__device__ __forceinline__ int64_t plane_offset(int64_t vecs, int nplanes, int64_t v, int64_t g) {
  return ((g >> 3) * nplanes * vecs + v) * 128 + (g & 7) * 16;
}

// The 16 inputs of a group: unconditional loads from clamped (always valid)
// addresses, then the mask, so no branches sit around the loads; zeros past
// k, for inactive threads and for a non-finite vector.  Returns sigma (0 for
// a non-finite vector).
template <int SIDE>
__device__ __forceinline__ int load_scaled(int64_t vecs, int64_t k, const double* __restrict__ X, int64_t ldx,
                                           int sigma, int64_t v, int64_t k0, bool active,
                                           double (&x)[kElems]) {
  const bool finite = sigma != INT32_MIN;
  sigma = finite ? sigma : 0;
  // lim = last valid c of this group
  const int64_t vc = v < vecs ? v : vecs - 1;
  const int64_t kc = k0 < k ? k0 : k - 1;
  const int lim = k0 < k ? (int)(k - k0 < kElems ? k - k0 : kElems) - 1 : 0;
  const double* first = SIDE == 0 ? X + vc * ldx + kc : X + kc * ldx + vc;
  const bool live = active && finite;
  if constexpr (SIDE == 0) {
    // a whole group of a row whose start is 16-byte aligned: eight 16-byte
    // loads (the vector memory path moves twice the bytes per request)
    if (k0 + kElems <= k && (((uintptr_t)X | (uintptr_t)(ldx * 8)) & 15) == 0) {
      const double2* p = reinterpret_cast<const double2*>(first);
#pragma unroll
      for (int c = 0; c < kElems / 2; ++c) {
        const double2 q = p[c];
        x[2 * c] = live ? q.x : 0.0;
        x[2 * c + 1] = live ? q.y : 0.0;
      }
      return sigma;
    }
  }
#pragma unroll
  for (int c = 0; c < kElems; ++c) {
    const int cc = c < lim ? c : lim;
    const double xv = SIDE == 0 ? first[cc] : first[(int64_t)cc * ldx];
    x[c] = (live && c <= lim && k0 + c < k) ? xv : 0.0;
  }
  return sigma;
}

// sigma from exps (keys_in: the column scan's exponent keys)
template <int SIDE>
__device__ __forceinline__ int load_group(int64_t vecs, int64_t k, const double* __restrict__ X,
                                          int64_t ldx, const int32_t* __restrict__ exps, bool keys_in,
                                          int t, int64_t v, int64_t k0, bool active, double (&x)[kElems]) {
  const int raw = active ? exps[v] : 0;
  return load_scaled<SIDE>(vecs, k, X, ldx, keys_in ? key_to_sigma((uint32_t)raw, t) : raw, v, k0, active, x);
}

template <int SIDE, int RM, bool TZ>
__global__ __launch_bounds__(256) void deconstruct_kernel(int64_t vecs, int64_t vstride, int64_t k,
                                                          int64_t kp, const double* __restrict__ X,
                                                          int64_t ldx, const int32_t* __restrict__ exps,
                                                          bool keys_in, int t,
                                                          int8_t* __restrict__ planes) {
  int64_t v, g;
  group_of(blockIdx.x, vecs, v, g);
  const bool active = v < vecs && g < kp / kElems;
  const int64_t k0 = g * kElems;
  double x[kElems];
  const int sigma = load_group<SIDE>(vecs, k, X, ldx, exps, keys_in, t, v, k0, active, x);
  // the split table, built while the loads are in flight
  __shared__ uint32_t lut[kSplitTable];
  for (int i = threadIdx.x; i < kSplitTable; i += 256) lut[i] = split_16_codes(i - 256);
  __syncthreads();
  if (!active) return;
  double y[kElems];
  uint32_t ylo[kElems];
  scale_round<TZ, RM>(x, sigma, y, ylo);
  emit_all<RM>(y, ylo, planes, vstride * 128, plane_offset(vstride, kPlanes, v, g), lut);
}

// ---- all-byte set (Sec. 5.1, candidate A) on the int8 route: the centred
// residue of a byte modulus lies in [-128, 127] and is stored as it stands,
// one int8 plane per modulus (8 bytes read, 15 written per element).

template <int I, bool NT>
__device__ __forceinline__ void emit_byte_modulus(const double (&y)[kElems],
                                                  const uint32_t (&yp)[kElems / 2], int8_t* planes,
                                                  int64_t plane_stride, int64_t off) {
  constexpr int M = kModulusA[I];
  uint4 w;
  w.x = residue_bytes<M>(y[0], y[1], y[2], y[3], yp[0], yp[1]);
  w.y = residue_bytes<M>(y[4], y[5], y[6], y[7], yp[2], yp[3]);
  w.z = residue_bytes<M>(y[8], y[9], y[10], y[11], yp[4], yp[5]);
  w.w = residue_bytes<M>(y[12], y[13], y[14], y[15], yp[6], yp[7]);
  put16<NT>(planes + (int64_t)I * plane_stride + off, w);
}

template <int FIRST, bool NT, int... I>
__device__ __forceinline__ void emit_some_bytes(std::integer_sequence<int, I...>, const double (&y)[kElems],
                                                const uint32_t (&ylo)[kElems], int8_t* planes,
                                                int64_t plane_stride, int64_t off) {
  uint32_t yp[kElems / 2];
#pragma unroll
  for (int c = 0; c < kElems / 2; ++c) yp[c] = low_halves(ylo[2 * c], ylo[2 * c + 1]);
  (emit_byte_modulus<FIRST + I, NT>(y, yp, planes, plane_stride, off), ...);
}
template <int RM, bool NT = true>
__device__ __forceinline__ void emit_all_bytes(const double (&y)[kElems], const uint32_t (&ylo)[kElems],
                                               int8_t* planes, int64_t plane_stride, int64_t off) {
  if constexpr (RM != 3) {
    emit_some_bytes<0, NT>(std::make_integer_sequence<int, kRA>{}, y, ylo, planes, plane_stride, off);
  } else {
    [&]<int... G>(std::integer_sequence<int, G...>) {
      ([&] {
        constexpr double N = (double)group_product(kModulusA, G * kGroupA, kGroupA);
        double z[kElems];
        uint32_t zlo[kElems];
        reduce_group(y, N, 1.0 / N, z, zlo);
        emit_some_bytes<G * kGroupA, NT>(std::make_integer_sequence<int, kGroupA>{}, z, zlo, planes, plane_stride,
                                     off);
      }(),
       ...);
    }(std::make_integer_sequence<int, kRA / kGroupA>{});
  }
}

// RM: the residue mode (1, 2 or 3, as for residue_low).
template <int SIDE, int RM, bool TZ>
__global__ __launch_bounds__(256) void deconstruct_bytes_kernel(int64_t vecs, int64_t vstride, int64_t k,
                                                                int64_t kp, const double* __restrict__ X,
                                                                int64_t ldx,
                                                                const int32_t* __restrict__ exps,
                                                                bool keys_in, int t,
                                                                int8_t* __restrict__ planes) {
  int64_t v, g;
  group_of(blockIdx.x, vecs, v, g);
  const bool active = v < vecs && g < kp / kElems;
  if (!active) return;
  const int64_t k0 = g * kElems;
  double x[kElems], y[kElems];
  uint32_t ylo[kElems];
  const int sigma = load_group<SIDE>(vecs, k, X, ldx, exps, keys_in, t, v, k0, true, x);
  scale_round<TZ, RM>(x, sigma, y, ylo);
  emit_all_bytes<RM>(y, ylo, planes, vstride * 128, plane_offset(vstride, kRA, v, g));
}

// Both operands' byte planes in one launch, after scan_both_kernel: blocks
// below `ablocks` take A (its sigma in ea), the others B, whose column keys
// they combine from the scan's `slabs` partial maxima (in LDS: 32 vectors x 8
// threads) and whose first k block writes eb for the reconstruction.
// ablocks = 0: B alone.
template <int RM, bool TZ, bool NT>
__global__ __launch_bounds__(256) void deconstruct_bytes_both_kernel(
    int64_t ablocks, int64_t m, int64_t n, int64_t k, int64_t kp, const double* __restrict__ A, int64_t lda,
    const int32_t* __restrict__ ea, int8_t* __restrict__ pa, const double* __restrict__ B, int64_t ldb,
    const uint32_t* __restrict__ part, int slabs, int t, int32_t* __restrict__ eb, int8_t* __restrict__ pb) {
  __shared__ uint32_t keys[8][32];
  double x[kElems], y[kElems];
  uint32_t ylo[kElems];
  int64_t v, g;
  if (blockIdx.x < ablocks) {
    group_of(blockIdx.x, m, v, g);
    if (v >= m) return;
    const int sigma = load_scaled<0>(m, k, A, lda, ea[v], v, g * kElems, true, x);
    scale_round<TZ, RM>(x, sigma, y, ylo);
    emit_all_bytes<RM, NT>(y, ylo, pa, m * 128, plane_offset(m, kRA, v, g));
    return;
  }
  const int64_t block = (int64_t)blockIdx.x - ablocks, vb = (n + 31) / 32;
  group_of(block, n, v, g);
  {
    const int64_t kv = (block % vb) * 32 + (threadIdx.x & 31);
    uint32_t key = 0;
    if (kv < n) {
#pragma unroll 4
      for (int i = threadIdx.x >> 5; i < slabs; i += 8) {
        const uint32_t o = part[(int64_t)i * n + kv];
        key = o > key ? o : key;
      }
    }
    keys[threadIdx.x >> 5][threadIdx.x & 31] = key;
  }
  __syncthreads();
  const int in = (int)(v % 32);  // the thread's vector within the block
  uint32_t key = keys[0][in];
#pragma unroll
  for (int i = 1; i < 8; ++i) key = keys[i][in] > key ? keys[i][in] : key;
  if (v >= n) return;
  const int raw = key_to_sigma(key, t);
  if (g == 0) eb[v] = raw;
  const int sigma = load_scaled<1>(n, k, B, ldb, raw, v, g * kElems, true, x);
  scale_round<TZ, RM>(x, sigma, y, ylo);
  emit_all_bytes<RM, NT>(y, ylo, pb, n * 128, plane_offset(n, kRA, v, g));
}

// ---- accurate mode (Sec. 2, Eq. (alpha)): the magnitude digit of every
// element, ceil(16 |x| 2^-e) in {0..16} with e the vector's frexp exponent,
// as one int8 plane in the plane layout (the operand of the bound product).
// exps holds -e (the exponent scan at t = 0; with keys_in the column scan's
// keys).  16 |x| 2^-e is exact in FP64 unless it falls below the normal
// range, where its ceiling is 1; a non-finite vector gets zero digits.
template <int SIDE>
__global__ __launch_bounds__(256) void digits_kernel(int64_t vecs, int64_t k, int64_t kp,
                                                     const double* __restrict__ X, int64_t ldx,
                                                     const int32_t* __restrict__ exps, bool keys_in,
                                                     int8_t* __restrict__ digits) {
  int64_t v, g;
  group_of(blockIdx.x, vecs, v, g);
  if (v >= vecs || g >= kp / kElems) return;
  double x[kElems];
  const int ne = load_group<SIDE>(vecs, k, X, ldx, exps, keys_in, 0, v, g * kElems, true, x);
  int d[kElems];
#pragma unroll
  for (int c = 0; c < kElems; ++c) {
    const double a = __builtin_fabs(x[c]);
    const double u = __builtin_ceil(__builtin_ldexp(a, 4 + ne));
    d[c] = a == 0.0 ? 0 : (u < 1.0 ? 1 : (int)u);
  }
  uint4 w;
  w.x = pack_bytes(d[0], d[1], d[2], d[3]);
  w.y = pack_bytes(d[4], d[5], d[6], d[7]);
  w.z = pack_bytes(d[8], d[9], d[10], d[11]);
  w.w = pack_bytes(d[12], d[13], d[14], d[15]);
  put16(digits + plane_offset(vecs, 1, v, g), w);
}

struct DecArgs {
  int64_t blocks, vecs, vstride, k, kp;
  const double* X;
  int64_t ldx;
  const int32_t* exps;
  bool keys_in;
  int t;
  int8_t* planes;
};

template <int SIDE, bool BYTES, int RM, bool TZ>
void launch_one(const DecArgs& a, hipStream_t stream) {
  if constexpr (BYTES)
    hipLaunchKernelGGL((deconstruct_bytes_kernel<SIDE, RM, TZ>), dim3((unsigned)a.blocks), dim3(256), 0,
                       stream, a.vecs, a.vstride, a.k, a.kp, a.X, a.ldx, a.exps, a.keys_in, a.t, a.planes);
  else if constexpr (RM != 2)  // the nearest-quotient bound of RM 2 holds for byte moduli only
    hipLaunchKernelGGL((deconstruct_kernel<SIDE, RM, TZ>), dim3((unsigned)a.blocks), dim3(256), 0, stream,
                       a.vecs, a.vstride, a.k, a.kp, a.X, a.ldx, a.exps, a.keys_in, a.t, a.planes);
}

template <int SIDE, bool BYTES>
void launch_side(int rm, bool tz, const DecArgs& a, hipStream_t stream) {
  if (rm == 1) {
    if (tz) launch_one<SIDE, BYTES, 1, true>(a, stream);
    else launch_one<SIDE, BYTES, 1, false>(a, stream);
  } else if (rm == 2) {
    if (tz) launch_one<SIDE, BYTES, 2, true>(a, stream);
    else launch_one<SIDE, BYTES, 2, false>(a, stream);
  } else {
    if (tz) launch_one<SIDE, BYTES, 3, true>(a, stream);
    else launch_one<SIDE, BYTES, 3, false>(a, stream);
  }
}

}  // namespace

hipError_t launch_digits(int side, int64_t vecs, int64_t k, int64_t kp, const double* X, int64_t ldx,
                         const int32_t* exps, bool keys_in, int8_t* digits, hipStream_t stream) {
  if (vecs <= 0 || kp <= 0) return hipSuccess;
  const int64_t blocks = ((vecs + 31) / 32) * (kp / 128);
  if (blocks > (int64_t)UINT32_MAX) return hipErrorInvalidValue;
  if (side == 0)
    hipLaunchKernelGGL(digits_kernel<0>, dim3((unsigned)blocks), dim3(256), 0, stream, vecs, k, kp, X, ldx,
                       exps, keys_in, digits);
  else
    hipLaunchKernelGGL(digits_kernel<1>, dim3((unsigned)blocks), dim3(256), 0, stream, vecs, k, kp, X, ldx,
                       exps, keys_in, digits);
  return hipGetLastError();
}

hipError_t launch_deconstruct(int set, int quant, int side, int64_t vecs, int64_t vstride, int64_t k,
                              int64_t kp, int t, const double* X, int64_t ldx, const int32_t* exps,
                              bool keys_in, int8_t* planes, hipStream_t stream) {
  if (vstride < vecs || t > kMaxScaleBits) return hipErrorInvalidValue;
  if (vecs <= 0 || kp <= 0) return hipSuccess;
  const bool bytes = set == kSetBytes;
  const bool tz = quant == kQuantTZ;
  // |y| <= 2^t: ylo from kMagic, then (the byte moduli at t = 52) split off,
  // else y reduced per group of moduli first
  const int mode = t <= (bytes ? 51 : 50) ? 1 : (bytes && t == 52 ? 2 : 3);
  const DecArgs a{((vecs + 31) / 32) * (kp / 128), vecs, vstride, k, kp, X, ldx, exps, keys_in, t, planes};
  if (side == 0) {
    if (bytes) launch_side<0, true>(mode, tz, a, stream);
    else launch_side<0, false>(mode, tz, a, stream);
  } else {
    if (bytes) launch_side<1, true>(mode, tz, a, stream);
    else launch_side<1, false>(mode, tz, a, stream);
  }
  return hipGetLastError();
}

hipError_t launch_deconstruct_bytes_both(int quant, int64_t m, int64_t n, int64_t k, int64_t kp, int t,
                                         const double* A, int64_t lda, const int32_t* ea, int8_t* pa,
                                         const double* B, int64_t ldb, const uint32_t* part, int64_t slabs,
                                         int32_t* eb, int8_t* pb, hipStream_t stream) {
  if (m <= 0 || n <= 0 || kp <= 0 || slabs > INT32_MAX || t > kMaxScaleBits) return hipErrorInvalidValue;
  const int64_t ablocks = pa ? ((m + 31) / 32) * (kp / 128) : 0;
  const int64_t blocks = ablocks + ((n + 31) / 32) * (kp / 128);
  if (blocks > (int64_t)UINT32_MAX) return hipErrorInvalidValue;
  const bool tz = quant == kQuantTZ;
  const int mode = t <= 51 ? 1 : (t == 52 ? 2 : 3);  // as in launch_deconstruct
  // streaming plane stores, but for long k and planes that the last-level
  // cache holds with room plain ones, which the products then find there
  // (2048^3, 120 MiB, 198 -> 188 us a call, 900 x 700 x 4096 98.8 -> 93.1, 700 x
  // 900 x 3000 78.4 -> 73.9; within 2 % either way at 256 x 256 and 512 x 512; no
  // better at short k, nor at 2000 x 4000 x 4000, 343 MiB)
  const bool nt = kp < 2048 || kRA * (m + n) * kp > (int64_t)128 << 20;
#define OZ_BOTH(MODE, TZ, NT)                                                                                     \
  hipLaunchKernelGGL((deconstruct_bytes_both_kernel<MODE, TZ, NT>), dim3((unsigned)blocks), dim3(256), 0, stream, \
                     ablocks, m, n, k, kp, A, lda, ea, pa, B, ldb, part, (int)slabs, t, eb, pb)
#define OZ_BOTH_TZ(MODE)                  \
  if (tz && nt) OZ_BOTH(MODE, true, true); \
  else if (tz) OZ_BOTH(MODE, true, false); \
  else if (nt) OZ_BOTH(MODE, false, true); \
  else OZ_BOTH(MODE, false, false)
  if (mode == 1) {
    OZ_BOTH_TZ(1);
  } else if (mode == 2) {
    OZ_BOTH_TZ(2);
  } else {
    OZ_BOTH_TZ(3);
  }
#undef OZ_BOTH_TZ
#undef OZ_BOTH
  return hipGetLastError();
}

}  // namespace oz
