// Reconstruction (Alg. 3): Garner's mixed-radix digits of the twelve (or,
// for the all-byte set, fifteen) centred residues (Eq. (garner)), Horner
// recombination (Eq. (horner)), the lift to [-M/2, M/2), and one rounding
// of X 2^(-sigma_i - tau_j) to FP64.
// One thread per output; the residue loads coalesce along the output row.
// 24 bytes in and 8 out per output (8 more in for C -= ...): the mix of
// reads and writes bounds it at the rate of a plain copy, with the VALU work
// (about 140 instructions per output) hidden under it.
//
// Integer work per output, all exact:
//  - centred digits in one reduction each: v_j = (c_j w_j - sum_{l<j} v_l
//    R_lj) mod m_j with w_j and R_lj = (m_0..m_{l-1}) w_j mod m_j centred
//    compile-time constants.  The residue GEMM's compact int16 residues c'_j
//    are the true ones divided by a per-modulus factor f_j and reduced to
//    |c'_j| <= 0.51 m_j: the term is then c'_j (f_j w_j mod m_j).  Every
//    term is below 567 * 545 in magnitude, the sum of at most twelve below
//    2^22, so for odd m_j the FP32 quotient
//    rint(s / m_j) errs by less than 1/(2 m_j), the least distance of s / m_j
//    from a half integer: one rint and one multiply-add give the centred
//    digit.  m_j = 1024 takes the low ten bits.
//  - centred digits make X = Xl + P Xh a balanced mixed-radix number with
//    P = m_0..m_5 (even) and halves Xl = v_0 + m_0 (v_1 + ... m_4 v_5),
//    |Xl| < P, and Xh likewise over m_6..m_11 with |Xh| <= (Q-1)/2, Q odd.
//    Its range is [-M/2 - 544, M/2 - 545]; the few values below -M/2 are
//    moved up by M (Xh += Q), which gives exactly the lift to [-M/2, M/2).
//  - Horner pairs digits with 24-bit multiply-adds (|pair| < 2^20) and joins
//    the three pairs of a half in 64-bit arithmetic.
//  - |X| = H P + L with H = |Xh| < 2^53 and |L| < P, formed as a 128-bit
//    integer and rounded once.
#include <hip/hip_runtime.h>

#include <utility>

#include "dispatch.hpp"
#include "fp64_round.hpp"
#include "garner_bytes.hpp"
#include "kernels.hpp"
#include "moduli.hpp"
#include "native_dot.hpp"

namespace oz {
namespace {

// centred weight of digit l in the equation of digit j (times w_j), and w_j;
// as template variables so that they are compile-time immediates
template <int L, int J>
inline constexpr int kGarnerWeight =
    centred_const((int64_t)radix_mod(L, J) * garner_w(J) % kModulus[J], kModulus[J]);
template <int J>
inline constexpr int kGarnerW = centred_const(garner_w(J), kModulus[J]);
// the same for the residue GEMM's compact outputs, which leave out the
// factor compact_scale(j): w_j times it
template <int J>
inline constexpr int kGarnerWCompact =
    centred_const((int64_t)garner_w(J) * compact_scale(J) % kModulus[J], kModulus[J]);

constexpr bool garner_sums_fit() {
  // |c_j w_j| + sum_{l<j} |v_l R_lj| < 2^22 with |v| <= m/2 and |c| <= 0.51 m
  // (compact residues are reduced but not wrapped into the centred range)
  for (int j = 0; j < kR; ++j) {
    const int64_t mj = kModulus[j];
    int64_t s = (mj / 2 + mj / 50 + 1) * (mj / 2 + 1);
    for (int l = 0; l < j; ++l) s += (kModulus[l] / 2 + 1) * (mj / 2 + 1);
    if (s >= (int64_t)1 << 22) return false;
  }
  return true;
}
static_assert(garner_sums_fit(), "Garner sums stay below 2^22");

// The sum over earlier digits runs on v_dot2_i32_i16, two terms per
// instruction: digits and weights are centred residues, |.| <= 544, so they
// fit int16.  Word Q of the weights of digit J holds -R_lJ for l = 2Q, 2Q+1
// (0 for l >= J); word Q of the digits holds v_2Q (low half) and v_2Q+1.
constexpr uint32_t garner_pack(int q, int j) {
  uint32_t w = 0;
  for (int i = 0; i < 2; ++i) {
    const int l = 2 * q + i;
    if (l < j) {
      const int r = centred_const((int64_t)radix_mod(l, j) * garner_w(j) % kModulus[j], kModulus[j]);
      w |= (uint32_t)(-r & 0xffff) << (16 * i);
    }
  }
  return w;
}
template <int Q, int J>
inline constexpr int kGarnerPack = (int)garner_pack(Q, J);
static_assert(kModulus[0] / 2 < 32767, "centred weights and digits fit int16");

typedef short v2s __attribute__((ext_vector_type(2)));

// digit J from the residue c_J and the packed earlier digits
template <int J, bool COMPACT>
__device__ __forceinline__ void garner_digit(const int (&c)[kR], int (&v)[kR], uint32_t (&packed)[kR / 2]) {
  constexpr int M = kModulus[J];
  // every factor is below 2^11 in magnitude: 24-bit multiplies are exact
  int s = __mul24(c[J], COMPACT ? kGarnerWCompact<J> : kGarnerW<J>);
  [&]<int... Q>(std::integer_sequence<int, Q...>) {
    ((s = __builtin_amdgcn_sdot2(__builtin_bit_cast(v2s, packed[Q]),
                                 __builtin_bit_cast(v2s, kGarnerPack<Q, J>), s, false)),
     ...);
  }(std::make_integer_sequence<int, (J + 1) / 2>{});
  int d;
  if constexpr (M == 1024) {
    d = ((s + 512) & 1023) - 512;
  } else {
    const int q = (int)__builtin_rintf((float)s * (1.0f / M));
    d = s - __mul24(q, M);  // |q| < 2^13
  }
  v[J] = d;
  // an even digit opens its word (the high half's weight is 0 until the
  // odd digit fills it); an odd one completes it
  if constexpr (J % 2 == 0)
    packed[J / 2] = (uint32_t)d;
  else
    packed[J / 2] = (packed[J / 2] & 0xffffu) | ((uint32_t)d << 16);
}

// Residue q of output (row, col): a buffer load with the row's scalar base
// (row-uniform) and the column's 32-bit byte offset, shared by all twelve;
// streaming (nt), as every residue is read once.
template <typename RT>
__device__ __forceinline__ int load_residue(const RT* rowbase, int n, int col) {
  // readfirstlane returns int: take both halves as uint32_t before widening
  // (a sign-extended low half would corrupt the high one)
  const uint64_t v = (uint64_t)rowbase;
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v);
  const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
  const void* base = (const void*)(((uint64_t)hi << 32) | lo);
  const __amdgpu_buffer_rsrc_t rs =
      __builtin_amdgcn_make_buffer_rsrc((void*)base, (short)0, n * (int)sizeof(RT), 0x00020000);
  if constexpr (sizeof(RT) == 1)
    return (int)(int8_t)__builtin_amdgcn_raw_buffer_load_b8(rs, col, 0, 2);
  else if constexpr (sizeof(RT) == 2)
    return (int)(int16_t)__builtin_amdgcn_raw_buffer_load_b16(rs, col * 2, 0, 2);
  else
    return (int)__builtin_amdgcn_raw_buffer_load_b32(rs, col * 4, 0, 2);
}

// rowq: residues of this output row for modulus 0 (row-uniform); the
// modulus-q row sits mn elements further per q.  NaN on a row or column flagged
// non-finite.
template <typename RT>
__device__ __forceinline__ double reconstruct_one(const RT* rowq, int64_t mn, int n, int col, int sa,
                                                  int sb) {
  if (sa == INT32_MIN || sb == INT32_MIN) return __builtin_nan("");
  int c[kR], v[kR];
  uint32_t packed[kR / 2];
#pragma unroll
  for (int q = 0; q < kR; ++q) c[q] = load_residue(rowq + q * mn, n, col);
  [&]<int... J>(std::integer_sequence<int, J...>) {
    (garner_digit<J, sizeof(RT) == 2>(c, v, packed), ...);
  }(std::make_integer_sequence<int, kR>{});
  const int e = -sa - sb;
  double out;
  if (!round_fast(v, e, out)) out = round_exact(v, e);
  return out;
}

// ---- all-byte set (Sec. 5.1, candidate A): garner_bytes.hpp
template <typename RT>
__device__ __forceinline__ double reconstruct_one_a(const RT* rowq, int64_t mn, int n, int col,
                                                    int sa, int sb) {
  if (sa == INT32_MIN || sb == INT32_MIN) return __builtin_nan("");
  int c[kRA];
#pragma unroll
  for (int q = 0; q < kRA; ++q) c[q] = load_residue(rowq + q * mn, n, col);
  return garner_bytes(c, -sa - sb);
}

// Grid: x over 256-column strips, y over rows (strided by gridDim.y).
template <bool BYTES, typename RT>
__global__ __launch_bounds__(256) void reconstruct_kernel(int64_t m, int64_t n,
                                                          const RT* __restrict__ cres,
                                                          const int32_t* __restrict__ ea,
                                                          const int32_t* __restrict__ eb,
                                                          double* __restrict__ C, int64_t ldc,
                                                          int subtract) {
  const int64_t col = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (col >= n) return;
  const int64_t mn = m * n;
  const int sb = eb[col];
  for (int64_t row = blockIdx.y; row < m; row += gridDim.y) {
    const double r = BYTES ? reconstruct_one_a(cres + row * n, mn, (int)n, (int)col, ea[row], sb)
                           : reconstruct_one(cres + row * n, mn, (int)n, (int)col, ea[row], sb);
    // C streams through once: non-temporal load and store (with the
    // residues' nt loads, the 32768^2 update 8.14 -> 7.74 ms; the all-byte
    // set and 8192^3 unchanged)
    double* out = C + row * ldc + col;
    __builtin_nontemporal_store(subtract ? __builtin_nontemporal_load(out) - r : r, out);
  }
}

// The byte moduli's compact residues through LDS: a block takes kRun
// consecutive outputs in row-major order -- the planes are row-major without
// gaps, so rows of any length fill every lane -- and brings their kRun bytes
// of each plane in by LDS-DMA, sixteen bytes a lane.  Byte loads by the
// threads themselves (64 bytes a wavefront and plane) left too few bytes in
// flight for the memory's latency.  A thread then takes outputs tid + 256 j,
// so that C moves in whole lines.  ALIGNED: every plane starts on a dword
// (m n a multiple of 4); otherwise a plane's bytes start up to three bytes
// into its slab.
// With the CRT sum's shorter arithmetic, strips of columns against runs:
// 32768^2 C -= AB 7.6 -> 5.9 ms (5.6 TB/s), 8192^2 476 -> 413 us, 4096^2 115 ->
// 94 us, 100000 x 100 114 -> 65 us, 262144 x 8 131 -> 20 us; with Garner's
// digits runs gained nothing on square outputs.  Small and wide outputs from
// stored planes keep the strips (reconstruct_strips in dispatch.hpp).
constexpr int kRun = 1024, kSlab = kRun + 256, kPerThread = kRun / 256;
using lds_ptr_r = __attribute__((address_space(3))) void*;

// NATIVE: flagged outputs are re-issued here; else they get `fill` (NaN, or +0
// where the native re-issue's own launch supplies them).
template <bool ALIGNED, bool NATIVE>
__global__ __launch_bounds__(256) void reconstruct_runs_kernel(int64_t mn, int n, int64_t ldc,
                                                               const int8_t* __restrict__ cres,
                                                               const int32_t* __restrict__ ea,
                                                               const int32_t* __restrict__ eb,
                                                               double* __restrict__ C, int subtract,
                                                               double fill, NativeOperands nat) {
  __shared__ __attribute__((aligned(16))) int8_t slab[kRA * kSlab];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int64_t i0 = (int64_t)blockIdx.x * kRun;
  for (int q = wave; q < kRA; q += 4) {
    const int64_t at = q * mn + i0, start = ALIGNED ? at : at & ~(int64_t)3;
    // reads past the residues give zero; their last dword is read whole (the
    // residues' buffer is padded to 256 bytes)
    const int64_t left = (kRA * mn - start + 3) & ~(int64_t)3;
    const uint64_t v = (uint64_t)(cres + start);
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v), hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
        (void*)(((uint64_t)hi << 32) | lo), (short)0,
        __builtin_amdgcn_readfirstlane(left < kSlab ? (int)left : kSlab), 0x00020000);
    __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (lds_ptr_r)(slab + q * kSlab), 16, lane * 16, 0, 0, 2);
    if (!ALIGNED)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (lds_ptr_r)(slab + q * kSlab + kRun), 4, kRun + lane * 4, 0, 0, 2);
  }
  const int64_t row0 = i0 / n;
  const int col0 = (int)(i0 - row0 * n);
  const float rn = 1.0f / (float)n;
  __builtin_amdgcn_s_waitcnt(0);
  __syncthreads();
  // output o of the run: rows onward from row0 and the column; below 1024
  // columns the FP32 quotient of c + 1/2 (c < 2^11) is off by far less than the
  // 1/(2n) to an integer
  auto place = [&](int o, int& dr, int& col) __attribute__((always_inline)) {
    col = col0 + o;
    dr = n >= kRun ? (col >= n ? 1 : 0) : (int)(((float)col + 0.5f) * rn);
    col -= dr * n;
  };
  auto residues = [&](int o, int (&c)[kRA]) __attribute__((always_inline)) {
#pragma unroll
    for (int q = 0; q < kRA; ++q) c[q] = slab[q * kSlab + (ALIGNED ? 0 : (int)((q * mn + i0) & 3)) + o];
  };
  // bit j: output tid + 256 j awaits Garner's digits, or its re-issue
  unsigned declined = 0;
  [[maybe_unused]] unsigned flagged = 0;
#pragma unroll
  for (int j = 0; j < kPerThread; ++j) {
    const int o = threadIdx.x + 256 * j;
    if (i0 + o >= mn) break;
    int dr, col;
    place(o, dr, col);
    const int sa = ea[row0 + dr], sb = eb[col];
    double* out = C + (row0 + dr) * ldc + col;
    const double old = subtract ? __builtin_nontemporal_load(out) : 0.0;
    double r = fill;
    if (sa != INT32_MIN && sb != INT32_MIN) {
      int c[kRA];
      residues(o, c);
      if (!crt_bytes(c, -sa - sb, r)) {
        declined |= 1u << j;
        continue;
      }
    } else if constexpr (NATIVE) {
      flagged |= 1u << j;
      continue;
    }
    __builtin_nontemporal_store(subtract ? old - r : r, out);
  }
  // apart from the loop, whose code would hold Garner's path four times over
  // (short launches wait for their instructions)
  for (; declined; declined &= declined - 1) {
    const int o = threadIdx.x + 256 * __builtin_ctz(declined);
    int dr, col, c[kRA];
    place(o, dr, col);
    residues(o, c);
    const double r = garner_exact(c, -ea[row0 + dr] - eb[col]);
    double* out = C + (row0 + dr) * ldc + col;
    *out = subtract ? *out - r : r;
  }
  if constexpr (NATIVE) {
    if (!flagged) return;
    const auto row_of = [&](int j) __attribute__((always_inline)) {
      int dr, col;
      place(threadIdx.x + 256 * j, dr, col);
      return dr;
    };
    // a flagged row is up to four outputs of every thread: where all of the
    // wavefront's lie on one row and some thread has several, together (1024
    // columns at k = 4096 add 0.49 ms, one after another 0.77), an unflagged one
    // repeating the thread's first
    const int first = __builtin_ctz(flagged), dr0 = __builtin_amdgcn_readfirstlane(row_of(first));
    bool one_row = true;
#pragma unroll
    for (int j = 0; j < kPerThread; ++j)
      if (flagged >> j & 1) one_row = one_row && row_of(j) == dr0;
    if (__any(flagged & (flagged - 1)) && __all(one_row)) {
      uint32_t cols[kPerThread];
      double s[kPerThread];
#pragma unroll
      for (int j = 0; j < kPerThread; ++j) {
        int dr, col;
        place(threadIdx.x + 256 * (flagged >> j & 1 ? j : first), dr, col);
        cols[j] = (uint32_t)col;
      }
      native_dots<kPerThread, 4>(nat.A + (row0 + dr0) * nat.lda, nat.B, cols, nat.ldb, nat.k, s);
#pragma unroll
      for (int j = 0; j < kPerThread; ++j) {
        if (!(flagged >> j & 1)) continue;
        double* out = C + (row0 + dr0) * ldc + cols[j];
        *out = subtract ? *out - s[j] : s[j];
      }
      return;
    }
    for (; flagged; flagged &= flagged - 1) {
      int dr, col;
      place(threadIdx.x + 256 * __builtin_ctz(flagged), dr, col);
      const double d = native_dot(nat.A + (row0 + dr) * nat.lda, nat.B, (uint32_t)col, nat.ldb, nat.k);
      double* out = C + (row0 + dr) * ldc + col;
      *out = subtract ? *out - d : d;
    }
  }
}

// One block per 256 x 256 output tile (row tiles strided by gridDim.y):
// the flags of the tile's rows and columns are loaded coalesced and OR-ed
// across the block, so a tile with none -- every tile, on finite inputs --
// costs two loads and a barrier.  Otherwise each thread walks its column of
// the tile and re-issues the flagged outputs: C = dot, or C = C - dot.
// It runs apart from the reconstruction (whose loop it would slow), which
// then fills those outputs with +0: after it for C = AB, before it for
// C -= AB (C - (+0) leaves every value, NaN and infinities included, as it is).
__global__ __launch_bounds__(256) void native_reissue_kernel(int64_t m, int64_t n,
                                                             const int32_t* __restrict__ ea,
                                                             const int32_t* __restrict__ eb,
                                                             NativeOperands nat, double* C,
                                                             int64_t ldc, int subtract) {
  __shared__ int rowflag[256];
  const int64_t col = (int64_t)blockIdx.x * 256 + threadIdx.x;
  const bool colflag = col < n && eb[col] == INT32_MIN;
  const int64_t tiles = (m + 255) / 256;
  for (int64_t t = blockIdx.y; t < tiles; t += gridDim.y) {
    const int64_t row0 = t * 256, r = row0 + threadIdx.x;
    const bool rf = r < m && ea[r] == INT32_MIN;
    rowflag[threadIdx.x] = rf;
    if (__syncthreads_or(rf || colflag) && col < n) {
      const int rows = m - row0 < 256 ? (int)(m - row0) : 256;
      for (int i = 0; i < rows; ++i) {
        if (!rowflag[i] && !colflag) continue;
        const int64_t row = row0 + i;
        const double d = native_dot(nat.A + row * nat.lda, nat.B + (int64_t)blockIdx.x * 256, threadIdx.x, nat.ldb,
                                    nat.k);
        double* out = C + row * ldc + col;
        *out = subtract ? *out - d : d;
      }
    }
    __syncthreads();
  }
}

__global__ __launch_bounds__(256) void zero_c_kernel(int64_t m, int64_t n, double* C, int64_t ldc) {
  const int64_t col = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (col >= n) return;
  for (int64_t row = blockIdx.y; row < m; row += gridDim.y) C[row * ldc + col] = 0.0;
}

// Two rows per thread at least (rows y and y + gridDim.y): measured against
// one, the reconstruction of 8192^3 0.465 -> 0.397 ms (all-byte set 0.49 ->
// 0.43), of the 32768^2 x 1024 update 8.40 -> 8.08 ms (8.0 -> 7.5), same
// results; four, eight or sixteen rows, or two adjacent rows, are no better
// across shapes.
dim3 grid_for(int64_t m, int64_t n) {
  const int64_t y = (m + 1) / 2;
  return dim3((unsigned)((n + 255) / 256), (unsigned)(y < 65535 ? y : 65535));
}

hipError_t launch_native(int64_t m, int64_t n, const int32_t* ea, const int32_t* eb, const NativeOperands& nat,
                         double* C, int64_t ldc, int subtract, hipStream_t stream) {
  hipLaunchKernelGGL(native_reissue_kernel,
                     dim3((unsigned)((n + 255) / 256), (unsigned)(m < 16776960 ? (m + 255) / 256 : 65535)), dim3(256),
                     0, stream, m, n, ea, eb, nat, C, ldc, subtract);
  return hipGetLastError();
}

// The byte moduli's compact residues, in runs; the native re-issue inside
// the kernel for up to 2^22 outputs, where a launch of its own is 5 to 10 %
// of the call (1024^3: 4 of 52 us), and apart beyond.
template <bool NATIVE>
void launch_runs(int64_t m, int64_t n, const int8_t* cres, const int32_t* ea, const int32_t* eb, double* C,
                 int64_t ldc, int subtract, double fill, const NativeOperands& nat, hipStream_t stream) {
  const dim3 grid((unsigned)((m * n + kRun - 1) / kRun));
  if (m * n % 4 == 0)
    hipLaunchKernelGGL((reconstruct_runs_kernel<true, NATIVE>), grid, dim3(256), 0, stream, m * n, (int)n, ldc, cres,
                       ea, eb, C, subtract, fill, nat);
  else
    hipLaunchKernelGGL((reconstruct_runs_kernel<false, NATIVE>), grid, dim3(256), 0, stream, m * n, (int)n, ldc, cres,
                       ea, eb, C, subtract, fill, nat);
}

template <bool BYTES, typename RT>
hipError_t launch_rec(int64_t m, int64_t n, const RT* cres, const int32_t* ea, const int32_t* eb,
                      double* C, int64_t ldc, int subtract, const NativeOperands& nat,
                      hipStream_t stream) {
  if (m <= 0 || n <= 0) return hipSuccess;
  constexpr bool RUNS = BYTES && sizeof(RT) == 1;
  const bool strips = !RUNS || (!nat.A && reconstruct_strips(m, n));
  if (!strips && (m * n + kRun - 1) / kRun > (int64_t)UINT32_MAX) return hipErrorInvalidValue;
  const bool inside = RUNS && nat.A && m * n <= 1 << 22, apart = nat.A && !inside;
  const double fill = nat.A ? 0.0 : __builtin_nan("");
  if (apart && subtract) {
    const hipError_t e = launch_native(m, n, ea, eb, nat, C, ldc, subtract, stream);
    if (e != hipSuccess) return e;
  }
  if (strips) {
    hipLaunchKernelGGL((reconstruct_kernel<BYTES, RT>), grid_for(m, n), dim3(256), 0, stream, m, n, cres, ea, eb, C,
                       ldc, subtract);
  } else if constexpr (RUNS) {
    if (inside)
      launch_runs<true>(m, n, cres, ea, eb, C, ldc, subtract, fill, nat, stream);
    else
      launch_runs<false>(m, n, cres, ea, eb, C, ldc, subtract, fill, nat, stream);
  }
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess || !apart || subtract) return e;
  return launch_native(m, n, ea, eb, nat, C, ldc, subtract, stream);
}

}  // namespace

hipError_t launch_reconstruct_i32(int64_t m, int64_t n, const int32_t* cres, const int32_t* ea,
                                  const int32_t* eb, double* C, int64_t ldc, int subtract,
                                  hipStream_t stream) {
  return launch_rec<false, int32_t>(m, n, cres, ea, eb, C, ldc, subtract, NativeOperands{}, stream);
}

hipError_t launch_reconstruct_i16(int64_t m, int64_t n, const int16_t* cres, const int32_t* ea,
                                  const int32_t* eb, double* C, int64_t ldc, int subtract,
                                  hipStream_t stream) {
  return launch_rec<false, int16_t>(m, n, cres, ea, eb, C, ldc, subtract, NativeOperands{}, stream);
}

hipError_t launch_reconstruct_bytes_i32(int64_t m, int64_t n, const int32_t* cres,
                                        const int32_t* ea, const int32_t* eb, double* C,
                                        int64_t ldc, int subtract, hipStream_t stream) {
  return launch_rec<true, int32_t>(m, n, cres, ea, eb, C, ldc, subtract, NativeOperands{}, stream);
}

hipError_t launch_reconstruct_bytes_i8(int64_t m, int64_t n, const int8_t* cres, const int32_t* ea,
                                       const int32_t* eb, double* C, int64_t ldc, int subtract,
                                       const NativeOperands& nat, hipStream_t stream) {
  return launch_rec<true, int8_t>(m, n, cres, ea, eb, C, ldc, subtract, nat, stream);
}

hipError_t launch_zero_c(int64_t m, int64_t n, double* C, int64_t ldc, hipStream_t stream) {
  if (m <= 0 || n <= 0) return hipSuccess;
  hipLaunchKernelGGL(zero_c_kernel, grid_for(m, n), dim3(256), 0, stream, m, n, C, ldc);
  return hipGetLastError();
}

}  // namespace oz
