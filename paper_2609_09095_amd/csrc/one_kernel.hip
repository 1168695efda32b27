// The whole emulated product (Alg. 1) in one launch, for products small
// enough that launches and their drains, not work, bound the staged path
// (eight kernels of 1.5 to 15 us each at 512^3).
//
// A block owns a 32 x 32 output tile: it scans its 32 rows of A and 32
// columns of B for their exponents, then walks k in chunks of 64 --
// quantising its 64 vectors' slices, reducing them to the fifteen byte
// residues straight into LDS, and multiplying on v_mfma_i32_32x32x32_i8 with
// wavefront w owning modulus w -- and reconstructs its outputs from the
// residues, exchanged through LDS.  Nothing but A, B and C touches memory.
//
// The conversion bounds it: every element is converted once per tile row or
// column it serves, 4 elements per thread and chunk at about 44 VALU
// instructions each, so a block takes a few us plus about 1.5 us per chunk
// whatever the matrix cores do.  32 x 32 tiles rather than 64 x 64 (half the
// conversions per output) because the path is for sizes whose 64 x 64 tiles
// would leave most CUs idle.  Two LDS buffers (120 KiB) so that one barrier
// per chunk suffices: a chunk's products run while faster wavefronts convert
// the next one.
#include <utility>

#include "dispatch.hpp"
#include "exponent_key.hpp"
#include "garner_bytes.hpp"
#include "kernels.hpp"
#include "moduli.hpp"
#include "native_dot.hpp"
#include "residues.hpp"

namespace oz {
namespace {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v16i __attribute__((ext_vector_type(16)));

constexpr int OT = 32;        // output tile edge
constexpr int OK = 64;        // k per chunk
constexpr int OE = 4;         // k per thread and chunk
constexpr int OSLAB = OT * OK;  // bytes of one modulus's slab
static_assert(kRA <= 16, "one modulus per wavefront");
// sums of int8 products stay in int32
static_assert(kOneKernelMaxK * 128 * 128 < (int64_t)INT32_MAX, "exact int32 sums");

__constant__ int kModO[16] = {kModulusA[0],  kModulusA[1],  kModulusA[2],  kModulusA[3],
                              kModulusA[4],  kModulusA[5],  kModulusA[6],  kModulusA[7],
                              kModulusA[8],  kModulusA[9],  kModulusA[10], kModulusA[11],
                              kModulusA[12], kModulusA[13], kModulusA[14], 1};

// 64-byte rows: the 16-byte chunk index XOR-ed with bits 1-2 and bit 3 of the
// row, so that fragment reads of consecutive rows hit distinct banks
__device__ __forceinline__ int oswz(int row) { return ((row >> 1) & 3) ^ ((row >> 3) & 1); }

// four residue bytes of every modulus FIRST + I into its slab
template <int FIRST, int... I>
__device__ __forceinline__ void put_residues(std::integer_sequence<int, I...>, const double (&y)[OE],
                                             const uint32_t (&ylo)[OE], int8_t* slab) {
  const uint32_t y01 = low_halves(ylo[0], ylo[1]), y23 = low_halves(ylo[2], ylo[3]);
  ((*reinterpret_cast<uint32_t*>(slab + (FIRST + I) * OSLAB) =
        residue_bytes<kModulusA[FIRST + I]>(y[0], y[1], y[2], y[3], y01, y23)),
   ...);
}

// RM: the residue mode (1, 2 or 3, as for residue_low)
template <int RM, bool TZ>
__global__ __launch_bounds__(1024) void one_kernel(int m, int n, int k, int tiles_n, const double* __restrict__ A,
                                                   int64_t lda, const double* __restrict__ B, int64_t ldb,
                                                   int t, double* __restrict__ C, int64_t ldc, int subtract) {
  // [buffer][side][modulus][slab]
  __shared__ __attribute__((aligned(1024))) int8_t lds[2][2][kRA * OSLAB];
  __shared__ uint32_t part[8][OT];  // column maxima of each wavefront of side 1
  __shared__ int sig[2][OT];        // sigma of the tile's rows, tau of its columns
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int row0 = (int)(blockIdx.x / (unsigned)tiles_n) * OT, col0 = (int)(blockIdx.x % (unsigned)tiles_n) * OT;

  // conversion: wavefronts 0-7 take A, a row's 16 lanes 4 consecutive k each;
  // wavefronts 8-15 take B, 32 lanes along the columns
  const bool isb = wave >= 8;
  const int vec = isb ? lane & 31 : 4 * wave + (lane >> 4);
  const int kg = isb ? 2 * (wave - 8) + (lane >> 5) : lane & 15;
  const bool live = isb ? col0 + vec < n : row0 + vec < m;
  const int at = vec * OK + (((kg >> 2) ^ oswz(vec)) << 4) + 4 * (kg & 3);

  // the thread's elements of chunk s, through a buffer resource at the
  // chunk's first element: 32-bit byte offsets (the host takes this path for
  // leading dimensions up to kOneKernelMaxLd), and past k or past the matrix
  // an offset beyond the resource, which reads zero without a branch
  const double* base = isb ? B + col0 : A + (int64_t)row0 * lda;
  const int64_t chunk_step = isb ? OK * ldb : OK;
  const int estep = isb ? (int)ldb * 8 : 8;
  const int voff = isb ? vec * 8 + OE * kg * estep : vec * (int)lda * 8 + OE * kg * 8;
  constexpr int kRecords = 0x7FFFFFFF, kBeyond = (int)0x80000000;
  auto load = [&](int s, double (&x)[OE]) __attribute__((always_inline)) {
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
        (void*)(base + s * chunk_step), (short)0, kRecords, 0x00020000);
    const int left = live ? k - s * OK - OE * kg : 0;  // valid elements from here
#pragma unroll
    for (int c = 0; c < OE; ++c)
      x[c] = __builtin_bit_cast(
          double, __builtin_amdgcn_raw_buffer_load_b64(rs, c < left ? voff + c * estep : kBeyond, 0, 0));
  };

  const int chunks = (k + OK - 1) / OK;
  double x[OE], xn[OE];
  // exponent scan, last chunk first: chunk 0 stays in registers
  uint64_t mx = 0;
#pragma unroll 4
  for (int s = chunks - 1; s >= 0; --s) {
    load(s, x);
#pragma unroll
    for (int c = 0; c < OE; ++c) {
      const uint64_t a = __builtin_bit_cast(uint64_t, x[c]) & kAbsMask;
      mx = a > mx ? a : mx;
    }
  }
  uint32_t key = exponent_key(mx);
  if (!isb) {
#pragma unroll
    for (int off = 8; off > 0; off >>= 1) {
      const uint32_t o = (uint32_t)__shfl_xor((int)key, off, 64);
      key = o > key ? o : key;
    }
    if ((lane & 15) == 0) sig[0][vec] = key_to_sigma(key, t);
  } else {
    const uint32_t o = (uint32_t)__shfl_xor((int)key, 32, 64);
    key = o > key ? o : key;
    if (lane < 32) part[wave - 8][lane] = key;
  }
  __syncthreads();
  if (tid < OT) {
    uint32_t mk = part[0][tid];
#pragma unroll
    for (int w = 1; w < 8; ++w) mk = part[w][tid] > mk ? part[w][tid] : mk;
    sig[1][tid] = key_to_sigma(mk, t);
  }
  __syncthreads();
  const int sv = sig[isb][vec];
  const bool dead = sv == INT32_MIN;  // a non-finite vector: zero planes
  const int sigma = dead ? 0 : sv;

  v16i acc{};
  const int fr = lane & 31, fh = lane >> 5;
  for (int s = 0; s < chunks; ++s) {
    if (s + 1 < chunks) load(s + 1, xn);
    if (dead) {
#pragma unroll
      for (int c = 0; c < OE; ++c) x[c] = 0.0;
    }
    double y[OE];
    uint32_t ylo[OE];
    scale_round<TZ, RM>(x, sigma, y, ylo);
    int8_t* slab = &lds[s & 1][isb][at];
    if constexpr (RM != 3) {
      put_residues<0>(std::make_integer_sequence<int, kRA>{}, y, ylo, slab);
    } else {
      [&]<int... G>(std::integer_sequence<int, G...>) {
        ([&] {
          constexpr double N = (double)group_product(kModulusA, G * kGroupA, kGroupA);
          double z[OE];
          uint32_t zlo[OE];
          reduce_group(y, N, 1.0 / N, z, zlo);
          put_residues<G * kGroupA>(std::make_integer_sequence<int, kGroupA>{}, z, zlo, slab);
        }(),
         ...);
      }(std::make_integer_sequence<int, kRA / kGroupA>{});
    }
    // the other buffer was last read before the previous barrier
    __syncthreads();
    if (wave < kRA) {
      const int8_t* sa = &lds[s & 1][0][wave * OSLAB + fr * OK];
      const int8_t* sb = &lds[s & 1][1][wave * OSLAB + fr * OK];
#pragma unroll
      for (int ks = 0; ks < OK / 32; ++ks) {
        const int o = ((2 * ks + fh) ^ oswz(fr)) << 4;
        acc = __builtin_amdgcn_mfma_i32_32x32x32_i8(*reinterpret_cast<const v4i*>(sa + o),
                                                    *reinterpret_cast<const v4i*>(sb + o), acc, 0, 0, 0);
      }
    }
#pragma unroll
    for (int c = 0; c < OE; ++c) x[c] = xn[c];
  }

  // centred residues, 16 bytes per output, into the buffer that the last
  // chunk did not use (last read before the last barrier)
  int8_t* res = lds[chunks & 1][0];
  if (wave < kRA) {
    const double md = (double)kModO[wave], minv = 1.0 / md;
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      const int row = 8 * (v >> 2) + 4 * fh + (v & 3);
      const double xd = (double)acc[v];
      // (+m/2 of m = 256 stores as -128)
      res[(row * OT + fr) * 16 + wave] = (int8_t)(int)__builtin_fma(-__builtin_rint(xd * minv), md, xd);
    }
  }
  __syncthreads();
  const int row = tid >> 5, col = tid & 31;
  if (row0 + row < m && col0 + col < n) {
    const v4i w = *reinterpret_cast<const v4i*>(res + tid * 16);
    const int sa = sig[0][row], sb = sig[1][col];
    double r;
    if (sa == INT32_MIN || sb == INT32_MIN) {
      r = native_dot(A + (int64_t)(row0 + row) * lda, B + col0, (uint32_t)col, ldb, k);
    } else {
      int c[kRA];
#pragma unroll
      for (int q = 0; q < kRA; ++q) c[q] = (int)(int8_t)(w[q >> 2] >> (8 * (q & 3)));
      r = garner_bytes(c, -sa - sb);
    }
    double* out = C + (int64_t)(row0 + row) * ldc + col0 + col;
    *out = subtract ? *out - r : r;
  }
}

}  // namespace

hipError_t launch_one_kernel(int quant, int64_t m, int64_t n, int64_t k, int t, const double* A, int64_t lda,
                             const double* B, int64_t ldb, double* C, int64_t ldc, int subtract,
                             hipStream_t stream) {
  if (m <= 0 || n <= 0) return hipSuccess;
  const int64_t tm = (m + OT - 1) / OT, tn = (n + OT - 1) / OT;
  if (k < 1 || k > kOneKernelMaxK || lda > kOneKernelMaxLd || ldb > kOneKernelMaxLd || m > kOneKernelMaxVecs ||
      n > kOneKernelMaxVecs || tm * tn > INT32_MAX || t > kMaxScaleBits)
    return hipErrorInvalidValue;
  const bool tz = quant == kQuantTZ;
  // |y| <= 2^t, as in the deconstruction of the byte moduli
  const int mode = t <= 51 ? 1 : (t == 52 ? 2 : 3);
#define OZ_ONE(MODE, TZ)                                                                                        \
  hipLaunchKernelGGL((one_kernel<MODE, TZ>), dim3((unsigned)(tm * tn)), dim3(1024), 0, stream, (int)m, (int)n, \
                     (int)k, (int)tn, A, lda, B, ldb, t, C, ldc, subtract)
  if (mode == 1 && tz) OZ_ONE(1, true);
  else if (mode == 1) OZ_ONE(1, false);
  else if (mode == 2 && tz) OZ_ONE(2, true);
  else if (mode == 2) OZ_ONE(2, false);
  else if (tz) OZ_ONE(3, true);
  else OZ_ONE(3, false);
#undef OZ_ONE
  return hipGetLastError();
}

}  // namespace oz
