// Storage mode F for A in tall/skinny products (Alg. 1's storage modes,
// Sec. 6.2: the hybrid of a materialised small operand and a streamed large
// one), all-byte set: B's residue planes are stored once, while A is read
// as FP64 inside the product kernel -- scaled by 2^sigma, quantised and
// reduced to its byte residues per K stage (Eq. (scale), Alg. 2) straight
// into LDS, never written to HBM as planes.  For at most 128 columns one
// output tile spans all of B (lambda_A = 1: every element of A is converted
// once per modulus it serves).
//
// A block owns 128 rows of A, all (at most 128) columns and G = 5 moduli, or G =
// 3 where so few strips leave CUs idle (fused_moduli in dispatch.hpp); its
// 16 wavefronts convert a 128 x 64 slab per stage, then multiply it with B's
// slabs on v_mfma_i32_32x32x32_i8 (32 x 32 outputs per wavefront and
// modulus), the next slab's FP64 loads in flight meanwhile.  The blocks of one
// row strip (15 / G of them) are dealt to the same XCD back to back, so the
// strip's FP64 comes from HBM once and from that XCD's L2 for the others.
//
// VALU work bounds it (61 % of the cycles with G = 3, the matrix cores 19 %,
// and the stage barriers keep the two phases apart), and loads, quantising
// and addresses are paid once per group of moduli: three moduli per block
// took 5.53 ms at 262144 x 128 x 4096, five 4.64 ms.  Five fit 128 registers
// (80 accumulators) because a row's FP64 values are reloaded in place as soon
// as they are converted, one stage ahead (two sets, two stages ahead, were
// worth 3 % with three moduli), addresses are 32-bit offsets recomputed from
// the lane index, and no masks are kept.
#include "dispatch.hpp"
#include "kernels.hpp"
#include "moduli.hpp"
#include "residues.hpp"

namespace oz {
namespace {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v16i __attribute__((ext_vector_type(16)));

constexpr int FBN = 128;   // columns of B (all of them)
constexpr int FBK = 64;    // k per stage
constexpr int kSegF = 1024;  // stages (65536 k) between reductions of the int32 sums
// residue bytes in [-128, 127]: products up to 2^14 in magnitude; the sums of
// kSegF stages, plus the largest value a reduction leaves, fit in int32
static_assert((int64_t)kSegF * FBK * 128 * 128 + 128 < (int64_t)INT32_MAX, "int32 sums exact between reductions");

__constant__ int kModF[kRA] = {kModulusA[0],  kModulusA[1],  kModulusA[2],  kModulusA[3],
                               kModulusA[4],  kModulusA[5],  kModulusA[6],  kModulusA[7],
                               kModulusA[8],  kModulusA[9],  kModulusA[10], kModulusA[11],
                               kModulusA[12], kModulusA[13], kModulusA[14]};
__constant__ double kModD[kRA] = {kModulusA[0],  kModulusA[1],  kModulusA[2],  kModulusA[3],
                                  kModulusA[4],  kModulusA[5],  kModulusA[6],  kModulusA[7],
                                  kModulusA[8],  kModulusA[9],  kModulusA[10], kModulusA[11],
                                  kModulusA[12], kModulusA[13], kModulusA[14]};
// RN(1/m) for the quotient route; 0 for m = 256, whose residue
// byte is the low byte of y itself
__constant__ double kInvQ[kRA] = {
    0.0,                 1.0 / kModulusA[1],  1.0 / kModulusA[2],  1.0 / kModulusA[3],
    1.0 / kModulusA[4],  1.0 / kModulusA[5],  1.0 / kModulusA[6],  1.0 / kModulusA[7],
    1.0 / kModulusA[8],  1.0 / kModulusA[9],  1.0 / kModulusA[10], 1.0 / kModulusA[11],
    1.0 / kModulusA[12], 1.0 / kModulusA[13], 1.0 / kModulusA[14]};
static_assert(kModulusA[0] == 256, "the power of two comes first");
// RN(1/m) for the reductions of the int32 sums
__constant__ double kInvF[kRA] = {
    1.0 / kModulusA[0],  1.0 / kModulusA[1],  1.0 / kModulusA[2],  1.0 / kModulusA[3],
    1.0 / kModulusA[4],  1.0 / kModulusA[5],  1.0 / kModulusA[6],  1.0 / kModulusA[7],
    1.0 / kModulusA[8],  1.0 / kModulusA[9],  1.0 / kModulusA[10], 1.0 / kModulusA[11],
    1.0 / kModulusA[12], 1.0 / kModulusA[13], 1.0 / kModulusA[14]};

// mode 3's group products N (below 2^24 for G = 3, 2^40 for G = 5) and RN(1/N)
template <int G>
struct GroupConst {
  static_assert(groups_in_range(kModulusA, G), "one exact reduction per group");
  double n[kRA / G], inv[kRA / G];
};
template <int G>
constexpr GroupConst<G> make_groups() {
  GroupConst<G> r{};
  for (int i = 0; i < kRA / G; ++i) {
    double p = 1.0;
    for (int j = 0; j < G; ++j) p *= kModulusA[i * G + j];
    r.n[i] = p;
    r.inv[i] = 1.0 / p;
  }
  return r;
}
template <int G>
__constant__ GroupConst<G> kGroupF = make_groups<G>();

// y mod 2^32 of an integer-valued y with |y| <= 2^52, where y + 1.5 2^52 is
// no longer exact: h = floor(y 2^-32) (the scaling is exact), y - h 2^32 in
// [0, 2^32) by one exact FMA, converted.
__device__ __forceinline__ uint32_t low32_split(double y) {
  const double h = __builtin_floor(y * 0x1p-32);
  return (uint32_t)__builtin_fma(-h, 0x1p32, y);
}

// LDS slabs: rows of 64 bytes (one stage), the 16-byte chunk index XOR-ed
// with bits 1-2 of the row and then with bit 3, so that the fragment reads
// at one chunk of 8 consecutive rows (128 bytes a cycle) and of 16 (256
// bytes a cycle) hit distinct 16-byte bank groups.
__device__ __forceinline__ int fswz(int row) { return ((row >> 1) & 3) ^ ((row >> 3) & 1); }

// int8 fragment of a 32-row block for one 32-byte K step of a 64-byte stage:
// lane half fh takes chunk 2 ks + fh of its row
__device__ __forceinline__ v4i ffrag(const int8_t* base, int r, int ks, int fh) {
  return *reinterpret_cast<const v4i*>(base + r * FBK + (((2 * ks + fh) ^ fswz(r)) << 4));
}

__device__ __forceinline__ const int8_t* uniform_ptr_f(const int8_t* p) {
  const uint64_t v = (uint64_t)p;
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v);
  const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
  return (const int8_t*)(((uint64_t)hi << 32) | lo);
}

using lds_ptr_f = __attribute__((address_space(3))) void*;

// The lane index, computed afresh where it is used. The fused kernel runs
// at the register limit, and a lane offset held across the k loop is
// spilled; its reload from scratch waits on the vector-memory counter and
// so drains the look-ahead loads with it. A volatile asm is neither hoisted
// nor merged.
__device__ __forceinline__ int lane_now() {
  int l;
  asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=v"(l));
  return l;
}

// End of a pipeline stage. Each wave waits for its own LDS writes and its
// LDS-DMA, then the workgroup meets at the barrier. When keep_a is set, the
// last four vector loads (A's FP64 values for the stage after next, issued
// after the DMA) may stay outstanding: vmcnt(4) expcnt(0) lgkmcnt(0). Any
// other load path issues at least four loads there, and the counter retires
// in issue order. The barrier is a bare instruction behind a compiler memory
// barrier, because the release fence of __syncthreads() drains every
// outstanding vector load.
__device__ __forceinline__ void stage_barrier(bool keep_a) {
  if (keep_a)
    __builtin_amdgcn_s_waitcnt(0x0004);
  else
    __builtin_amdgcn_s_waitcnt(0);
  asm volatile("s_barrier" ::: "memory");
}

// Centred residue of an int32 sum modulo m (as cmod_i32 in the residue GEMM).
// m as a double from the table: converted in the kernel it would be held in
// vector registers across the k loop.
__device__ __forceinline__ int cmod_sum(int x, double m, double minv) {
  const double xd = (double)x;
  const double q = __builtin_rint(xd * minv);
  return (int)__builtin_fma(-q, m, xd);
}

// 128 rows of A per block, 16 wavefronts: wavefront w converts rows
// 8 w .. 8 w + 7 of each slab and owns the 32 x 32 outputs (w / 4, w % 4) of
// every modulus of its group.
constexpr int FBM = kFusedRows;
// Leading dimensions of A below this go through a buffer resource: 8 lda is
// then a positive signed 24-bit factor and 128 rows stay below 2^31 bytes.
constexpr int64_t kBufLda = (int64_t)1 << 20;
static_assert(8 * (kBufLda - 1) < (1 << 23) && FBM * 8 * kBufLda < (int64_t)1 << 31, "row offsets of the buffer loads");
// MODE: the residue route by the range of y -- 1: ylo = y + 1.5 2^52
// (|y| <= 2^51); 2: ylo by low32_split (|y| <= 2^52); 3: y first reduced
// modulo the product of the block's G moduli, which keeps their residues,
// by one rounded quotient and one exact FMA, then mode 1 (|y| <= 2^58).
template <int G, int MODE, bool TZ, bool BUF>
__global__ __launch_bounds__(1024, 1) void fused_bytes_kernel(
    int64_t m, int64_t n, int64_t k, int64_t kp, const double* __restrict__ A, int64_t lda,
    const int32_t* __restrict__ sigma, const int8_t* __restrict__ pb, int8_t* __restrict__ cres,
    int64_t strips) {
  static_assert(kRA % G == 0, "modulus groups");
  constexpr int NG = kRA / G;
  // two buffers of each, every buffer its own LDS object: the compiler then
  // tells the buffer that LDS-DMA fills from the one being read, and does
  // not wait for the DMA before the reads
  __shared__ __attribute__((aligned(1024))) int8_t lds_a0[G][FBM * FBK];
  __shared__ __attribute__((aligned(1024))) int8_t lds_a1[G][FBM * FBK];
  __shared__ __attribute__((aligned(1024))) int8_t lds_b0[G][FBN * FBK];
  __shared__ __attribute__((aligned(1024))) int8_t lds_b1[G][FBN * FBK];
  // block -> (strip, group): the NG blocks of a strip go to one XCD (block b
  // runs on XCD b % 8), one after the other
  const uint32_t b = blockIdx.x, o = b >> 3;
  const int64_t strip = (int64_t)(o / NG) * 8 + (b & 7);
  const int grp = (int)(o % NG);
  if (strip >= strips) return;
  const int64_t row0 = strip * FBM;

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wr = wave >> 2, wc = wave & 3;  // 4 x 4 wavefronts of 32 x 32 outputs
  const int fr = lane & 31, fh = lane >> 5;

  // conversion: lane l takes k = 2 (l % 16), + 1 and the same 32 on of row
  // 8 wave + 4 i + l / 16, i = 0, 1: 16 lanes sweep a row's 512 bytes in two
  // loads of whole cache lines (four consecutive k per lane, each line
  // touched by both loads, cost 3 %)
  int sg[2];
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int r = 8 * wave + 4 * i + (lane >> 4);
    const int64_t arow = row0 + r;
    const bool ok = arow < m;
    const int sv = ok ? sigma[arow] : 0;
    const bool live = ok && sv != INT32_MIN;
    sg[i] = live ? sv : 0;
  }

  int mods[G];
  double qinv[G];
#pragma unroll
  for (int g = 0; g < G; ++g) {
    mods[g] = kModF[grp * G + g];
    qinv[g] = kInvQ[grp * G + g];
  }
  const double gn = kGroupF<G>.n[grp], gninv = kGroupF<G>.inv[grp];

  const int nstage = (int)(kp / FBK);
  // x[4 i + c]: row 8 wave + 4 i + lane / 16, k = 2 (lane % 16) + c % 2 +
  // 32 (c / 2) of the next stage to convert; a row's four are reloaded for
  // the stage after it as soon as they are converted.
  // x holds the raw values.  Nothing is masked: rows past m feed outputs that
  // are not stored, rows holding a NaN or an infinity outputs that the
  // reconstruction replaces, and k past the end meets B's zero padding, so
  // any residue bytes will do there.  Whole stages take the 16-byte loads,
  // the last, partial one clamped single loads; full: stage s is known to
  // lie inside k.
  // BUF: whole stages read the strip's rows through one buffer resource, at
  // 32-bit byte offsets from its first row by signed 24-bit products (the host
  // takes it for lda < kBufLda only, so that a row's bytes fit one and 128
  // rows stay below 2^31); rows past m read as zero, and a row may start at
  // any double.
  const int lda8 = (int)(lda * 8);
  const int arec = BUF ? (int)((m - row0 < FBM ? m - row0 : FBM) * lda8) : 0;
  const __amdgpu_buffer_rsrc_t ars = __builtin_amdgcn_make_buffer_rsrc(
      (void*)uniform_ptr_f((const int8_t*)(A + row0 * lda)), (short)0, arec, 0x00020000);
  double x[8];
  auto load_a = [&](int i, int s, bool full) __attribute__((always_inline)) {
    const int l = lane_now();
    if (BUF && (full || (int64_t)s * FBK + FBK <= k)) {
      const int off = __mul24(8 * wave + 4 * i + (l >> 4), lda8) + 16 * (l & 15);
      const int so = s * FBK * 8;
      const double2 p = __builtin_bit_cast(double2, __builtin_amdgcn_raw_buffer_load_b128(ars, off, so, 0));
      const double2 q = __builtin_bit_cast(double2, __builtin_amdgcn_raw_buffer_load_b128(ars, off + 256, so, 0));
      x[4 * i] = p.x;
      x[4 * i + 1] = p.y;
      x[4 * i + 2] = q.x;
      x[4 * i + 3] = q.y;
    } else {
      const int64_t arow = row0 + 8 * wave + 4 * i + (l >> 4);
      const double* row = A + (arow < m ? arow : m - 1) * lda;
      const int64_t k0 = (int64_t)s * FBK + 2 * (l & 15);
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        const int64_t kk = k0 + (c & 1) + 32 * (c >> 1);
        x[4 * i + c] = row[kk < k ? kk : k - 1];
      }
    }
  };
  // two byte pairs per row and modulus: k = ck, ck + 1 in chunk ck / 16 of
  // the row, swizzled, and k + 32 two chunks on
  auto convert = [&](int i, int buf) __attribute__((always_inline)) {
    const int l = lane_now(), ck = 2 * (l & 15);
    const int r = 8 * wave + 4 * i + (l >> 4);
    double y[4];
    uint32_t ylo[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const double v = __builtin_ldexp(x[4 * i + c], sg[i]);
      y[c] = TZ ? __builtin_trunc(v) : __builtin_rint(v);
      if constexpr (MODE == 3) y[c] = __builtin_fma(-__builtin_rint(y[c] * gninv), gn, y[c]);
      ylo[c] = MODE == 2 ? low32_split(y[c]) : low_word(y[c] + kMagic);
    }
    const uint32_t y01 = low_halves(ylo[0], ylo[1]), y23 = low_halves(ylo[2], ylo[3]);
    const int at = r * FBK + (((ck >> 4) ^ fswz(r)) << 4) + (ck & 15);
#pragma unroll
    for (int g = 0; g < G; ++g) {
      // for M = 256 (RN(1/M) taken as 0) q = 0: y's own low bytes
      const uint32_t word = residue_bytes(y[0], y[1], y[2], y[3], y01, y23,
                                          u16x2{(uint16_t)-mods[g], (uint16_t)-mods[g]}, qinv[g]);
      int8_t* slab = (buf ? lds_a1 : lds_a0)[g];
      *reinterpret_cast<uint16_t*>(slab + at) = (uint16_t)word;
      *reinterpret_cast<uint16_t*>(slab + (at ^ 32)) = (uint16_t)(word >> 16);
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  // B's slabs of stage s: for each of the G moduli, 128 rows x 64 bytes,
  // by LDS-DMA (eight 1 KiB loads per modulus, spread over the wavefronts):
  // lane l lands at row 16 d + l / 4, physical chunk l % 4, and fetches
  // the global chunk that the swizzle puts there; columns past n read zero.
  const int brecs = __builtin_amdgcn_readfirstlane((int)(n * 128));
  auto load_b = [&](int s, int buf) __attribute__((always_inline)) {
    const int64_t kb = s >> 1, h = s & 1;
#pragma unroll
    for (int j = 0; j < (8 * G + 15) / 16; ++j) {
      const int d = wave + 16 * j;
      if (d >= 8 * G) break;
      const int g = d >> 3, dd = d & 7;
      const int mod = grp * G + g;
      const int8_t* piece = uniform_ptr_f(pb + ((kb * kRA + mod) * n) * 128 + h * 64);
      const __amdgpu_buffer_rsrc_t rs =
          __builtin_amdgcn_make_buffer_rsrc((void*)piece, (short)0, brecs, 0x00020000);
      const int row = 16 * dd + (lane >> 2);
      const int gchunk = (lane & 3) ^ fswz(row);
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (lds_ptr_f)(&(buf ? lds_b1 : lds_b0)[g][16 * dd * FBK]), 16,
                                               row * 128 + gchunk * 16, 0, 0, 0);
    }
  };

  v16i acc[G];
#pragma unroll
  for (int g = 0; g < G; ++g) acc[g] = v16i{};

  // stage s: the MFMAs of stage s run on the LDS buffers cur = s % 2, then
  // stage s + 1 (loaded during stage s - 1) is converted into the other
  // buffers, each row's values giving way to its loads of stage s + 2.
  // inner: a stage of the main loop, whose next stage exists and whose
  // look-ahead stage lies inside k. The look-ahead there is unconditional
  // and takes one load path, so that the compiler sees every look-ahead
  // register consumed and keeps the loads in flight across the barrier.
  // B's DMA goes out before A's loads, so that the end-of-stage wait can
  // leave the latter outstanding.
  auto step = [&](int s, int cur, bool inner) __attribute__((always_inline)) {
    const int nxt = cur ^ 1;
    const bool next = inner || s + 1 < nstage;
    const bool more = inner || s + 2 < nstage;
    if (next) load_b(s + 1, nxt);
    // the lane's fragment offsets recomputed (lane_now), not held
    const int l = lane_now(), r = l & 31, f = l >> 5;
#pragma unroll
    for (int g = 0; g < G; ++g) {
      const int8_t* la = (cur ? lds_a1 : lds_a0)[g];
      const int8_t* lb = (cur ? lds_b1 : lds_b0)[g];
#pragma unroll
      for (int ks = 0; ks < 2; ++ks)
        acc[g] = __builtin_amdgcn_mfma_i32_32x32x32_i8(ffrag(la, wr * 32 + r, ks, f),
                                                       ffrag(lb, wc * 32 + r, ks, f), acc[g], 0, 0, 0);
      // one modulus's fragments at a time in registers
      __builtin_amdgcn_sched_barrier(0);
    }
    if (next) {
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        // one row's values at a time in registers
        __builtin_amdgcn_sched_barrier(0);
        convert(i, nxt);
        __builtin_amdgcn_sched_barrier(0);
        if (more) load_a(i, s + 2, inner);
      }
    }
    if (((s + 1) % kSegF) == 0 && next) {
#pragma unroll
      for (int g = 0; g < G; ++g)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[g][v] = cmod_sum(acc[g][v], kModD[grp * G + g], kInvF[grp * G + g]);
    }
    stage_barrier(more);
  };

  // (kp is a multiple of 128: at least two stages)
#pragma unroll
  for (int i = 0; i < 2; ++i) load_a(i, 0, false);
  load_b(0, 0);
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    convert(i, 0);
    load_a(i, 1, false);
  }
  __builtin_amdgcn_s_waitcnt(0);
  __syncthreads();
  // the main loop runs while the look-ahead stages are full; the last
  // stages take the guarded steps
  const int nfull = (int)(k / FBK);
  int s = 0;
  for (; s + 3 < nfull; s += 2) {
    step(s, 0, true);
    step(s + 1, 1, true);
  }
  for (; s < nstage; s += 2) {
    step(s, 0, false);
    if (s + 1 < nstage) step(s + 1, 1, false);
  }

  // epilogue: centred residues (+m/2 of m = 256 stores as -128), int8, into
  // the compact [15][m][n] layout of the materialised path
  const int64_t col = wc * 32 + fr;
#pragma unroll
  for (int g = 0; g < G; ++g) {
    int8_t* out = cres + (int64_t)(grp * G + g) * m * n;
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      const int64_t row = row0 + wr * 32 + 8 * (v >> 2) + 4 * fh + (v & 3);
      if (row < m && col < n) out[row * n + col] = (int8_t)cmod_sum(acc[g][v], kModD[grp * G + g], kInvF[grp * G + g]);
    }
  }
}

template <int G, int MODE, bool TZ>
hipError_t launch_fused_g(int64_t m, int64_t n, int64_t k, int64_t kp, const double* A, int64_t lda,
                          const int32_t* sigma, const int8_t* pb, int8_t* cres, hipStream_t stream) {
  const int64_t strips = (m + FBM - 1) / FBM;
  const int64_t blocks = (strips + 7) / 8 * 8 * (kRA / G);
  if (blocks > (int64_t)UINT32_MAX) return hipErrorInvalidValue;
  if (lda < kBufLda)
    hipLaunchKernelGGL((fused_bytes_kernel<G, MODE, TZ, true>), dim3((unsigned)blocks), dim3(1024), 0,
                       stream, m, n, k, kp, A, lda, sigma, pb, cres, strips);
  else
    hipLaunchKernelGGL((fused_bytes_kernel<G, MODE, TZ, false>), dim3((unsigned)blocks), dim3(1024), 0,
                       stream, m, n, k, kp, A, lda, sigma, pb, cres, strips);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_fused_bytes(int quant, int64_t m, int64_t n, int64_t k, int64_t kp, int t,
                              const double* A, int64_t lda, const int32_t* sigma, const int8_t* pb,
                              int8_t* cres, hipStream_t stream) {
  if (n > FBN || kp % 128 || kp <= 0 || m <= 0 || n <= 0 || t > kMaxScaleBits) return hipErrorInvalidValue;
  const bool tz = quant == kQuantTZ;
  // |y| <= 2^t: the nearest quotient up to 2^52, then the group reduction
  const int mode = t <= 51 ? 1 : (t == 52 ? 2 : 3);
  const bool three = fused_moduli(m) == 3;
#define OZ_FUSED_G(G, MODE)                                                                \
  return tz ? launch_fused_g<G, MODE, true>(m, n, k, kp, A, lda, sigma, pb, cres, stream) \
            : launch_fused_g<G, MODE, false>(m, n, k, kp, A, lda, sigma, pb, cres, stream)
#define OZ_FUSED(MODE)           \
  if (three) OZ_FUSED_G(3, MODE); \
  OZ_FUSED_G(5, MODE)
  if (mode == 1) {
    OZ_FUSED(1);
  }
  if (mode == 2) {
    OZ_FUSED(2);
  }
  OZ_FUSED(3);
#undef OZ_FUSED
#undef OZ_FUSED_G
}

}  // namespace oz
