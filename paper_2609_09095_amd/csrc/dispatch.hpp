// The rules by which ozaki25_dgemm* choose between their launches, from sizes
// alone.  Plain C++, so that they also compile for the host's tests.
#pragma once

#include <cstdint>

namespace oz {

// Storage mode F for A (at most 128 columns, at least kFusedMinRows rows):
// A is converted inside the product kernel, so the workspace holds no planes
// of A and the products need no split of k.
constexpr int64_t kFusedMinRows = 1024;
constexpr bool fused_a(int64_t m, int64_t n) { return n <= 128 && m >= kFusedMinRows; }

// Moduli per block of the tall/skinny product (three or five).  A block has
// 128 rows, strips are dealt to the 8 XCDs in turn, and a CU holds one block,
// so an XCD with `per` strips runs its 15 / G blocks each in rounds of 32.  A
// round of five moduli takes 4/3 of one of three (conversion is paid once per
// group): five wherever that gives fewer or cheaper rounds, three where it
// would only leave CUs idle.  All-byte calls with n = 128, k = 2000, five /
// three: 1100 rows (1 round / 1) 105 / 83 us, 4096 (1 / 1) 112 / 94, 6528 (1 /
// 2) 120 / 160, 10880 (2 / 2) 219 / 171, 13056 (2 / 3) 223 / 241, 22000 (3 / 4)
// 348 / 348, 44000 (5 / 7) 618 / 648; 1024 x 128 x 131072 4.67 / 3.55 ms.
constexpr int64_t kFusedRows = 128;
constexpr int fused_moduli(int64_t m) {
  const int64_t per = ((m + kFusedRows - 1) / kFusedRows + 7) / 8;
  const int64_t r5 = (3 * per + 31) / 32, r3 = (5 * per + 31) / 32;
  return 4 * r5 > 3 * r3 ? 3 : 5;
}

// The one-launch product's limits: rows and columns (32-bit indices), k
// (exact int32 sums; the rule below never asks for more), and leading
// dimensions (32-bit offsets within a 64-row chunk).
constexpr int64_t kOneKernelMaxVecs = (int64_t)1 << 24, kOneKernelMaxK = 4096, kOneKernelMaxLd = (int64_t)1 << 21;

// Whether a product runs as one launch (launch_one_kernel) rather than the
// staged kernels: by the measured times of both on the whole card (256 CUs),
// in tenths of a us.  One launch takes about 5 us and 2.25 per 64-k chunk for
// every round of 256 32 x 32 tiles (a block per CU); the staged path about 20,
// 12.5 per 2^20 outputs and 0.75 per chunk, or in storage mode F 22, 2.3 per
// 2^10 rows and 0.75 per chunk.  Both sides: 64^3 7.1 / 20.1, 512^3 24.3 / 29.7,
// 512 x 512 x 768 31.7 / 34.8, 1024 x 1024 x 64 26.3 / 35.7, 16384 x 32 x 128
// 18.0 / 62; beyond the line 256 x 256 x 1024 35.1 / 31.9, 2048 x 2048 x 64
// 98.6 / 71.9.
constexpr bool one_kernel(int64_t m, int64_t n, int64_t k, int64_t lda, int64_t ldb) {
  if (m > kOneKernelMaxVecs || n > kOneKernelMaxVecs || k > kOneKernelMaxK || lda > kOneKernelMaxLd ||
      ldb > kOneKernelMaxLd)
    return false;
  const int64_t tiles = ((m + 31) / 32) * ((n + 31) / 32), chunks = (k + 63) / 64;
  const int64_t rounds = (tiles + 255) / 256;
  const int64_t staged = fused_a(m, n) ? 220 + 23 * m / 1024 : 200 + 125 * m * n / (1 << 20);
  return 2 * rounds * (50 + 22 * chunks) + rounds * chunks <= 2 * staged + 15 * chunks;
}

// The joint exponent scan: rows of B per slab (each slab leaves one partial
// maximum per column), slabs, and blocks -- one per row of A, or per four rows
// of at most kShortRow elements, and one per slab and strip of 64 columns.
constexpr int64_t kShortRow = 1024;
constexpr int64_t scan_both_rows(int64_t n, int64_t k) {
  return (n + 63) / 64 * ((k + 63) / 64) <= 1024 ? 64 : 256;
}
constexpr int64_t scan_both_slabs(int64_t n, int64_t k) {
  const int64_t rows = scan_both_rows(n, k);
  return (k + rows - 1) / rows;
}
constexpr int64_t scan_both_blocks(int64_t m, int64_t n, int64_t k) {
  return (k <= kShortRow ? (m + 3) / 4 : m) + (n + 63) / 64 * scan_both_slabs(n, k);
}

// Whether both operands' scans share one launch and both deconstructions
// another (k padded to kp):
//  - the partial column maxima need room (bytes);
//  - at most kJointSlabs of them per column: every block of B's deconstruction
//    reads the maxima of its columns, so that work grows with slabs times
//    blocks, that is with k^2.  Calls with joint and with separate launches:
//    512 x 128 x 32768 (512 slabs) 179 / 199 us, 64 x 64 x 262000 (1024) 388 /
//    415, 16 x 16 x 524288 (2048) 439 / 459, 1 x 1 x 2^20 (4096) 769 / 712, 1 x
//    1 x 2^22 (16384) 4.52 / 2.71 ms; in storage mode F 1024 x 64 x 262144 (1024)
//    9.64 / 9.63, 1024 x 128 x 524288 (2048) 19.28 / 19.21;
//  - the launch's work-items must stay below 2^32 (16777215 rows of more than
//    1024 elements are within it alone, but not with B's slabs beside them);
//  - together the operands must fit the last-level cache's 256 MiB, beyond
//    which interleaved runs of one operand at a time are faster (with A
//    converted inside the product kernel, only scanned here, there is no such
//    limit).
constexpr int64_t kJointSlabs = 2048, kJointBlocks = ((int64_t)1 << 24) - 1;  // blocks of 256 work-items
constexpr bool both_at_once(int64_t m, int64_t n, int64_t k, int64_t kp, int64_t room) {
  const int64_t slabs = scan_both_slabs(n, k);
  return slabs <= kJointSlabs && scan_both_blocks(m, n, k) <= kJointBlocks &&
         slabs * n * (int64_t)sizeof(uint32_t) <= room &&
         (fused_a(m, n) || (m + n) * kp * (int64_t)sizeof(double) <= (int64_t)256 << 20);
}

// Whether the int8 product's blocks are placed in one contiguous range of the
// block order per XCD (a modulus's tiles then share an L2) rather than dealt
// over the XCDs in turn.  Only few tiles per modulus have that to gain, and
// not where a multiple of four splits, dealt in turn, already gives every XCD
// its own part of k, where a block has few stages of 128 k, or where the stages
// are so many that the planes pass through the L2 anyway.  Calls on stored
// planes, in turn / in ranges (tiles, splits):
//  - 1024^3 (16, 1) 30.3 / 29.6 us, 1283 x 1025 x 640 (30, 1) 41.9 / 40.0, 1500 x
//    1500 x 4096 (36, 1) 179 / 171, 1024 x 1024 x 40000 (16, 1) 600 / 554, 1283 x
//    1025 x 12000 (30, 1) 331 / 301, 760 x 760 x 8192 (9, 3) 108 / 95, 1100 x 1100 x
//    3000 (25, 2) 103 / 99, 500 x 1000 x 54000 (8, 2) 428 / 415, 760 x 500 x 30000
//    (6, 5) 220 / 213;
//  - 1024 x 1024 x 384 (16, 1) 22.5 / 25.7, 500 x 500 x 1024 (4, 2) 23.4 / 25.8, 2048
//    x 2048 x 16384 (64, 1) 912 / 930, 500 x 500 x 2000 (4, 4) 27.7 / 30.1, 783 x 708
//    x 40000 (12, 4) 432 / 467, 700 x 300 x 40000 (6, 5) 226 / 248, 1391 x 983 x
//    16384 (24, 2) 390 / 401.
constexpr bool xcd_ranges(int64_t tiles, int64_t stages, int64_t splits) {
  if (tiles * splits > 128 || splits % 4 == 0 || stages / splits < (splits > 1 || tiles <= 20 ? 8 : 3)) return false;
  if (splits == 1) return tiles <= 32 || stages <= 64;
  return tiles <= 10 ? splits < 4 || stages <= 240 : stages <= 64;
}

// Whether the reconstruction from stored byte planes (no native re-issue)
// takes strips of 256 columns, a thread per output and row, rather than runs
// of 1024 consecutive outputs: where runs are too few to fill the chip (below 64
// columns from the third or fourth output that a run's thread would take, one
// after another), and for whole strips (every store then starts on a line) of
// up to 2^21 outputs.
// Strips / runs: 64 x 1024 4.2 / 5.2 us, 256 x 1024 4.6 / 6.1, 128 x 4096 6.4 /
// 7.0, 11 x 93106 8.9 / 10.2, 2048 x 1024 13.9 / 15.1, level at 4096 x 1024;
// whole calls at k = 1 128 x 40 11.4 / 12.3, 1021 x 32 12.1 / 12.9, 28 x 32 11.1 / 11.5; the
// other way 4080 x 257 16.6 / 9.7, 16384 x 64 12.2 / 9.1, 1023 x 1025 11.3 /
// 10.3, 262144 x 8 131 / 20.
constexpr bool reconstruct_strips(int64_t m, int64_t n) {
  const int64_t mn = m * n;
  if (n < 64) return n >= 24 && mn > (n >= 40 ? 512 : 768) && mn <= 1 << 15;
  return mn <= 1 << 18 || (mn <= 1 << 20 && n >= 4096) || (mn <= 1 << 21 && n % 256 == 0);
}

}  // namespace oz
