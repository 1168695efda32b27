// Host check of crt_bytes (crt_bytes.hpp), compiled with g++ by
// tests/test_host_crt.py: wherever it claims a result, that is round_exact_a's
// bit for bit.  Cases: random X of every magnitude; values at and next to
// powers of two, FP64 midpoints and the limbs' boundaries; the ends of
// [-M/2, M/2); normal, subnormal and overflow scales.  Also checked: random
// values are claimed almost always, with a subnormal result too, those of few significant bits always, and zero gives +0.  Exit status 0 on success.
#include <cstdio>
#include <cstring>

#include "fp64_round.hpp"
#include "crt_bytes.hpp"

using namespace oz;
typedef __int128 i128;

static uint64_t st = 0x9E3779B97F4A7C15ull;
static uint64_t rnd() {
  st ^= st << 13;
  st ^= st >> 7;
  st ^= st << 17;
  return st;
}
static i128 M;
static long claimed = 0, declined = 0, bad = 0;

static bool check(i128 X, int e) {
  if (X < -M / 2 || X >= M / 2) return false;
  int c[kRA], v[kRA];
  i128 x = X;
  for (int j = 0; j < kRA; ++j) {
    const int m = kModulusA[j];
    int r = (int)(X % m);
    if (r < 0) r += m;
    // either end of the even modulus's range, as the products deliver it
    c[j] = 2 * r > m || (2 * r == m && (rnd() & 1)) ? r - m : r;
    int d = (int)(x % m);
    if (d < 0) d += m;
    if (2 * d >= m) d -= m;
    v[j] = d;
    x = (x - d) / m;
  }
  double f;
  if (!crt_bytes(c, e, f)) {
    ++declined;
    return false;
  }
  ++claimed;
  const double w = round_exact_a(half_value_a<0, kSplitA>(v), half_value_a<kSplitA, kRA>(v), e);
  if (memcmp(&f, &w, 8)) {
    if (bad++ < 5) printf("X %016llx%016llx e %d: %a, exact %a\n", (unsigned long long)(X >> 64), (unsigned long long)X, e, f, w);
  }
  return true;
}

int main() {
  M = 1;
  for (int j = 0; j < kRA; ++j) M *= kModulusA[j];
  const int scales[] = {0, -100, -1030, -1074, -1100, -1150, 900, 960, 1023, -60};
  long random_claimed = 0, random_all = 0, sub_claimed = 0, sub_all = 0;
  for (int it = 0; it < 3000000; ++it) {
    i128 X = ((i128)rnd() << 64) | (i128)rnd();
    X >>= 10 + (int)(rnd() % 117);
    ++random_all;
    random_claimed += X >= -M / 2 && X < M / 2 ? check(X, -100) : 1;
    check(X, scales[it % 10]);
    // a subnormal result, down to its last bits and zero
    const i128 Y = X < 0 ? -X : X;
    int top = 127;
    while (top > 0 && !(Y >> top)) --top;
    if (Y && Y < M / 2) {
      ++sub_all;
      sub_claimed += check(X, -1023 - top - (int)(rnd() % 56));
    }
  }
  for (int b = 0; b <= 117; ++b)
    for (int l = -1; l <= b; ++l)
      for (int d = -2; d <= 2; ++d)
        for (int s = 0; s < 10; ++s) {
          const i128 X = ((i128)1 << b) + (l < 0 ? 0 : (i128)1 << l) + d;
          check(X, scales[s]);
          check(-X, scales[s]);
        }
  // midpoints: 53 random bits, a half, and a step either side
  for (int it = 0; it < 1000000; ++it) {
    const int sh = 1 + (int)(rnd() % 64);
    i128 X = ((i128)((rnd() >> 11) | (1ull << 52)) << sh) + ((i128)1 << (sh - 1)) + (int)(rnd() % 3) - 1;
    check(rnd() & 1 ? X : -X, scales[it % 10]);
  }
  for (int it = 0; it < 200000; ++it) {
    const i128 d = (i128)(rnd() >> (rnd() % 64));
    check(M / 2 - 1 - d, -100);
    check(-M / 2 + d, -100);
    check((M / 2 - 1 - d) - ((i128)rnd() << (rnd() % 50)), -100);
  }
  // next to and on the ties of shallow subnormals
  for (int it = 0; it < 1000000; ++it) {
    const int sh = 60 + (int)(rnd() % 4), drop = 1 + (int)(rnd() % 8);
    i128 X = (((i128)((rnd() >> 11) | (1ull << 52)) >> drop) << (sh + drop)) + ((i128)1 << (sh + drop - 1)) + (int)(rnd() % 5) - 2;
    if (it & 8) X -= (i128)(rnd() >> 40);
    check(rnd() & 1 ? X : -X, -1074 - sh - drop);
  }
  // few significant bits (products of integers, of FP32 values, of powers of
  // two): every one is claimed, ties and powers of two among them
  long few_claimed = 0, few_all = 0;
  for (int it = 0; it < 1000000; ++it) {
    const int bits = 1 + (int)(rnd() % 57), sh = (int)(rnd() % (117 - bits));
    i128 X = (i128)(rnd() >> (64 - bits) | 1ull << (bits - 1));
    if (it % 4 == 0) X = (i128)1 << (bits - 1);
    X <<= sh;
    if (X >= M / 2) continue;
    few_all += 2;
    few_claimed += check(X, -100) + check(-X, -100);
  }
  int z[kRA] = {};
  double f = 1.0;
  const bool zero = crt_bytes(z, 5, f) && f == 0.0 && !__builtin_signbit(f);
  printf("claimed %ld declined %ld mismatches %ld; random claimed %ld of %ld; few bits %ld of %ld; subnormal %ld of %ld; zero %d\n",
         claimed, declined, bad, random_claimed, random_all, few_claimed, few_all, sub_claimed, sub_all, (int)zero);
  return bad || !zero || random_claimed < random_all * 0.999 || few_claimed < few_all ||
         sub_claimed < sub_all * 0.999;
}
