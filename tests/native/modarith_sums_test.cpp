// Host-side check of the lazy reductions (their bounds, and their residues
// against 128-bit integer division) on random and extreme operands.
#include <stdio.h>
#include <math.h>

#include "../../paper_2605_17222_amd/csrc/modarith.hpp"

typedef unsigned __int128 u128;
using namespace ckks;

static uint64_t s = 0x9e3779b97f4a7c15ull;
static uint64_t rnd() {
  s ^= s << 13; s ^= s >> 7; s ^= s << 17;
  return s;
}

int main() {
  // odd moduli at both ends of every size class (primality does not matter here)
  const uint64_t qs[] = {(1ull << 61) - 1, (1ull << 60) + 1, (1ull << 60) - 93, (1ull << 58) + 3, (1ull << 58) - 27,
                         (1ull << 54) - 33, (1ull << 46) + 15, (1ull << 47) - 115};
  long fails = 0, checks = 0;
  for (uint64_t q : qs) {
    const u128 r = (~(u128)0) / q;
    const uint32_t inv64 = (uint32_t)(uint64_t)(r >> 64);
    const int sh = 63 - __builtin_clzll(q);
    const uint64_t mu = (uint64_t)(((u128)1 << (64 + sh)) / q);
    for (int it = 0; it < 200000; ++it) {
      uint64_t a = rnd(), b = rnd(), w = rnd() % q, x = rnd() % (4 * q);
      if (it < 8) { a = it & 1 ? ~0ull : 0; b = it & 2 ? ~0ull : 0; w = it & 4 ? q - 1 : 0; }
      // mulhi64_under: the floor or one less
      const uint64_t hi = (uint64_t)(((u128)a * b) >> 64), un = mulhi64_under(a, b);
      fails += !(un == hi || un + 1 == hi);
      // shoup_add: adds a value below 3q congruent to a w
      const uint64_t wp = (uint64_t)(((u128)w << 64) / q);
      const uint64_t t = shoup_add(x, a, w, wp, q) - x;
      fails += !((u128)t < (u128)3 * q && t % q == (uint64_t)((u128)a * w % q));
      // reduce64: below 2q + 2^32
      const uint64_t y = reduce64(a, q, inv64);
      fails += !((u128)y < (u128)2 * q + ((u128)1 << 32) && y % q == a % q);
      // barrett_sum of up to 4 products of residues
      u128 acc = 0;
      for (int j = 0; j < 4; ++j) acc += (u128)(it < 4 ? q - 1 : rnd() % q) * (it < 4 ? q - 1 : rnd() % q);
      if (it == 5) acc = 0;
      fails += barrett_sum(U128{(uint64_t)acc, (uint64_t)(acc >> 64)}, q, mu, sh) != (uint64_t)(acc % q);
      // mac128
      U128 m = {a, w};
      u128 ref = (((u128)w << 64) | a) + (u128)(b >> 3) * w;
      mac128(m, b >> 3, w);
      fails += !(m.lo == (uint64_t)ref && m.hi == (uint64_t)(ref >> 64));
      checks += 5;
    }
  }
  // fp_mulmod_var for |x| <= 16 q: congruent and at most 7/8 q
  const uint64_t fq[] = {1099511922689ull, 1073692673ull, (1ull << 46) - 21, 35184372088321ull};
  for (uint64_t q : fq) {
    const double qd = (double)q, qi = 1.0 / qd;
    for (int it = 0; it < 300000; ++it) {
      const int64_t lim = 16 * (int64_t)q;
      int64_t x = (int64_t)(rnd() % (2 * (uint64_t)lim + 1)) - lim;
      uint64_t y = rnd() % q;
      if (it < 4) { x = it & 1 ? lim : -lim; y = it & 2 ? q - 1 : q / 2; }
      const double v = fp_mulmod_var((double)x, (double)y, qd, qi);
      __int128 ref = (__int128)x * y % (__int128)q, got = (__int128)(int64_t)v - ref;
      fails += !(fabs(v) <= 0.875 * qd && v == (double)(int64_t)v && got % (__int128)q == 0);
      ++checks;
    }
  }
  printf("%ld checks, %ld failures\n", checks, fails);
  return fails ? 1 : 0;
}
