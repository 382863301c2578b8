// Host check of mac128's carry chain (the same steps as its instructions on the
// device) on operands that carry at every place: halves of all ones, of one bit
// and of none, accumulators a step from 2^64 and 2^96, factors at the largest
// modulus.
#include <stdio.h>

#include "../../paper_2605_17222_amd/csrc/modarith.hpp"

typedef unsigned __int128 u128;
using namespace ckks;

int main() {
  const uint64_t f[] = {0, 1, 2, 0x7fffffffull, 0x80000000ull, 0xffffffffull, 1ull << 32, 0x1fffffffull << 32,
                        (0x1fffffffull << 32) | 1, (1ull << 60) - 1, (1ull << 61) - 2, (1ull << 61) - 1};
  const uint64_t w[] = {0, 1, 0xfffffffeull, 0xffffffffull, 1ull << 32, 0xffffffff00000000ull, 0xffffffff00000001ull,
                        ~0ull - 1, ~0ull};
  long fails = 0, checks = 0;
  for (uint64_t a : f)
    for (uint64_t b : f)
      for (uint64_t lo : w)
        for (uint64_t hi : w) {
          U128 m = {lo, hi};
          const u128 ref = (((u128)hi << 64) | lo) + (u128)a * b;
          mac128(m, a, b);
          fails += !(m.lo == (uint64_t)ref && m.hi == (uint64_t)(ref >> 64));
          ++checks;
        }
  // sums of 64 products of the largest residues below 2^61: just within 128 bits
  U128 m = {0, 0};
  u128 ref = 0;
  for (int i = 0; i < 64; ++i) {
    const uint64_t a = (1ull << 61) - 2 - (i & 1);
    mac128(m, a, (1ull << 61) - 2);
    ref += (u128)a * ((1ull << 61) - 2);
    fails += !(m.lo == (uint64_t)ref && m.hi == (uint64_t)(ref >> 64));
    ++checks;
  }
  printf("%ld checks, %ld failures\n", checks, fails);
  return fails ? 1 : 0;
}
