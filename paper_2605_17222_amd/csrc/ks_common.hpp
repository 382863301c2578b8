// Shared by the element-wise kernels of the LT (key switch, plaintext
// multiply-accumulate, and the two fused).
#pragma once
#include "internal.hpp"
#include "modarith.hpp"

namespace ckks {

constexpr int kThreads = 256;

// Operands read once per launch (keys, digits, plaintexts, products) are
// loaded with the non-temporal hint: they stream through without displacing
// cached data, which lifts the achieved read bandwidth on gfx950.  Outputs
// that the next kernel streams the same way (the rotation products read by
// the multiply-accumulate, the accumulators, the automorphism's result) are
// stored non-temporally too: measured, that speeds up the reader (the MAC
// by about 8%).  The gather's accumulators, which the ModDown that follows
// reads right away, use ordinary stores.
__device__ __forceinline__ uint64_t ld_nt(const uint64_t* p) { return __builtin_nontemporal_load(glb(p)); }

// Bytes between the polynomials of a key [beta_max][2] (index 2 b + s):
// packed polynomials of pk_bytes each, or [kmax][N] words each.
__device__ __forceinline__ size_t poly_stride(bool packed, uint64_t pk_bytes, int kmax, size_t n) {
  return packed ? pk_bytes : (size_t)kmax * n * 8;
}

// Bytes of the first `count` limbs of a PQ polynomial, packed or not.
inline double limb_bytes(const ckks_params* P, int count, bool packed) {
  double b = 0;
  for (int i = 0; i < count; ++i) b += (packed && P->primes[i] < kNarrowLimit ? 5.0 : 8.0) * P->n;
  return b;
}

}  // namespace ckks
