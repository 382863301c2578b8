// The butterflies of the transforms (ntt.hip), in integers and in FP64, and how
// far each lets values grow; for the host too, whose test runs whole networks of
// them.
#pragma once
#include "internal.hpp"
#include "modarith.hpp"

namespace ckks {

// How far an integer-path prime lets values grow within 64 bits:
//   kFree (q < 2^58, 64 q): a forward transform of 16 stages adds at most
//     16 * 3q = 48 q, and starts from [0, q), from [0, 2q + 2^32) or, with q at
//     most kFromSigned, from [0, 2^63 + q] (residues() below); an inverse round of 4
//     stages from [0, 3q) ends below 48 q, its sums reduced once a round;
//   kRounds (q < 2^60, 16 q): forward, all values reduced to [0, 2q + 2^32) at
//     each round of at most 4 stages (+ 12 q); inverse, sums reduced after two
//     stages (12 q) and at the end of a round;
//   kStages (q < 2^61, 8 q): one operand of each butterfly reduced (5 q + 2^32
//     forward, 6 q inverse).
enum Lazy { kFree, kRounds, kStages };
__host__ __device__ __forceinline__ Lazy lazy_of(uint64_t q) {
  return q < (1ull << 58) ? kFree : (q < (1ull << 60) ? kRounds : kStages);
}
constexpr uint64_t kFromSigned = 1ull << 57;
static_assert(kFromSigned <= (1ull << 63) / (1 + 16 * 3), "2^63 + q + 48 q within 64 bits");

__host__ __device__ __forceinline__ double as_d(uint64_t u) { return __builtin_bit_cast(double, u); }
__host__ __device__ __forceinline__ uint64_t as_u(double d) { return __builtin_bit_cast(uint64_t, d); }

// The arithmetic of one direction and path on a thread's NW words (integer
// residues, or double bits on the FP path).
template <bool FP, bool FWD, int NW = 16>
struct Butterflies {
  const PrimeDev& pr;
  const uint64_t q, q3;
  const Lazy lazy;
  const uint32_t inv64;  // integer path: floor(2^64 / q), below 2^18
  const double qd, qi;
  uint64_t cy = 0;  // inverse, integer path: a multiple of q that no value exceeds
  uint64_t v[NW];

  __host__ __device__ __forceinline__ explicit Butterflies(const PrimeDev& r)
      : pr(r), q(r.q), q3(3 * r.q), lazy(lazy_of(r.q)), inv64((uint32_t)r.r_hi), qd(r.qd), qi(r.qinv_d) {}

  // One butterfly between words u and u + d; the twiddle is (w, wp): the value
  // and its Shoup word, or, on the FP path, w as double bits alone (a product
  // that forms its quotient from x w costs as many operations as one that
  // takes w/q, and half the twiddle words).
  __host__ __device__ __forceinline__ void bfly(int u, int d, uint64_t tw_w, uint64_t tw_p) {
    if (FP) {
      const double w = as_d(tw_w);
      const double X = as_d(v[u]), Y = as_d(v[u + d]);
      if (FWD) {
        const double r = fp_mulmod_var(Y, w, qd, qi);
        v[u] = as_u(X + r);
        v[u + d] = as_u(X - r);
      } else {
        v[u] = as_u(X + Y);
        v[u + d] = as_u(fp_mulmod_var(X - Y, w, qd, qi));
      }
    } else if (FWD) {
      const uint64_t X = v[u];
      // X + t and X - t + 3q, t = v w - qhat q
      const uint64_t sum = shoup_add(X, v[u + d], tw_w, tw_p, q);
      v[u] = sum;
      v[u + d] = 2 * X + q3 - sum;
    } else {
      const uint64_t X = v[u], Y = v[u + d];
      v[u] = X + Y;
      v[u + d] = shoup_add(0, X - Y + cy, tw_w, tw_p, q);
    }
  }
  // Integer path, stage k of a round, its butterflies d apart.  Before it: the
  // inverse's cy, and the forward's operands that have to be reduced, all at once:
  // a test of the class in each butterfly kept the compiler from overlapping them
  // (one limb forward, a 60-bit prime at N = 2^14: 15.7 -> 12.8 us a call; 34 limbs at
  // N = 2^15: 22.8 -> 19.9; column pass of 128 plaintexts of 44 54-bit limbs 1.14 ->
  // 0.99 ms).  After it: the inverse's sums that have to be reduced.
  __host__ __device__ __forceinline__ void stage_begin(int k, int d) {
    if (!FP && !FWD) cy = q3 << (lazy == kFree ? k : (lazy == kRounds ? k & 1 : 0));
    if (!FP && FWD && lazy == kStages) {
#pragma unroll
      for (int u = 0; u < NW; ++u)
        if (!(u & d)) v[u] = reduce64(v[u], q, inv64);
    }
  }
  __host__ __device__ __forceinline__ void stage_end(int k, bool last, int d) {
    if (FP || FWD) return;
    if (last || lazy == kStages || (lazy == kRounds && (k & 1))) {
#pragma unroll
      for (int u = 0; u < NW; ++u)
        if (!(u & d)) v[u] = reduce64(v[u], q, inv64);
    }
  }
  // Between rounds of at most 4 stages.
  __host__ __device__ __forceinline__ void recentre() {
    if (FP) {
#pragma unroll
      for (int u = 0; u < NW; ++u) v[u] = as_u(fp_reduce(as_d(v[u]), qd, qi));
    } else if (FWD && lazy == kRounds) {
#pragma unroll
      for (int u = 0; u < NW; ++u) v[u] = reduce64(v[u], q, inv64);
    }
  }
  // Canonical residues arrive as integers; the FP path converts them.
  __host__ __device__ __forceinline__ void convert_in() {
    if (FP) {
#pragma unroll
      for (int u = 0; u < NW; ++u) v[u] = as_u(u64_to_d(v[u]));
    }
  }
  // Signed coefficients |m| <= 2^62 -> representatives the first round can start
  // from.  m + K q (K q: the least multiple of q above 2^62) is in
  // [0, 2^63 + q]: up to kFromSigned a whole transform's growth (48 q) still fits on
  // top of that (q just below 2^58 would pass 2^64 by a quarter); larger primes
  // reduce it to [0, 2q + 2^32) (exact as a double on the FP path, which does too),
  // those too small for reduce64 by a quotient in FP64: |m / q| there is within one
  // of the floor, so r lands in [-q, 2q).  (Every prime that way took half as many
  // operations as its 8 butterfly stages: column pass of 128 plaintexts of 44 54-bit
  // limbs 1.33 -> 1.14 ms.)
  __host__ __device__ __forceinline__ void residues() {
    if (q < (1ull << 33)) {
      const int64_t qs = (int64_t)q;
#pragma unroll
      for (int u = 0; u < NW; ++u) {
        const int64_t m = (int64_t)v[u];
        int64_t r = m - (int64_t)floor((double)m * qi) * qs;
        r = r < 0 ? r + qs : r;
        v[u] = (uint64_t)(r >= qs ? r - qs : r);
      }
    } else {
#pragma unroll
      for (int u = 0; u < NW; ++u) v[u] += pr.above62;
      if (FP || q > kFromSigned) {
#pragma unroll
        for (int u = 0; u < NW; ++u) v[u] = reduce64(v[u], q, inv64);
      }
    }
  }
  // Final values -> canonical residues: forward, and inverse with the factor
  // N^-1.
  __host__ __device__ __forceinline__ uint64_t canon(uint64_t x) const {
    if (FWD) return FP ? fp_canon(as_d(x), qd, qi) : csub(csub(reduce64(x, q, inv64), q), q);
    return FP ? fp_canon(fp_mulmod(as_d(x), pr.ninv_d, pr.ninv_q, qd), qd, qi) : shoup(x, pr.ninv, pr.ninv_sh, q);
  }
};

}  // namespace ckks
