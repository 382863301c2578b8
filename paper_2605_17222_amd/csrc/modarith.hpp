// 64-bit modular arithmetic on the gfx950 vector ALU.
//
// Residues are uint64 below primes q < 2^61.  There is no 64x64->128 multiply
// instruction: a full product is four 32x32->64 multiply-adds
// (v_mad_u64_u32).  Three reductions are used, each where it is cheapest:
//  * Shoup multiplication by a constant w with w' = floor(w 2^64 / q) (NTT
//    twiddles, scaling constants): result in [0, 2q).
//  * Montgomery REDC of a 128-bit sum x < q 2^64 (basis conversion, whose
//    constants are stored premultiplied by 2^64): x 2^-64 mod q.
//  * Barrett reduction of any 128-bit value with floor(2^128 / q) (key-switch
//    and plaintext inner products, whose operands are both data).
// Lazy (non-canonical) intermediate ranges are documented at each use.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace ckks {

struct U128 {
  uint64_t lo, hi;
};

// Full 64x64 -> 128 product from four 32x32 -> 64 multiply-adds.
__host__ __device__ __forceinline__ U128 mul_wide(uint64_t a, uint64_t b) {
  const uint32_t a0 = (uint32_t)a, a1 = (uint32_t)(a >> 32);
  const uint32_t b0 = (uint32_t)b, b1 = (uint32_t)(b >> 32);
  const uint64_t p00 = (uint64_t)a0 * b0;
  const uint64_t t = (uint64_t)a0 * b1 + (p00 >> 32);          // < 2^64
  const uint64_t u = (uint64_t)a1 * b0 + (uint32_t)t;          // < 2^64
  U128 r;
  r.hi = (uint64_t)a1 * b1 + ((t >> 32) + (u >> 32));
  r.lo = (u << 32) | (uint32_t)p00;
  return r;
}

__host__ __device__ __forceinline__ uint64_t mulhi64(uint64_t a, uint64_t b) { return mul_wide(a, b).hi; }

__host__ __device__ __forceinline__ void add128(U128& acc, U128 v) {
  acc.lo += v.lo;
  acc.hi += v.hi + (acc.lo < v.lo ? 1 : 0);
}

__host__ __device__ __forceinline__ uint64_t csub(uint64_t x, uint64_t q) { return x >= q ? x - q : x; }

__host__ __device__ __forceinline__ uint64_t add_mod(uint64_t a, uint64_t b, uint64_t q) { return csub(a + b, q); }
__host__ __device__ __forceinline__ uint64_t sub_mod(uint64_t a, uint64_t b, uint64_t q) { return a >= b ? a - b : a + q - b; }

// a * w mod q in [0, 2q) for any a < 2^64, w < q, wp = floor(w 2^64 / q).
__host__ __device__ __forceinline__ uint64_t shoup_lazy(uint64_t a, uint64_t w, uint64_t wp, uint64_t q) {
  return a * w - mulhi64(a, wp) * q;
}
__host__ __device__ __forceinline__ uint64_t shoup(uint64_t a, uint64_t w, uint64_t wp, uint64_t q) {
  return csub(shoup_lazy(a, w, wp, q), q);
}

// x 2^-64 mod q for x < q 2^64, qinv_neg = -q^-1 mod 2^64; result canonical.
__host__ __device__ __forceinline__ uint64_t redc(U128 x, uint64_t q, uint64_t qinv_neg) {
  const uint64_t m = x.lo * qinv_neg;
  const uint64_t t = x.hi + mulhi64(m, q) + (x.lo != 0 ? 1 : 0);
  return csub(t, q);
}

// x mod q for any x < 2^128, with (r_hi, r_lo) = floor(2^128 / q).
// qhat = floor(x r / 2^128) satisfies x/q - 2 < qhat <= x/q, so x - qhat q is
// in [0, 2q) and is computed modulo 2^64.
__host__ __device__ __forceinline__ uint64_t barrett128(U128 x, uint64_t q, uint64_t r_lo, uint64_t r_hi) {
  const uint64_t c0 = mulhi64(x.lo, r_lo);
  const U128 p1 = mul_wide(x.lo, r_hi);
  const U128 p2 = mul_wide(x.hi, r_lo);
  uint64_t s = p1.lo + c0;
  uint64_t carry = s < c0 ? 1 : 0;
  s += p2.lo;
  carry += s < p2.lo ? 1 : 0;
  const uint64_t qhat = x.hi * r_hi + p1.hi + p2.hi + carry;
  return csub(x.lo - qhat * q, q);
}

// Carries in inline assembly.  On gfx950 the compiler keeps at least two wait states
// between a vector instruction that writes a mask (a carry, a select) and one that
// reads it, but it does not look into asm statements: between two of them it left
// one, or none.  So a mask is read in the statement that wrote it, with that
// distance kept there, or in a later one behind two wait states of its own.

// acc += a b for a, b < 2^61 (the cross products' sum stays below 2^63):
// four multiply-adds and one carry chain, against fifteen instructions for
// mul_wide and add128 (the waits cost nothing measurable: (4,4,4) at N = 2^16,
// level 24 397 us fused with and without them).
__host__ __device__ __forceinline__ void mac128(U128& acc, uint64_t a, uint64_t b) {
  const uint32_t a0 = (uint32_t)a, a1 = (uint32_t)(a >> 32);
  const uint32_t b0 = (uint32_t)b, b1 = (uint32_t)(b >> 32);
  uint64_t m = (uint64_t)a0 * b1;
  m += (uint64_t)a1 * b0;
  const uint64_t hi = acc.hi + (uint64_t)a1 * b1;
  uint64_t lo = acc.lo;
#ifdef __HIP_DEVICE_COMPILE__
  uint64_t c, d;
  asm("v_mad_u64_u32 %0, %1, %2, %3, %0" : "+v"(lo), "=s"(c) : "v"(a0), "v"(b0));
  uint32_t w1 = (uint32_t)(lo >> 32), w2 = (uint32_t)hi, w3 = (uint32_t)(hi >> 32), mh = (uint32_t)(m >> 32);
  asm("v_add_co_u32_e64 %0, %4, %0, %6\n\t"
      "s_nop 0\n\t"
      "v_addc_co_u32_e64 %3, %5, 0, %3, %5\n\t"
      "v_addc_co_u32_e64 %1, %4, %1, %3, %4\n\t"
      "s_nop 1\n\t"
      "v_addc_co_u32_e64 %2, %4, 0, %2, %4"
      : "+v"(w1), "+v"(w2), "+v"(w3), "+v"(mh), "=&s"(d), "+s"(c)
      : "v"((uint32_t)m));
#else  // the same steps
  const uint32_t c = __builtin_add_overflow(lo, (uint64_t)a0 * b0, &lo) ? 1 : 0;
  const uint32_t mh = (uint32_t)(m >> 32) + c;
  const uint64_t s1 = (lo >> 32) + (uint32_t)m, s2 = (uint64_t)(uint32_t)hi + mh + (s1 >> 32);
  const uint32_t w1 = (uint32_t)s1, w2 = (uint32_t)s2, w3 = (uint32_t)(hi >> 32) + (uint32_t)(s2 >> 32);
#endif
  acc.lo = (uint32_t)lo | ((uint64_t)w1 << 32);
  acc.hi = w2 | ((uint64_t)w3 << 32);
}

// a b / 2^64 rounded down, or one less: the low partial product and its carry
// are left out.
__host__ __device__ __forceinline__ uint64_t mulhi64_under(uint64_t a, uint64_t b) {
  const uint32_t a0 = (uint32_t)a, a1 = (uint32_t)(a >> 32);
  const uint32_t b0 = (uint32_t)b, b1 = (uint32_t)(b >> 32);
  uint64_t m = (uint64_t)a0 * b1;
  uint32_t ch;
#ifdef __HIP_DEVICE_COMPILE__
  uint64_t c;
  asm("v_mad_u64_u32 %0, %1, %3, %4, %0\n\t"
      "s_nop 1\n\t"
      "v_cndmask_b32_e64 %2, 0, 1, %1"
      : "+v"(m), "=&s"(c), "=v"(ch)
      : "v"(a1), "v"(b0));
#else
  ch = __builtin_add_overflow(m, (uint64_t)a1 * b0, &m) ? 1 : 0;
#endif
  return (uint64_t)a1 * b1 + ((m >> 32) | ((uint64_t)ch << 32));
}

// x + a w - qhat q (mod 2^64) with qhat = mulhi64_under(a, wp): adds
// a w mod q to x lazily.  With wp = floor(w 2^64 / q) the Shoup remainder
// a w - floor(a wp / 2^64) q is below q (1 + a / 2^64), so what is added is in
// [0, 3q) for any a < 2^64.
__host__ __device__ __forceinline__ uint64_t shoup_add(uint64_t x, uint64_t a, uint64_t w, uint64_t wp, uint64_t q) {
  const uint64_t h = mulhi64_under(a, wp), nq = 0 - q;
  const uint32_t a0 = (uint32_t)a, a1 = (uint32_t)(a >> 32), w0 = (uint32_t)w, w1 = (uint32_t)(w >> 32);
  const uint32_t h0 = (uint32_t)h, h1 = (uint32_t)(h >> 32), n0 = (uint32_t)nq, n1 = (uint32_t)(nq >> 32);
  uint64_t r = (uint64_t)a0 * w0 + x;
  r += (uint64_t)h0 * n0;
  const uint32_t hi = (uint32_t)(r >> 32) + a0 * w1 + a1 * w0 + h0 * n1 + h1 * n0;
  return (uint32_t)r | ((uint64_t)hi << 32);
}

// x mod q up to multiples of q, in [0, 2q + 2^32), for any x < 2^64 and
// q > 2^32, with inv64 = floor(2^64 / q): the quotient estimate
// floor(floor(x / 2^32) inv64 / 2^32) is at most x / q and falls short of it by
// less than 2 + 2^32 / q.
__host__ __device__ __forceinline__ uint64_t reduce64(uint64_t x, uint64_t q, uint32_t inv64) {
  const uint32_t e = (uint32_t)(((x >> 32) * inv64) >> 32);
  const uint64_t nq = 0 - q;
  const uint64_t r = (uint64_t)e * (uint32_t)nq + x;
  return (uint32_t)r | ((uint64_t)((uint32_t)(r >> 32) + e * (uint32_t)(nq >> 32)) << 32);
}

// x mod q for a sum x of at most 4 products of residues (x < 4 q^2, q < 2^61):
// with s = bits(q) - 1, x / 2^s < 2^64 and mu = floor(2^(64+s) / q) < 2^64, and
// qhat = (x >> s) mu / 2^64 falls short of x / q by less than 1 (the shift)
// + 1 (mu) + 2 (mulhi64_under), so x - qhat q is in [0, 4q).
__host__ __device__ __forceinline__ uint64_t barrett_sum(U128 x, uint64_t q, uint64_t mu, int s) {
  const uint64_t xh = (x.lo >> s) | (x.hi << 1 << (63 - s));
  uint64_t r = x.lo - mulhi64_under(xh, mu) * q;
  r = csub(r, 2 * q);
  return csub(r, q);
}

// ---- exact FP64 arithmetic for primes q < 2^46 ----------------------------
// Residues are doubles holding exact integers.  A product x*w (0 <= w < q) is
// reduced with an FMA two-product, so the remainder is exact:
//   t = rint(x * fl(w/q)),  h + l = t*q exactly,  r = fl(x*w - h) - l.
// |fl(x fl(w/q)) - x w/q| <= |x| 2^-52, so for |x| <= 16 q < 2^50 we get
// |x w/q - t| <= 1/2 + 2^-2 and |r| <= 0.75 q; x*w - h = (x*w - t q) + l with
// |l| <= ulp(h)/2 <= 2^45, so it is an integer below 2^53 and the FMA that
// forms it is exact.

// x < 2^52 as a double: the bits of 2^52 with x as the significand are the
// double 2^52 + x (one OR into the high word), and subtracting 2^52 is exact.
__host__ __device__ __forceinline__ double u64_to_d(uint64_t x) {
  return __builtin_bit_cast(double, x | 0x4330000000000000ull) - 4503599627370496.0;
}

__host__ __device__ __forceinline__ double fp_mulmod(double x, double w, double wq, double q) {
  const double t = rint(x * wq);
  const double h = t * q;
  const double l = fma(t, q, -h);
  return fma(x, w, -h) - l;
}

// x * y mod q without a precomputed quotient, q < 2^46, |x| <= 16 q, |y| <= q:
// h = fl(x y) and l = x y - h (exact, |l| <= ulp(h)/2 <= 2^42) are the
// two-product; |x y / q| < 2^50 and h fl(1/q) is within three roundings of it,
// so t = rint(h fl(1/q)) is within 1/2 + 3/8 of x y / q; h - t q is an integer
// below 2^53 in magnitude, so the FMA that forms it is exact, and so is the
// result h - t q + l, congruent to x y and at most 7/8 q in magnitude (for
// |x| <= 4 q at most 0.6 q).
__host__ __device__ __forceinline__ double fp_mulmod_var(double x, double y, double q, double qinv) {
  const double h = x * y;
  const double l = fma(x, y, -h);
  const double t = rint(h * qinv);
  return fma(-t, q, h) + l;
}

// |x| < 2^52 -> x mod q in [-q/2 - 1, q/2 + 1] (an exact FMA: the result is below q).
__host__ __device__ __forceinline__ double fp_reduce(double x, double q, double qinv) {
  return fma(-rint(x * qinv), q, x);
}

// |x| < 2^52 -> canonical residue in [0, q) as uint64 (the residue r is an
// integer below 2^52, so 2^52 + r is exact and its significand is r).
__host__ __device__ __forceinline__ uint64_t fp_canon(double x, double q, double qinv) {
  double r = fp_reduce(x, q, qinv);
  r = r < 0 ? r + q : r;
  r = r >= q ? r - q : r;
  return __builtin_bit_cast(uint64_t, r + 4503599627370496.0) & ((1ull << 52) - 1);
}

// sum_j y_j c_j for NS <= 16 terms with y_j, c_j < 2^60, from 30-bit halves
// (y_j = y1_j 2^30 + y0_j, c_j = c1_j 2^30 + c0_j): every partial product is below
// 2^60, so each of the four column sums stays below 2^64 and a term costs four
// 32x32+64 multiply-adds with no carry handling; the columns are combined
// once: c00 + (c01 + c10) 2^30 + c11 2^60 < 2^125.
// k[j] = {c0, c1}: the constant already split.
template <int NS>
__host__ __device__ __forceinline__ U128 dot_split30(const uint32_t* y0, const uint32_t* y1, const uint32_t (*k)[2]) {
  uint64_t c00 = 0, c01 = 0, c10 = 0, c11 = 0;
#pragma unroll
  for (int j = 0; j < NS; ++j) {
    const uint32_t k0 = k[j][0], k1 = k[j][1];
    c00 += (uint64_t)y0[j] * k0;
    c01 += (uint64_t)y0[j] * k1;
    c10 += (uint64_t)y1[j] * k0;
    c11 += (uint64_t)y1[j] * k1;
  }
  U128 acc = {c00, 0};
  add128(acc, U128{c01 << 30, c01 >> 34});
  add128(acc, U128{c10 << 30, c10 >> 34});
  add128(acc, U128{c11 << 60, c11 >> 4});
  return acc;
}

// Bit reversal of the low `bits` bits.
__device__ __forceinline__ uint32_t bitrev(uint32_t x, int bits) { return __brev(x) >> (32 - bits); }

// NTT-domain automorphism index.  With g the Galois element, position p of
// phi_g(a) holds a at position br((g (2 br(p) + 1) mod 2N - 1) / 2).
__device__ __forceinline__ uint32_t auto_index(uint32_t p, uint32_t g, int log_n) {
  const uint32_t l = bitrev(p, log_n);
  const uint32_t e = (uint32_t)(((uint64_t)g * (2u * l + 1u)) & ((2u << log_n) - 1u));
  return bitrev((e - 1u) >> 1, log_n);
}

// Packed narrow limbs are runs of kPackChunk coefficients: the run's 32-bit
// low words, then its 8-bit high bytes (5 kPackChunk bytes), so one limb is a
// single contiguous stream.
constexpr size_t kPackChunk = 256;

#ifdef __HIPCC__
// Limb l (prime pr) of a polynomial at `poly`, stored packed (the limb starts
// at byte pr.pk_off; a narrow prime's limb is in runs as above) or as
// [limbs][N] 64-bit words.  Both are uniform over a block whose limb index is
// uniform, so a kernel branches once on `narrow` and then issues straight-line
// loads.
struct LimbRef {
  const uint8_t* b;  // first byte of the limb
  bool narrow;       // 32 + 8-bit planes (else N 64-bit words)
};
template <typename PrimeT>  // the library's per-prime table entry (pk_off, narrow)
__device__ __forceinline__ size_t limb_off(int l, size_t n, bool packed, const PrimeT& pr) {
  return packed ? (size_t)pr.pk_off : (size_t)l * n * 8;
}
template <typename PrimeT>
__device__ __forceinline__ LimbRef limb_ref(const void* poly, int l, size_t n, bool packed, const PrimeT& pr) {
  return {reinterpret_cast<const uint8_t*>(poly) + limb_off(l, n, packed, pr), packed && pr.narrow};
}
// Global memory, said in the pointer's type: a pointer out of a table that the
// compiler cannot trace would otherwise be read by flat loads.
#define CKKS_GLOBAL __attribute__((address_space(1)))
__device__ __forceinline__ const CKKS_GLOBAL uint64_t* glb(const uint64_t* p) { return (const CKKS_GLOBAL uint64_t*)p; }
__device__ __forceinline__ CKKS_GLOBAL uint64_t* glb(uint64_t* p) { return (CKKS_GLOBAL uint64_t*)p; }
// Word p of a limb; non-temporal loads, these operands are read once per launch.
template <bool NARROW>
__device__ __forceinline__ uint64_t ld_word(const uint8_t* b, size_t p, size_t n) {
  if constexpr (NARROW) {
    const CKKS_GLOBAL uint8_t* c = (const CKKS_GLOBAL uint8_t*)b + (p / kPackChunk) * (5 * kPackChunk);
    const size_t r = p % kPackChunk;
    const uint64_t lo = __builtin_nontemporal_load((const CKKS_GLOBAL uint32_t*)c + r);
    const uint64_t hi = __builtin_nontemporal_load(c + 4 * kPackChunk + r);
    return lo | (hi << 32);
  } else {
    return __builtin_nontemporal_load((const CKKS_GLOBAL uint64_t*)b + p);
  }
}
#endif

}  // namespace ckks
