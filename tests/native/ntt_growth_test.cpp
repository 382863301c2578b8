// Host check of how far the transforms' lazy integers grow: whole networks of the
// kernels' own butterflies (csrc/butterflies.hpp), over primes at both ends of
// every class, against the same networks in exact arithmetic.  The inputs make
// the growth largest: every output's sum starts at coefficient 0, so that one is
// at the ends of the signed range or at q - 1.
#include <stdio.h>
#include <math.h>

#include <vector>

#include "../../paper_2605_17222_amd/csrc/butterflies.hpp"

typedef unsigned __int128 u128;
using namespace ckks;

static uint64_t s = 0x9e3779b97f4a7c15ull;
static uint64_t rnd() {
  s ^= s << 13; s ^= s >> 7; s ^= s << 17;
  return s;
}
static uint64_t mm(uint64_t a, uint64_t b, uint64_t q) { return (uint64_t)((u128)a * b % q); }
static uint64_t pw(uint64_t a, uint64_t e, uint64_t q) {
  uint64_t r = 1;
  for (; e; e >>= 1, a = mm(a, a, q))
    if (e & 1) r = mm(r, a, q);
  return r;
}
static bool prime(uint64_t n) {
  for (uint64_t p : {2, 3, 5, 7, 11, 13, 17, 19, 23, 29, 31, 37}) {
    if (n % p == 0) return n == p;
    uint64_t d = n - 1;
    int r = 0;
    while (!(d & 1)) d >>= 1, ++r;
    uint64_t x = pw(p, d, n);
    bool ok = x == 1 || x == n - 1;
    for (int i = 1; i < r && !ok; ++i) ok = (x = mm(x, x, n)) == n - 1;
    if (!ok) return false;
  }
  return true;
}
// the last prime 1 mod two_n below x, or the first one above it
static uint64_t ntt_prime(uint64_t x, uint64_t two_n, bool below) {
  uint64_t c = x / two_n * two_n + 1;
  if (below ? c >= x : c <= x) c = below ? c - two_n : c + two_n;
  while (!prime(c)) c = below ? c - two_n : c + two_n;
  return c;
}
static uint32_t brev(uint32_t x, int bits) {
  uint32_t r = 0;
  for (int i = 0; i < bits; ++i) r |= (x >> i & 1) << (bits - 1 - i);
  return r;
}

struct Ring {
  int log_n;
  PrimeDev pr;
  std::vector<uint64_t> w, wp, iw, iwp;
  Ring(uint64_t q, int ln) : log_n(ln), pr() {
    const uint64_t n = 1ull << ln;
    pr.q = q;
    pr.r_hi = (uint64_t)((~(u128)0 / q) >> 64);
    pr.above62 = ((1ull << 62) / q + 1) * q;
    pr.ninv = pw(n, q - 2, q);
    pr.ninv_sh = (uint64_t)(((u128)pr.ninv << 64) / q);
    uint64_t g = 2;
    while (pw(g, (q - 1) / 2, q) != q - 1) ++g;
    const uint64_t psi = pw(g, (q - 1) / (2 * n), q), inv = pw(psi, q - 2, q);
    w.resize(n), wp.resize(n), iw.resize(n), iwp.resize(n);
    uint64_t a = 1, b = 1;
    for (uint32_t k = 0; k < n; ++k, a = mm(a, psi, q), b = mm(b, inv, q)) {
      const uint32_t r = brev(k, ln);
      w[r] = a, iw[r] = b;
    }
    for (uint32_t k = 0; k < n; ++k)
      wp[k] = (uint64_t)(((u128)w[k] << 64) / q), iwp[k] = (uint64_t)(((u128)iw[k] << 64) / q);
  }
};

// Words wrong after a transform whose rounds are `round` stages.
template <bool FWD>
static long wrong(const Ring& R, const std::vector<int64_t>& in, bool is_signed, int round) {
  const uint64_t q = R.pr.q;
  const int n = 1 << R.log_n;
  Butterflies<false, FWD, 2> F(R.pr);
  std::vector<uint64_t> v(n), e(n);
  for (int i = 0; i < n; i += 2) {
    F.v[0] = (uint64_t)in[i], F.v[1] = (uint64_t)in[i + 1];
    if (is_signed) F.residues();
    v[i] = F.v[0], v[i + 1] = F.v[1];
  }
  for (int i = 0; i < n; ++i) {
    const __int128 m = is_signed ? (__int128)in[i] % (__int128)q : (__int128)(uint64_t)in[i];
    e[i] = (uint64_t)(m < 0 ? m + q : m);
  }
  for (int k = 0; k < R.log_n; ++k) {
    const int st = FWD ? k : R.log_n - 1 - k, d = n >> (st + 1);
    const bool last = k + 1 == R.log_n || (k + 1) % round == 0;
    for (int y = 0; y < 1 << st; ++y)
      for (int x = 2 * d * y; x < 2 * d * y + d; ++x) {
        const uint64_t tw = FWD ? R.w[(1 << st) + y] : R.iw[(1 << st) + y];
        F.v[0] = v[x], F.v[1] = v[x + d];
        F.stage_begin(k % round, 1);
        F.bfly(0, 1, tw, FWD ? R.wp[(1 << st) + y] : R.iwp[(1 << st) + y]);
        F.stage_end(k % round, last, 1);
        if (last && k + 1 < R.log_n) F.recentre();
        v[x] = F.v[0], v[x + d] = F.v[1];
        const uint64_t X = e[x], Y = e[x + d], t = mm(FWD ? Y : X + q - Y, tw, q);
        e[x] = FWD ? (X + t) % q : (X + Y) % q;
        e[x + d] = FWD ? (X + q - t) % q : t;
      }
  }
  long bad = 0;
  for (int i = 0; i < n; ++i) bad += F.canon(v[i]) != (FWD ? e[i] : mm(e[i], R.pr.ninv, q));
  return bad;
}

int main() {
  long fails = 0, checks = 0;
  const int64_t top = 1ll << 62;
  for (int ln : {12, 14, 16}) {
    const uint64_t two_n = 2ull << ln;
    std::vector<uint64_t> qs;
    for (int bits : {61, 60, 58, 57, 54, 47}) qs.push_back(ntt_prime(1ull << bits, two_n, true));
    for (int bits : {60, 58, 57, 46}) qs.push_back(ntt_prime(1ull << bits, two_n, false));
    qs.push_back(ntt_prime((1ull << 63) / 49, two_n, false));  // past the bound of an unreduced start at 16 stages
    for (uint64_t q : qs) {
      const Ring R(q, ln);
      const int n = 1 << ln;
      std::vector<int64_t> x(n);
      for (int kind = 0; kind < 9; ++kind) {
        for (int i = 0; i < n; ++i) {
          const int64_t r = (int64_t)(rnd() >> 1) - top;  // uniform over [-2^62, 2^62)
          x[i] = kind == 0 ? 0 : kind == 1 ? (int64_t)(rnd() >> 23) - (1ll << 40) : kind == 2 ? top : kind == 3 ? -top
               : kind == 4 ? (i & 1 ? -top : top) : kind == 5 ? (i < 64 ? top : r) : kind == 6 ? (r < 0 ? -top : top) : r;
        }
        x[0] = kind == 3 ? -top : kind == 7 ? top - 1 : kind == 8 ? top / 10 * 9 : top;
        const long bad = wrong<true>(R, x, true, ln == 12 ? 3 : 4);
        if (bad) printf("N = 2^%d, q = %llu, signed input %d: %ld wrong words\n", ln, (unsigned long long)q, kind, bad);
        fails += bad != 0, ++checks;
      }
      for (int kind = 0; kind < 3; ++kind) {
        for (int i = 0; i < n; ++i) x[i] = (int64_t)(kind == 0 ? q - 1 : kind == 1 ? (i & 1 ? 0 : q - 1) : rnd() % q);
        fails += wrong<true>(R, x, false, ln == 12 ? 3 : 4) != 0;
        fails += wrong<false>(R, x, false, ln == 12 ? 3 : 4) != 0;
        checks += 2;
      }
    }
  }
  printf("%ld checks, %ld failures\n", checks, fails);
  return fails ? 1 : 0;
}
