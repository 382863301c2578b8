// The middle key switch fused with the plaintext multiply-accumulate
// (Algorithm 2 lines 8-14 in one kernel), by number of accumulators; its
// instantiations are spread over the ksmac_*.hip files.
#pragma once
#include "ks_common.hpp"

namespace ckks {

namespace {

constexpr uint32_t kXcds = 8;  // accelerator complex dies of the device, each with its own L2
static_assert(kKsMacAlign == kThreads * kXcds, "ksmac grid: whole workgroups per XCD");

// Thread (limb l, output position p) forms every term's (a_m, b_m) at p --
// read for unrotated terms, for rotated ones the key-switch product and add
// at the source position auto_index(p, gal) (a gather: eq. (8) keeps a
// wavefront's 64 positions in one aligned block) -- and folds it into NK
// pairs of accumulators right away.
//
// Bound by the words it reads: with the folds taken out it runs no faster, and
// its rate (6.4 TB/s through the L1s, 5.0 TB/s of it from HBM; the digits that
// later rotations gather again come from L2 but take the same path) is what a
// plain kernel reading 256 such streams reaches (6.2-6.4 TB/s).  That needs a
// term's loads all in flight at once, a term ahead of their use: so the loops have no branch around a load: the
// host pads absent plaintexts with a present one of the same term (masked to
// zero), gives every term the same operands, and sorts the terms into
// unrotated ones and groups of rotated terms that share a key; the pointers
// of a term come in with a few wide scalar loads.  The loads that run past the
// last term go to one word of the launch's own operands (a cache hit).
// Measured at N = 2^16, level 24 against loads behind per-operand branches
// (a pointer load and its wait each): (4,4,4) 439 -> 397 us, (4,32,4) 3.31 ->
// 2.78 ms, (1,16,4) 580 -> 581, packed 530 -> 486; (4,16,4) at N = 2^14,
// level 13, 318 (with 16 terms a launch) -> 197 us.  A key read once per group,
// whatever the group's size, against once per term: (3,7,3) 650 -> 453 us.

// The launch's arguments where they are, in the kernel-argument segment: read
// through a by-value parameter, kernels with more than 6 accumulators copied all
// of them into per-lane scratch (3.9 KB a lane).
typedef const __attribute__((address_space(4))) KsMacArgs KsMacArgsK;

template <int NK, int MB>
struct KsMacTerm {
  uint64_t d[MB], a, f[NK];
};
template <int MB>
struct KsMacKey {
  uint64_t k0[MB], k1[MB];
};

// Where a workgroup reads: limb l of keys (byte offset ko, ks bytes between
// polynomials), of plaintexts (fo), of PQ polynomials (lo words) and of
// Q-basis ones to be multiplied by P (lqo words; on the special primes, where
// P vanishes, limb 0).
struct KsMacWhere {
  size_t ko, ks, fo, lo, lqo, dn;
};

template <int NK, bool FN>
__device__ __forceinline__ void ksmac_load_f(uint64_t (&f)[NK], KsMacArgsK& a, int m, uint32_t p, size_t n,
                                             const KsMacWhere& w, bool live) {
#pragma unroll
  for (int k = 0; k < NK; ++k)
    f[k] = ld_word<FN>(reinterpret_cast<const uint8_t*>(a.f[m * NK + k]) + (live ? w.fo : 0), live ? p : 0, n);
}

// Term m of the launch, rotated: digits and add at src (ordinary loads: the
// launch's other rotations read them again, from this XCD's L2), plaintexts
// at p (non-temporal).  !live: past the last term.
template <int NK, int MB, bool FN>
__device__ __forceinline__ void ksmac_load(KsMacTerm<NK, MB>& o, KsMacArgsK& a, int m, uint32_t src, uint32_t p,
                                           size_t n, const KsMacWhere& w, bool live) {
  const CKKS_GLOBAL uint64_t* __restrict__ d = glb(a.db[m]) + (live ? w.lo : 0);
#pragma unroll
  for (int b = 0; b < MB; ++b) o.d[b] = d[b * w.dn + (live ? src : 0)];
  o.a = (glb(a.a[m]) + (live ? (a.meta[m] & kKsMacPscaled ? w.lqo : w.lo) : 0))[live ? src : 0];
  ksmac_load_f<NK, FN>(o.f, a, m, p, n, w, live);
}

template <int MB, bool KN>
__device__ __forceinline__ void ksmac_load_key(KsMacKey<MB>& o, KsMacArgsK& a, int g, uint32_t src, size_t n,
                                               const KsMacWhere& w, bool live) {
  const uint8_t* b = reinterpret_cast<const uint8_t*>(a.key[g]) + (live ? w.ko : 0);
#pragma unroll
  for (int i = 0; i < MB; ++i) {
    o.k0[i] = ld_word<KN>(b + (2 * i) * w.ks, live ? src : 0, n);
    o.k1[i] = ld_word<KN>(b + (2 * i + 1) * w.ks, live ? src : 0, n);
  }
}

// Absent plaintexts of term m (bits of its meta word) to zero.
template <int NK>
__device__ __forceinline__ void ksmac_mask(uint64_t (&f)[NK], uint32_t meta) {
  if ((meta & ((1u << NK) - 1)) == (1u << NK) - 1) return;
#pragma unroll
  for (int k = 0; k < NK; ++k) f[k] = (meta >> k & 1) ? f[k] : 0;
}

// The fold of one limb.  FP (primes below 2^46): operands as exact doubles,
// every product reduced on its own (fp_mulmod_var), sums of at most 64 terms
// of magnitude below q stay exact.
template <int NK, int MB>
struct KsMacFoldFp {
  const PrimeDev& pr;
  const double qd, qi, pm, pmq;  // pm, pmq: P mod q (below 2^46 on this path) and P/q
  double x[NK], y[NK], k0[MB], k1[MB];
  __device__ __forceinline__ explicit KsMacFoldFp(const PrimeDev& r)
      : pr(r), qd(r.qd), qi(r.qinv_d), pm((double)r.pmod), pmq(pm * qi) {
#pragma unroll
    for (int k = 0; k < NK; ++k) x[k] = y[k] = 0.0;
  }
  __device__ __forceinline__ void key(const KsMacKey<MB>& k) {
#pragma unroll
    for (int b = 0; b < MB; ++b) {
      k0[b] = u64_to_d(k.k0[b]);
      k1[b] = u64_to_d(k.k1[b]);
    }
  }
  __device__ __forceinline__ void products(double av, double bv, const uint64_t (&f)[NK]) {
#pragma unroll
    for (int k = 0; k < NK; ++k) {
      const double fd = u64_to_d(f[k]);
      x[k] += fp_mulmod_var(av, fd, qd, qi);
      y[k] += fp_mulmod_var(bv, fd, qd, qi);
    }
  }
  __device__ __forceinline__ void unrotated(uint64_t a, uint64_t b, const uint64_t (&f)[NK], bool pscaled) {
    double av = u64_to_d(a), bv = u64_to_d(b);
    if (pscaled) {  // (P c0', P c1')
      av = fp_mulmod(av, pm, pmq, qd);
      bv = fp_mulmod(bv, pm, pmq, qd);
    }
    products(av, bv, f);
  }
  __device__ __forceinline__ void rotated(const KsMacTerm<NK, MB>& o, bool pscaled) {
    double u = u64_to_d(o.a), v = 0.0;
    if (pscaled) u = fp_mulmod(u, pm, pmq, qd);
    // not reduced: |u| < 0.6 beta q + q <= 3.4 q, well within the 16 q that
    // fp_mulmod_var takes for its first operand, and below 4 q, so that the
    // products stay within 0.6 q
#pragma unroll
    for (int b = 0; b < MB; ++b) {
      const double d = u64_to_d(o.d[b]);
      u += fp_mulmod_var(d, k0[b], qd, qi);
      v += fp_mulmod_var(d, k1[b], qd, qi);
    }
    products(u, v, o.f);
  }
  __device__ __forceinline__ uint64_t out0(int k) const { return fp_canon(x[k], qd, qi); }
  __device__ __forceinline__ uint64_t out1(int k) const { return fp_canon(y[k], qd, qi); }
};

// Other primes: 64 x 64 -> 128-bit products summed lazily; the key-switch
// sums (at most 4 products) reduced with a 64-bit quotient estimate, the
// accumulators once at the end with floor(2^128 / q).
template <int NK, int MB>
struct KsMacFoldInt {
  const PrimeDev& pr;
  const uint64_t q;
  U128 x[NK], y[NK];
  uint64_t k0[MB], k1[MB];
  __device__ __forceinline__ explicit KsMacFoldInt(const PrimeDev& r) : pr(r), q(r.q) {
#pragma unroll
    for (int k = 0; k < NK; ++k) x[k] = y[k] = U128{0, 0};
  }
  __device__ __forceinline__ void key(const KsMacKey<MB>& k) {
#pragma unroll
    for (int b = 0; b < MB; ++b) {
      k0[b] = k.k0[b];
      k1[b] = k.k1[b];
    }
  }
  __device__ __forceinline__ void products(uint64_t av, uint64_t bv, const uint64_t (&f)[NK]) {
#pragma unroll
    for (int k = 0; k < NK; ++k) {
      mac128(x[k], av, f[k]);
      mac128(y[k], bv, f[k]);
    }
  }
  __device__ __forceinline__ void unrotated(uint64_t a, uint64_t b, const uint64_t (&f)[NK], bool pscaled) {
    if (pscaled) {  // (P c0', P c1'): zero on the special primes
      a = shoup(a, pr.pmod, pr.pmod_sh, q);
      b = shoup(b, pr.pmod, pr.pmod_sh, q);
    }
    products(a, b, f);
  }
  __device__ __forceinline__ void rotated(const KsMacTerm<NK, MB>& o, bool pscaled) {
    uint64_t addv = o.a;
    if (pscaled) addv = shoup(addv, pr.pmod, pr.pmod_sh, q);
    U128 u = {0, 0}, v = {0, 0};
#pragma unroll
    for (int b = 0; b < MB; ++b) {
      mac128(u, o.d[b], k0[b]);
      mac128(v, o.d[b], k1[b]);
    }
    products(add_mod(barrett_sum(u, q, pr.bs_mu, pr.bs_shift), addv, q), barrett_sum(v, q, pr.bs_mu, pr.bs_shift),
             o.f);
  }
  __device__ __forceinline__ uint64_t out0(int k) const { return barrett128(x[k], q, pr.r_lo, pr.r_hi); }
  __device__ __forceinline__ uint64_t out1(int k) const { return barrett128(y[k], q, pr.r_lo, pr.r_hi); }
};

// Layouts: KN / FN, the keys' / plaintexts' limb is packed narrow (32-bit and
// 8-bit planes).  GROUPED: some rotated terms share a key, else each has its own.
template <int NK, int MB, bool GROUPED, bool PK, bool PF, bool NARROW, typename Fold>
__device__ __forceinline__ void ksmac_body(KsMacArgsK& a, const PrimeDev& pr, int l, uint32_t p, size_t n,
                                           int log_n, int alpha) {
  constexpr bool KN = PK && NARROW, FN = PF && NARROW;
  KsMacWhere w;
  w.ko = limb_off(l, n, PK, pr);
  w.ks = poly_stride(PK, a.pk_poly_bytes, a.kmax, n);
  w.fo = limb_off(l, n, PF, pr);
  w.lo = (size_t)l * n;
  w.lqo = (size_t)max(l - alpha, 0) * n;
  w.dn = (size_t)a.K * n;
  Fold F(pr);
  KsMacTerm<NK, MB> t0, t1;
  KsMacKey<MB> key, key1;
  const int groups = a.groups;
  uint32_t src = 0;
  if (groups > 0) {
    src = auto_index(p, a.gal[0], log_n);
    ksmac_load_key<MB, KN>(key, a, 0, src, n, w, true);
    ksmac_load<NK, MB, FN>(t0, a, a.nu, src, p, n, w, true);
  }
  if (a.nu > 0) {
    uint64_t ua, ub, uf[NK];
    auto load_u = [&](uint64_t& x, uint64_t& y, uint64_t (&f)[NK], int m, bool live) {
      const size_t lo = live ? ((a.meta[m] & kKsMacPscaled) ? w.lqo : w.lo) : 0;
      x = ld_nt(a.a[m] + lo + (live ? p : 0));
      y = ld_nt(a.db[m] + lo + (live ? p : 0));
      ksmac_load_f<NK, FN>(f, a, m, p, n, w, live);
    };
    load_u(ua, ub, uf, 0, true);
    for (int m = 0; m < a.nu; ++m) {
      uint64_t va, vb, vf[NK];
      const bool live = m + 1 < a.nu;
      load_u(va, vb, vf, live ? m + 1 : m, live);
      __builtin_amdgcn_sched_barrier(0);
      const uint32_t meta = a.meta[m];
      ksmac_mask<NK>(uf, meta);
      F.unrotated(ua, ub, uf, meta & kKsMacPscaled);
      ua = va;
      ub = vb;
#pragma unroll
      for (int k = 0; k < NK; ++k) uf[k] = vf[k];
    }
  }
  auto fold = [&](KsMacTerm<NK, MB>& t, int m) {
    const uint32_t meta = a.meta[m];
    ksmac_mask<NK>(t.f, meta);
    F.rotated(t, meta & kKsMacPscaled);
  };
  if constexpr (!GROUPED) {
    // two terms, each with its own key, per iteration (operand sets alternate)
    for (int g = 0; g < groups; g += 2) {
      const bool l1 = g + 1 < groups, l2 = g + 2 < groups;
      const int g1 = l1 ? g + 1 : g, g2 = l2 ? g + 2 : g;
      src = auto_index(p, a.gal[g1], log_n);
      ksmac_load_key<MB, KN>(key1, a, g1, src, n, w, l1);
      ksmac_load<NK, MB, FN>(t1, a, a.nu + g1, src, p, n, w, l1);
      __builtin_amdgcn_sched_barrier(0);
      F.key(key);
      fold(t0, a.nu + g);
      if (!l1) break;
      src = auto_index(p, a.gal[g2], log_n);
      ksmac_load_key<MB, KN>(key, a, g2, src, n, w, l2);
      ksmac_load<NK, MB, FN>(t0, a, a.nu + g2, src, p, n, w, l2);
      __builtin_amdgcn_sched_barrier(0);
      F.key(key1);
      fold(t1, a.nu + g + 1);
    }
  } else {
    // two terms of a key per iteration; the last one or two of a group load the
    // next key
    int m = a.nu;
    for (int g = 0; g < groups; ++g) {
      F.key(key);
      const int end = (int)(a.meta[m] >> kKsMacEnd);
      for (; m + 2 < end; m += 2) {
        ksmac_load<NK, MB, FN>(t1, a, m + 1, src, p, n, w, true);
        __builtin_amdgcn_sched_barrier(0);
        fold(t0, m);
        ksmac_load<NK, MB, FN>(t0, a, m + 2, src, p, n, w, true);
        __builtin_amdgcn_sched_barrier(0);
        fold(t1, m + 1);
      }
      if (m + 1 < end) {
        ksmac_load<NK, MB, FN>(t1, a, m + 1, src, p, n, w, true);
        __builtin_amdgcn_sched_barrier(0);
        fold(t0, m);
        t0 = t1;
        ++m;
      }
      const bool live = g + 1 < groups;
      const int g1 = live ? g + 1 : g;
      src = auto_index(p, a.gal[g1], log_n);
      ksmac_load_key<MB, KN>(key, a, g1, src, n, w, live);
      ksmac_load<NK, MB, FN>(t1, a, live ? end : m, src, p, n, w, live);
      __builtin_amdgcn_sched_barrier(0);
      fold(t0, m);
      t0 = t1;
      m = end;
    }
  }
  const size_t off = w.lo + p;
#pragma unroll
  for (int k = 0; k < NK; ++k) {
    uint64_t xr = F.out0(k), yr = F.out1(k);
    if (a.accumulate) {
      xr = add_mod(xr, glb(a.out0[k])[off], pr.q);
      yr = add_mod(yr, glb(a.out1[k])[off], pr.q);
    }
    __builtin_nontemporal_store(xr, glb(a.out0[k]) + off);
    __builtin_nontemporal_store(yr, glb(a.out1[k]) + off);
  }
}

// Workgroup w of the launch runs on XCD w mod 8 (the dispatcher deals
// workgroups round-robin over the eight XCDs).  All XCDs work on one limb at a
// time, each on its own eighth of the positions: about 80 streams (the
// limb's words in every key and plaintext) are open at once instead of 8
// times as many, which HBM serves faster than whole limbs per XCD did
// ((4,4,4) at N = 2^16, level 24: 413 -> 397 us; (4,32,4) 2.87 -> 2.78 ms),
// and integer-path limbs, which cost more, load every XCD alike.
// The grid is (N / kThreads) x K with N / kThreads a multiple of 8.
// PK / PF: the keys / plaintexts of the launch are packed; a packed narrow
// limb (prime below 2^40, so on the FP64 path) is read from its planes.
template <int NK, int MB, bool GROUPED, bool PK, bool PF>
__global__ void __launch_bounds__(kThreads)
    ksmac_kernel(KsMacArgs, const PrimeDev* __restrict__ primes, int log_n, int alpha) {
  KsMacArgsK& a = *(KsMacArgsK*)__builtin_amdgcn_kernarg_segment_ptr();  // the first argument
  const uint32_t p = ((blockIdx.x % kXcds) * (gridDim.x / kXcds) + blockIdx.x / kXcds) * kThreads + threadIdx.x;
  const int l = (int)blockIdx.y;
  const PrimeDev& pr = primes[l];
  const size_t n = (size_t)1 << log_n;
  using Fp = KsMacFoldFp<NK, MB>;
  using Int = KsMacFoldInt<NK, MB>;
  if (pr.fp) {
    if constexpr (PK || PF) {
      if (pr.narrow) {
        ksmac_body<NK, MB, GROUPED, PK, PF, true, Fp>(a, pr, l, p, n, log_n, alpha);
        return;
      }
    }
    ksmac_body<NK, MB, GROUPED, PK, PF, false, Fp>(a, pr, l, p, n, log_n, alpha);
  } else {
    ksmac_body<NK, MB, GROUPED, PK, PF, false, Int>(a, pr, l, p, n, log_n, alpha);
  }
}

template <int NK, int MB, bool PK, bool PF>
void launch_ksmac_one(const ckks_params* P, const KsMacArgs& a, hipStream_t s) {
  const dim3 grid(P->n / kThreads, a.K), block(kThreads);
  if (a.groups < a.nr)
    hipLaunchKernelGGL((ksmac_kernel<NK, MB, true, PK, PF>), grid, block, 0, s, a, P->d_primes, P->log_n, P->alpha);
  else
    hipLaunchKernelGGL((ksmac_kernel<NK, MB, false, PK, PF>), grid, block, 0, s, a, P->d_primes, P->log_n, P->alpha);
}

template <int NK, int MB>
void launch_ksmac_mb(const ckks_params* P, const KsMacArgs& a, hipStream_t s) {
  if (a.key_packed && a.f_packed)
    launch_ksmac_one<NK, MB, true, true>(P, a, s);
  else if (a.key_packed)
    launch_ksmac_one<NK, MB, true, false>(P, a, s);
  else if (a.f_packed)
    launch_ksmac_one<NK, MB, false, true>(P, a, s);
  else
    launch_ksmac_one<NK, MB, false, false>(P, a, s);
}

}  // namespace

template <int NK>
hipError_t launch_ksmac_nk(const ckks_params* P, const KsMacArgs& a, hipStream_t s) {
  switch (a.beta) {
    case 1: launch_ksmac_mb<NK, 1>(P, a, s); break;
    case 2: launch_ksmac_mb<NK, 2>(P, a, s); break;
    case 3: launch_ksmac_mb<NK, 3>(P, a, s); break;
    case 4: launch_ksmac_mb<NK, 4>(P, a, s); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace ckks
