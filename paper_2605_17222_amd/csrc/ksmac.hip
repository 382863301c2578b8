// Launch of the fused middle layer (ksmac.hpp): argument checks and the choice
// of the instantiation.
#include <algorithm>

#include "ks_common.hpp"

namespace ckks {

template <int NK>
hipError_t launch_ksmac_nk(const ckks_params* P, const KsMacArgs& a, hipStream_t s);

hipError_t launch_ksmac(const ckks_params* P, const KsMacArgs& a, hipStream_t s) {
  // Geometry, checked before anything runs: term and accumulator counts
  // within the tables, groups that cover the rotated terms, each with a key,
  // every operand present (the kernel reads them unconditionally).
  const int nm = a.nu + a.nr;
  if (a.nu < 0 || a.nr < 0 || nm < 1 || nm > kMaxKsTerms || a.nk < 1 || a.nk > kMaxMacK || nm * a.nk > kMaxKsPts ||
      a.K < 1 || a.K > a.kmax || a.beta < 1 || a.beta > kMaxBeta || P->n % kKsMacAlign ||
      a.groups < (a.nr > 0) || a.groups > a.nr || a.groups > kMaxKsKeys)
    return hipErrorInvalidValue;
  for (int g = 0, m = a.nu; g < a.groups; ++g) {
    const int end = (int)(a.meta[m] >> kKsMacEnd);
    if (end <= m || end > nm || (g + 1 == a.groups) != (end == nm)) return hipErrorInvalidValue;
    m = end;
  }
  int nkeys = 0, ndig = 0, nadd = 0, nf = 0;
  for (int g = 0; g < a.groups; ++g) {
    if (!a.key[g]) return hipErrorInvalidValue;
    nkeys += std::find(a.key, a.key + g, a.key[g]) == a.key + g;
  }
  for (int m = 0; m < nm; ++m) {
    if (!a.a[m] || !a.db[m]) return hipErrorInvalidValue;
    if (m >= a.nu) {
      ndig += std::find(a.db + a.nu, a.db + m, a.db[m]) == a.db + m;
      nadd += std::find(a.a + a.nu, a.a + m, a.a[m]) == a.a + m;
    }
    for (int k = 0; k < a.nk; ++k) {
      if (!a.f[m * a.nk + k]) return hipErrorInvalidValue;
      nf += a.meta[m] >> k & 1;
    }
  }
  for (int k = 0; k < a.nk; ++k)
    if (!a.out0[k] || !a.out1[k]) return hipErrorInvalidValue;
  // algorithmic bytes: keys, digit sets, adds and unrotated products, the
  // plaintexts, the accumulators, each word once (packed limbs at their size)
  const double words = (double)a.K * ((double)a.beta * ndig + nadd + 2.0 * a.nu + 2.0 * a.nk * (a.accumulate ? 2 : 1));
  const double bytes = words * P->n * 8 + 2.0 * a.beta * nkeys * limb_bytes(P, a.K, a.key_packed) +
                       nf * limb_bytes(P, a.K, a.f_packed);
  ProfScope prof(CKKS_KERNEL_KSMAC, s, bytes);
  switch (a.nk) {
    case 1: return launch_ksmac_nk<1>(P, a, s);
    case 2: return launch_ksmac_nk<2>(P, a, s);
    case 3: return launch_ksmac_nk<3>(P, a, s);
    case 4: return launch_ksmac_nk<4>(P, a, s);
    case 5: return launch_ksmac_nk<5>(P, a, s);
    case 6: return launch_ksmac_nk<6>(P, a, s);
    case 7: return launch_ksmac_nk<7>(P, a, s);
    case 8: return launch_ksmac_nk<8>(P, a, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace ckks
