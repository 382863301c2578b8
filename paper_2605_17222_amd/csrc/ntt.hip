// Negacyclic NTT / inverse NTT over batches of limbs (gfx950).
//
// Layout (bit-reversed storage, Section V): word p of an NTT-form limb holds
// the evaluation at psi^(2 br(p) + 1).  The forward transform is the radix-2
// Cooley-Tukey network with twiddle psi^br(m + i) at stage m (log2 m = s),
// butterfly (x, x + N/2m); the inverse is the Gentleman-Sande network with
// psi^-br(m + i) and a final factor N^-1.  The PE butterflies of Section V
// (a0 +- a1 tf; (a0 + a1), (a0 - a1) tf) are exactly these, with the halving
// collected into N^-1.
//
// N <= 2^13: one kernel (ntt_full below).  A larger limb of N = N1 N2 words is
// transformed in two passes of log2 N1 and log2 N2 stages (at N = 2^16 a limb
// is 512 KiB, larger than one workgroup's LDS):
//   column pass: the first log2 N1 stages act on the N2 columns (stride N2)
//                independently;
//   row pass:    the last log2 N2 stages act on the N1 rows (contiguous)
//                independently.
// Inside a pass each thread keeps 16 words in registers: 4 stages run in
// registers, the words are exchanged through LDS, and the remaining stages run
// in registers again.
//
// Two arithmetic paths, chosen per limb (uniform over a workgroup):
//  * integer (q >= 2^46): lazy butterflies with Shoup twiddle products whose
//    quotient may be one short (mulhi64_under), so a product is in [0, 3q);
//    values grow within 64 bits and are reduced as seldom as the prime's size
//    allows (see Lazy in butterflies.hpp): about 16 instructions a butterfly
//    against 29 with an exact quotient and a conditional subtraction (32
//    plaintexts of 44 54-bit limbs at N = 2^16: column pass 401 -> 244 us, row
//    pass 476 -> 371, its twiddles from L2);
//  * FP64 (q < 2^46): residues are doubles holding exact integers, the
//    twiddle product is the exact FMA two-product remainder of modarith.hpp,
//    values are re-centred every 4 stages.  Between the two passes such a limb
//    is stored as raw double bits; the final pass writes canonical residues.
//
// Stage s of a sub-transform of P = 2^p points whose global twiddle base is B
// uses twiddle index B 2^s + (x >> (p - s)) for butterfly position x; B = 1
// for the column pass and B = N1 + row for the row pass.  The column pass
// reads its 2^p - 1 twiddles from the table (shared by all columns, so
// they stay in cache); the row pass of an FP64 limb would read a different
// 2^p - 1 for every row (the whole table, twice the limb's own bytes), so it
// forms them instead as G[s][y] R[row][s] mod q from two small tables (the
// factorisation is described at ntt_row_tables_size).
#include <type_traits>

#include "butterflies.hpp"
#include "internal.hpp"
#include "modarith.hpp"

namespace ckks {

namespace {

__device__ __forceinline__ int lds_pad(int i) { return i + (i >> 4); }

// A read-only table: read by scalar loads where the index is uniform, else by global (not flat) ones.
typedef const __attribute__((address_space(4))) uint64_t* TableWords;

// The range of a launch that limb number `limb` falls in (a branch-free binary
// search over as many steps as the launch has ranges: a walk over up to 32
// ranges costs a chain of dependent loads, which a short workgroup notices:
// 21.6 -> 17.4 us for 320 limbs of 2^13).
__device__ __forceinline__ int find_range(const NttArgs& a, int limb) {
  int ri = 0;
  for (int step = a.search; step > 0; step >>= 1) ri += limb >= a.start[ri + step] ? step : 0;
  return ri;
}

// The limb that workgroup row `y` of a launch works on: its range (kept in R,
// limb numbers from 0).
__device__ __forceinline__ int find_limb(const NttArgs& a, int y, LimbRange& R) {
  const int ri = find_range(a, y);
  R = a.r[ri];
  return y - a.start[ri];
}
__device__ __forceinline__ int find_limb(const NttSinArgs& a, int y, LimbRange& R) {
  const int item = a.interleave ? y % a.items : y / a.limbs;
  R = LimbRange{};
  R.in = reinterpret_cast<const uint64_t*>(a.in[item]);
  R.out = a.out[item];
  R.prime0 = a.prime0;
  return a.interleave ? y / a.items : y % a.limbs;
}
template <bool SIN>
using NttArgsOf = std::conditional_t<SIN, NttSinArgs, NttArgs>;

// SIN (forward column pass only): the input is the range's shared signed
// coefficients (NttSinArgs).
template <int PLOG, int G, bool COL, bool FWD, bool FP, bool SIN>
__device__ __forceinline__ void ntt_body(const LimbRange& R, int limb, const PrimeDev& pr, int log_n, int epi,
                                         uint64_t* lds, double* tws) {
  constexpr int P = 1 << PLOG;
  constexpr int T = P / 16;           // threads per sub-transform
  constexpr int RS = P + P / 16 + 1;  // LDS row stride (padded)
  Butterflies<FP, FWD> F(pr);
  uint64_t(&v)[16] = F.v;
  const int n = 1 << log_n;
  const TableWords tw = (TableWords)(pr.tw + (FWD ? 0 : ntt_twiddle_words(log_n, FP)));
  const bool first = (COL == FWD);  // first pass of the transform
  const uint64_t* __restrict__ src = (first ? R.in : R.out) + ((SIN && COL) ? 0 : (size_t)limb * n);
  uint64_t* __restrict__ dst = R.out + (size_t)limb * n;

  const int tid = threadIdx.x;
  int g, j;
  if (COL) {
    g = tid % G;
    j = tid / G;
  } else {
    j = tid % T;
    g = tid / T;
  }
  const int sub = blockIdx.x * G + g;  // column index (column pass) or row index (row pass)
  const int ncols = n >> PLOG;
  const uint32_t base = COL ? 1u : (uint32_t)((n >> PLOG) + sub);
  uint64_t* L = lds + g * RS;

  auto addr = [&](int x) -> size_t { return COL ? (size_t)x * ncols + sub : (size_t)sub * P + x; };

  // FP row pass: the factor tables of this direction, G (P doubles, shared
  // by every row) and the R factors of the workgroup's G rows, staged into
  // LDS once (stage_tw) so that no stage waits on a global load for its
  // twiddles.
  const double* tg = tws;
  const double* tr = tws + P + 2 * g * PLOG;
  auto stage_tw = [&]() {
    if (FP && !COL) {
      const double* __restrict__ gs = pr.trow + (FWD ? 0 : ntt_row_tables_size(log_n));
      const double* __restrict__ rs = gs + P + 2 * (size_t)(blockIdx.x * G) * PLOG;
      for (int e = tid; e < P; e += G * P / 16) tws[e] = gs[e];
      for (int e = tid; e < G * 2 * PLOG; e += G * P / 16) tws[P + e] = rs[e];
      __syncthreads();
    }
  };
  // Twiddle of stage s, group y (index base 2^s + y): the value and, on the
  // integer path, its Shoup word, as raw 64-bit words.
  auto twid = [&](int s, uint32_t y, uint64_t& w, uint64_t& wp) {
    if (FP && !COL) {
      // |w| <= 0.75 q
      w = as_u(fp_mulmod(tg[(1u << s) + y], tr[2 * s], tr[2 * s + 1], F.qd));
      wp = 0;
    } else {
      const uint32_t ti = (base << s) + y;
      w = tw[ti];
      wp = FP ? 0 : tw[n + ti];
    }
  };

  // Stages 0..3 in layout "x = j + T u": group y = u >> (4 - s), 2^s groups.
  auto round1 = [&]() {
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int s = FWD ? k : 3 - k;
      const int d = 8 >> s;
      uint64_t W[8], WP[8];
#pragma unroll
      for (int y = 0; y < (1 << s); ++y) twid(s, (uint32_t)y, W[y], WP[y]);
      F.stage_begin(k, d);
#pragma unroll
      for (int u = 0; u < 16; ++u)
        if (!(u & d)) F.bfly(u, d, W[u >> (4 - s)], WP[u >> (4 - s)]);
      F.stage_end(k, k == 3, d);
    }
  };
  // Stages 4..PLOG-1 in layout "x = 16 j + u": group (16 j + u) >> sh with
  // sh = PLOG - s <= 4, i.e. (16 j >> sh) + (u >> sh), 16 >> sh groups.
  auto round2 = [&]() {
#pragma unroll
    for (int k = 4; k < PLOG; ++k) {
      const int s = FWD ? k : PLOG - 1 - (k - 4);
      const int d = P >> (s + 1);
      const int sh = PLOG - s;
      const uint32_t y0 = (uint32_t)(16 * j) >> sh;
      uint64_t W[8], WP[8];
#pragma unroll
      for (int c = 0; c < (16 >> sh); ++c) twid(s, y0 + (uint32_t)c, W[c], WP[c]);
      F.stage_begin(k - 4, d);
#pragma unroll
      for (int u = 0; u < 16; ++u)
        if (!(u & d)) F.bfly(u, d, W[u >> sh], WP[u >> sh]);
      F.stage_end(k - 4, k == PLOG - 1, d);
    }
  };
  auto to_lds = [&](bool layout1) {
#pragma unroll
    for (int u = 0; u < 16; ++u) L[lds_pad(layout1 ? (j + T * u) : (16 * j + u))] = v[u];
  };
  auto from_lds = [&](bool layout1) {
#pragma unroll
    for (int u = 0; u < 16; ++u) v[u] = L[lds_pad(layout1 ? (j + T * u) : (16 * j + u))];
  };
  if (FWD) {
    if constexpr (SIN && COL) {
#pragma unroll
      for (int u = 0; u < 16; ++u) v[u] = src[addr(j + T * u)];
      F.residues();
    } else {
#pragma unroll
      for (int u = 0; u < 16; ++u) v[u] = __builtin_nontemporal_load(src + addr(j + T * u));
    }
    if (!COL) stage_tw();
    if (first)
      F.convert_in();
    else if (!FP)
      F.recentre();
    round1();
    F.recentre();
    to_lds(true);
    __syncthreads();
    from_lds(false);
    round2();
    if (COL) {
      // intermediate of the transform: lazy integers or double bits
#pragma unroll
      for (int u = 0; u < 16; ++u) dst[addr(16 * j + u)] = v[u];
    } else {
      __syncthreads();
      to_lds(false);
      __syncthreads();
      from_lds(true);
      const uint64_t* aux = (epi == EPI_SUBMUL) ? R.aux + (size_t)limb * n : nullptr;
      uint64_t c = 0, cs = 0;
      if (epi == EPI_SUBMUL) {
        c = R.sinv[limb];
        cs = R.sinv_sh[limb];
      }
#pragma unroll
      for (int u = 0; u < 16; ++u) {
        const int x = j + T * u;
        uint64_t y = F.canon(v[u]);
        if (epi == EPI_SUBMUL) y = shoup(__builtin_nontemporal_load(aux + addr(x)) - y + F.q, c, cs, F.q);
        dst[addr(x)] = y;
      }
    }
  } else {
    if (COL) {
#pragma unroll
      for (int u = 0; u < 16; ++u) v[u] = __builtin_nontemporal_load(src + addr(16 * j + u));
    } else {
#pragma unroll
      for (int u = 0; u < 16; ++u) v[u] = __builtin_nontemporal_load(src + addr(j + T * u));
      if (R.copy) {
        uint64_t* __restrict__ cp = R.copy + (size_t)limb * n;
#pragma unroll
        for (int u = 0; u < 16; ++u) cp[addr(j + T * u)] = v[u];
      }
      stage_tw();
      to_lds(true);
      __syncthreads();
      from_lds(false);
      __syncthreads();
    }
    if (first) F.convert_in();
    round2();
    F.recentre();
    to_lds(false);
    __syncthreads();
    from_lds(true);
    round1();
    if (!first) {
      // last pass: times N^-1, canonical
#pragma unroll
      for (int u = 0; u < 16; ++u) dst[addr(j + T * u)] = F.canon(v[u]);
    } else {
      F.recentre();
#pragma unroll
      for (int u = 0; u < 16; ++u) dst[addr(j + T * u)] = v[u];
    }
  }
}

template <int PLOG, int G, bool COL, bool FWD, bool SIN>
__global__ void __launch_bounds__(G*(1 << PLOG) / 16) __attribute__((amdgpu_waves_per_eu(COL ? 1 : 4)))
    ntt_pass(NttArgsOf<SIN> args, const PrimeDev* __restrict__ primes, int log_n, int epi) {
  constexpr int P = 1 << PLOG;
  constexpr int RS = P + P / 16 + 1;
  __shared__ uint64_t lds[G * RS];
  __shared__ double tws[COL ? 1 : P + G * 2 * PLOG];  // FP row pass twiddle factors
  LimbRange R;
  const int limb = find_limb(args, blockIdx.y, R);  // uniform over the workgroup
  const PrimeDev& pr = primes[R.prime0 + limb];
  if (pr.fp)
    ntt_body<PLOG, G, COL, FWD, true, SIN>(R, limb, pr, log_n, epi, lds, tws);
  else
    ntt_body<PLOG, G, COL, FWD, false, SIN>(R, limb, pr, log_n, epi, lds, tws);
}

// ---- N <= 2^13: a whole transform in one workgroup ---------------------------
// A limb of at most 2^13 words (64 KiB, 68 or 72 KiB padded) leaves room for two
// workgroups in a CU's LDS, so all its stages run in one kernel of N / 16
// threads (N / 8 at N = 2^12 and for small launches): rounds of at most 4 stages
// in registers with an LDS exchange between them, half the launches and half the
// memory traffic of two passes: (2,2,4) at N = 2^12 168 -> 117 us, the encoded
// plaintexts' forward passes of the dense LT at N = 2^13 4.84 -> 3.76 ms (2.05 now,
// with 128 plaintexts a launch and no test in the butterflies).  Bound
// by latency (few waves per SIMD) and VALU issue.  (At N = 2^14 a workgroup
// would take a whole CU, and a launch of a few dozen limbs a few dozen CUs:
// measured slower, 208 -> 276 us of forward passes at (4,4,8), level 22.)
// Stage s pairs words 2^(log N-1-s) apart with twiddle 2^s + (x >> (log N - s)),
// read from the full table (small enough at these N to stay in L2).  Round r's
// registers u are LW consecutive bits of x from bit fb up; its k stages use k
// of them.
template <int LOGN, int LW>  // 2^LW words per thread
struct FullRounds {
  static constexpr int kRoundsN = (LOGN + LW - 1) / LW;
  // as even as they divide, longer rounds first
  static constexpr int k(int r) { return LOGN / kRoundsN + (r < LOGN % kRoundsN ? 1 : 0); }
  static constexpr int s0(int r) { return r == 0 ? 0 : s0(r - 1) + k(r - 1); }
  // first of the LW bits of x that round r's registers stand for (the
  // last round's spare bit, if any, is above its stages)
  static constexpr int fb(int r) { return LOGN - s0(r) - LW > 0 ? LOGN - s0(r) - LW : 0; }
  static_assert(k(0) <= LW && s0(kRoundsN - 1) + k(kRoundsN - 1) == LOGN, "all stages");
};
template <int LW>
__device__ __forceinline__ uint32_t full_pad(uint32_t i) { return i + (i >> LW); }

// Word x of register u of thread t in the layout with field base FB.
template <int LW, int FB>
__device__ __forceinline__ uint32_t full_at(uint32_t t, int u) {
  return ((t >> FB) << (FB + LW)) | ((uint32_t)u << FB) | (t & ((1u << FB) - 1));
}

template <int LW, int FROM, int TO>
__device__ __forceinline__ void full_layout(uint64_t (&v)[(1 << LW)], uint32_t t, uint64_t* lds) {
  if constexpr (FROM != TO) {
#pragma unroll
    for (int u = 0; u < (1 << LW); ++u) lds[full_pad<LW>(full_at<LW, FROM>(t, u))] = v[u];
    __syncthreads();
#pragma unroll
    for (int u = 0; u < (1 << LW); ++u) v[u] = lds[full_pad<LW>(full_at<LW, TO>(t, u))];
    __syncthreads();
  }
}

// The twiddles of a stage: groups GB apart in the butterfly order, at most
// 2^(LW-1) per thread.
template <int LW>
struct FullTwiddles {
  uint64_t w[(1 << LW) / 2], wp[(1 << LW) / 2];
};
template <int LOGN, int LW, bool FWD, bool FP, int I, int J>
__device__ __forceinline__ void full_twiddles(FullTwiddles<LW>& T, TableWords tw, uint32_t t) {
  typedef FullRounds<LOGN, LW> FR;
  if constexpr (I < FR::kRoundsN) {
    constexpr int r = FWD ? I : FR::kRoundsN - 1 - I;
    constexpr int fb = FR::fb(r), s = FWD ? FR::s0(r) + J : FR::s0(r) + FR::k(r) - 1 - J, bp = LOGN - 1 - s - fb;
    const uint32_t y0 = (1u << s) + ((t >> fb) << (LW - 1 - bp));
#pragma unroll
    for (int c = 0; c < ((1 << LW) / 2 >> bp); ++c) {
      T.w[c] = tw[y0 + c];
      if (!FP) T.wp[c] = tw[(1 << LOGN) + y0 + c];
    }
  }
}

// Stage J of round I and all that follow, v arriving in the layout HAVE and
// leaving in that of the global memory accesses.  T holds the stage's twiddles;
// the next stage's are loaded before this one's butterflies.
template <int LOGN, int LW, bool FWD, bool FP, int I, int J, int HAVE>
__device__ __forceinline__ void full_stages(Butterflies<FP, FWD, (1 << LW)>& F, const FullTwiddles<LW>& T, TableWords tw, uint32_t t,
                                            uint64_t* lds) {
  typedef FullRounds<LOGN, LW> FR;
  if constexpr (I == FR::kRoundsN) {
    full_layout<LW, HAVE, LOGN - LW>(F.v, t, lds);
  } else {
    constexpr int r = FWD ? I : FR::kRoundsN - 1 - I;
    constexpr int fb = FR::fb(r), k = FR::k(r), s = FWD ? FR::s0(r) + J : FR::s0(r) + k - 1 - J;
    constexpr int bp = LOGN - 1 - s - fb, d = 1 << bp;  // the stage's bit among the registers
    if constexpr (J == 0) {
      full_layout<LW, HAVE, fb>(F.v, t, lds);
      if (I > 0) F.recentre();
    }
    constexpr bool last = J == k - 1;
    constexpr int I1 = last ? I + 1 : I, J1 = last ? 0 : J + 1;
    FullTwiddles<LW> T1;
    full_twiddles<LOGN, LW, FWD, FP, I1, J1>(T1, tw, t);
    __builtin_amdgcn_sched_barrier(0);
    F.stage_begin(J, d);
#pragma unroll
    for (int u = 0; u < (1 << LW); ++u)
      if (!(u & d)) F.bfly(u, d, T.w[u >> (bp + 1)], T.wp[u >> (bp + 1)]);
    F.stage_end(J, last, d);
    full_stages<LOGN, LW, FWD, FP, I1, J1, fb>(F, T1, tw, t, lds);
  }
}

template <int LOGN, int LW, bool FWD, bool FP, bool SIN>
__device__ __forceinline__ void ntt_full_body(const LimbRange& R, int limb, const PrimeDev& pr, int epi,
                                              uint64_t* lds) {
  constexpr int n = 1 << LOGN, kTop = LOGN - LW;  // global memory is accessed as x = u 2^kTop + t
  Butterflies<FP, FWD, (1 << LW)> F(pr);
  uint64_t(&v)[(1 << LW)] = F.v;
  const uint64_t* __restrict__ src = R.in + (SIN ? 0 : (size_t)limb * n);
  uint64_t* __restrict__ dst = R.out + (size_t)limb * n;
  const uint32_t t = threadIdx.x;
  auto at = [&](int u) -> uint32_t { return full_at<LW, kTop>(t, u); };
  if constexpr (SIN) {
#pragma unroll
    for (int u = 0; u < (1 << LW); ++u) v[u] = src[at(u)];
    F.residues();
  } else {
#pragma unroll
    for (int u = 0; u < (1 << LW); ++u) v[u] = __builtin_nontemporal_load(src + at(u));
  }
  if (!FWD && R.copy) {
    uint64_t* __restrict__ cp = R.copy + (size_t)limb * n;
#pragma unroll
    for (int u = 0; u < (1 << LW); ++u) cp[at(u)] = v[u];
  }
  const TableWords tw = (TableWords)(pr.tw + (FWD ? 0 : ntt_twiddle_words(LOGN, FP)));
  FullTwiddles<LW> T;
  full_twiddles<LOGN, LW, FWD, FP, 0, 0>(T, tw, t);
  F.convert_in();
  full_stages<LOGN, LW, FWD, FP, 0, 0, kTop>(F, T, tw, t, lds);
  if (FWD && epi == EPI_SUBMUL) {
    const uint64_t* aux = R.aux + (size_t)limb * n;
    const uint64_t c = R.sinv[limb], cs = R.sinv_sh[limb];
#pragma unroll
    for (int u = 0; u < (1 << LW); ++u)
      dst[at(u)] = shoup(__builtin_nontemporal_load(aux + at(u)) - F.canon(v[u]) + F.q, c, cs, F.q);
  } else {
#pragma unroll
    for (int u = 0; u < (1 << LW); ++u) dst[at(u)] = F.canon(v[u]);
  }
}

template <int LOGN, int LW, bool FWD, bool SIN>
__global__ void __launch_bounds__(1 << (LOGN - LW)) __attribute__((amdgpu_waves_per_eu(4)))
    ntt_full(NttArgsOf<SIN> args, const PrimeDev* __restrict__ primes, int epi) {
  __shared__ uint64_t lds[(1 << LOGN) + (1 << LOGN) / (1 << LW)];
  LimbRange R;
  const int limb = find_limb(args, blockIdx.x, R);
  const PrimeDev& pr = primes[R.prime0 + limb];
  if (pr.fp)
    ntt_full_body<LOGN, LW, FWD, true, SIN>(R, limb, pr, epi, lds);
  else
    ntt_full_body<LOGN, LW, FWD, false, SIN>(R, limb, pr, epi, lds);
}

// Sub-transforms per workgroup: 4096 / P (16 at N = 2^16: 256 threads,
// 128-byte column segments).  A quarter of that for launches over a few
// limbs (4x the workgroups) was measured slower: the inverse column pass
// over 9-10 limbs 0.106 -> 0.147 ms per (4,4,4) LT, its 32-byte column
// segments costing more than the extra workgroups gain.
template <int PLOG, bool COL, bool FWD, bool SIN>
hipError_t launch_pass(const ckks_params* P, const NttArgsOf<SIN>& a, int total, double words, int epi,
                       hipStream_t s) {
  constexpr int Pn = 1 << PLOG;
  constexpr int G = 4096 / Pn;
  const int subs = P->n >> PLOG;  // columns (column pass) or rows
  if (subs % G) return hipErrorInvalidValue;
  ProfScope prof(FWD ? (COL ? CKKS_KERNEL_NTT_FWD_COL : CKKS_KERNEL_NTT_FWD_ROW)
                     : (COL ? CKKS_KERNEL_NTT_INV_COL : CKKS_KERNEL_NTT_INV_ROW),
                 s, words * P->n * 8);
  hipLaunchKernelGGL((ntt_pass<PLOG, G, COL, FWD, SIN>), dim3(subs / G, total), dim3(G * Pn / 16), 0, s, a,
                     P->d_primes, P->log_n, epi);
  return hipGetLastError();
}

// Words moved per coefficient position: a read and a write of each limb, the
// kept limbs of the division epilogue, the copies of an inverse transform.
double words_of(const NttArgs& a, int total, int epi, bool copies) {
  double words = (double)total * (epi == EPI_SUBMUL ? 3 : 2);
  if (copies)
    for (int i = 0; i < a.nr; ++i) words += a.r[i].copy ? a.r[i].count : 0;
  return words;
}

template <int PA, int PB>
hipError_t launch_both(const ckks_params* P, bool forward, const NttArgs& a, int total, int epi, hipStream_t s) {
  hipError_t e;
  if (forward) {
    e = launch_pass<PA, true, true, false>(P, a, total, words_of(a, total, EPI_NONE, false), EPI_NONE, s);
    if (e != hipSuccess) return e;
    return launch_pass<PB, false, true, false>(P, a, total, words_of(a, total, epi, false), epi, s);
  }
  e = launch_pass<PB, false, false, false>(P, a, total, words_of(a, total, EPI_NONE, true), EPI_NONE, s);
  if (e != hipSuccess) return e;
  return launch_pass<PA, true, false, false>(P, a, total, words_of(a, total, EPI_NONE, false), EPI_NONE, s);
}

// Row passes of encoded plaintexts over integer-path primes are taken prime by
// prime, not item by item: such a pass reads twice as many twiddle words as
// data words, and this way they come from L2 after the first item (44 limbs of
// 54 bits x 32 plaintexts at N = 2^16: 416 -> 371 us; FP64-path limbs read small
// tables and are better off item by item, as are column passes, whose input all
// limbs of an item share).
template <int PA, int PB>
hipError_t launch_both_encoded(const ckks_params* P, NttSinArgs a, hipStream_t s) {
  const int total = a.items * a.limbs;
  a.interleave = 0;
  hipError_t e = launch_pass<PA, true, true, true>(P, a, total, total + a.items, EPI_NONE, s);
  if (e != hipSuccess) return e;
  a.interleave = 1;
  for (int l = 0; l < a.limbs; ++l)
    if (P->primes[a.prime0 + l] < kFpPrimeLimit) a.interleave = 0;
  return launch_pass<PB, false, true, true>(P, a, total, 2.0 * total, EPI_NONE, s);
}

// The whole transform in one launch.  Timed as the column pass of its
// direction.
template <int LOGN, int LW, bool FWD, bool SIN>
hipError_t launch_full(const ckks_params* P, const NttArgsOf<SIN>& a, int total, double words, int epi,
                       hipStream_t s) {
  ProfScope prof(FWD ? CKKS_KERNEL_NTT_FWD_COL : CKKS_KERNEL_NTT_INV_COL, s, words * P->n * 8);
  hipLaunchKernelGGL((ntt_full<LOGN, LW, FWD, SIN>), dim3(total), dim3(1 << (LOGN - LW)), 0, s, a, P->d_primes, epi);
  return hipGetLastError();
}

// Words per thread of the one-kernel transforms: 8 at N = 2^12 (16 against 8: one
// limb 12.4 -> 10.0 us, 640 limbs 28.7 -> 21.1, 2176 limbs 47 -> 42).  At N = 2^13 a
// launch of at most a limb per CU is bound by one workgroup's latency, so its
// limbs are spread over more waves too (one limb 16.3 -> 14.3, 250 limbs 22.5 ->
// 18.7); larger ones run faster with the fewer exchanges of 16 words (8 against 16:
// 260 limbs alike, 640 43.0 -> 40.9, 2176 109 -> 92).
template <bool FWD, bool SIN>
hipError_t launch_one_kernel(const ckks_params* P, const NttArgsOf<SIN>& a, int total, double words, int epi,
                             hipStream_t s) {
  if (P->log_n == 12) return launch_full<12, 3, FWD, SIN>(P, a, total, words, epi, s);
  if (total <= 256) return launch_full<13, 3, FWD, SIN>(P, a, total, words, epi, s);
  return launch_full<13, 4, FWD, SIN>(P, a, total, words, epi, s);
}

}  // namespace

hipError_t launch_ntt(const ckks_params* P, bool forward, const NttArgs& args, int total_limbs, int epi,
                      hipStream_t s) {
  if (total_limbs <= 0) return hipSuccess;
  NttArgs a = args;
  int at = 0;
  for (int i = 0; i < kMaxRanges; ++i) {
    a.start[i] = i < a.nr ? at : INT32_MAX;
    at += i < a.nr ? a.r[i].count : 0;
  }
  if (at != total_limbs) return hipErrorInvalidValue;
  static_assert((kMaxRanges & (kMaxRanges - 1)) == 0, "binary search");
  a.search = 0;
  for (int step = 1; step < a.nr; step *= 2) a.search = step;
  switch (P->log_n) {
    case 12:
    case 13: {
      const double words = words_of(a, total_limbs, epi, true);
      return forward ? launch_one_kernel<true, false>(P, a, total_limbs, words, epi, s)
                     : launch_one_kernel<false, false>(P, a, total_limbs, words, epi, s);
    }
    case 14: return launch_both<7, 7>(P, forward, a, total_limbs, epi, s);
    case 15: return launch_both<8, 7>(P, forward, a, total_limbs, epi, s);
    case 16: return launch_both<8, 8>(P, forward, a, total_limbs, epi, s);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_ntt_encoded(const ckks_params* P, const NttSinArgs& a, hipStream_t s) {
  if (a.items < 1 || a.items > kMaxEnc || a.limbs < 1 || a.prime0 < 0 || a.prime0 + a.limbs > P->Kmax())
    return hipErrorInvalidValue;
  const int total = a.items * a.limbs;
  switch (P->log_n) {
    case 12:
    case 13: return launch_one_kernel<true, true>(P, a, total, total + a.items, EPI_NONE, s);
    case 14: return launch_both_encoded<7, 7>(P, a, s);
    case 15: return launch_both_encoded<8, 7>(P, a, s);
    case 16: return launch_both_encoded<8, 8>(P, a, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace ckks
