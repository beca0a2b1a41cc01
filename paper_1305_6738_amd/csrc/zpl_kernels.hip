// zpl_kernels.hip -- gfx950 kernels of the Zipf (xmin = 1) MLE + KS Monte
// Carlo path of Rappos & Robert (2013): CDF/guide table build, the replicate
// kernels (lane, wave and heavy forms), the dataset fit, order-statistic
// selection, and the bootstrap count.
//
// Per replicate (Sect. 3/4 of the paper): n draws from eq. (1) by inverse CDF
// with a Philox4x32-10 counter stream, S = sum ln x (exact 128-bit fixed
// point), alpha_hat from eq. (2), D from eq. (3) over the distinct values.
// None of this is a dense contraction: the kernels are VALU/LDS work laid out
// for wave64, with LDS-resident tables and histograms.
#include <hip/hip_runtime.h>

#include "zpl_kernels.hpp"
#include "zpl_math.hpp"

namespace zpl {

// ---------------------------------------------------------------------------
// Wave-level helpers (wave64).
// ---------------------------------------------------------------------------
__device__ __forceinline__ int lane_id() { return (int)(threadIdx.x & 63u); }

__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

__device__ __forceinline__ uint32_t shfl_xor_u32(uint32_t v, int m) {
  return (uint32_t)__shfl_xor((int)v, m, 64);
}
__device__ __forceinline__ uint64_t shfl_xor_u64(uint64_t v, int m) {
  const uint32_t lo = shfl_xor_u32((uint32_t)v, m);
  const uint32_t hi = shfl_xor_u32((uint32_t)(v >> 32), m);
  return ((uint64_t)hi << 32) | lo;
}
__device__ __forceinline__ uint32_t wave_sum_u32(uint32_t v) {
#pragma unroll
  for (int m = 32; m > 0; m >>= 1) v += shfl_xor_u32(v, m);
  return v;
}
__device__ __forceinline__ U128 wave_sum_u128(U128 v) {
#pragma unroll
  for (int m = 32; m > 0; m >>= 1) {
    const uint64_t lo = shfl_xor_u64(v.lo, m);
    const uint64_t hi = shfl_xor_u64(v.hi, m);
    u128_add(v, lo, hi);
  }
  return v;
}
__device__ __forceinline__ uint64_t lanes_below(int lane) {
  return lane == 0 ? 0ull : (~0ull >> (64 - lane));
}

// base plus the number of mask's lanes below this one.
__device__ __forceinline__ uint32_t place_below(uint64_t mask, uint32_t base = 0u) {
  return (uint32_t)__builtin_amdgcn_mbcnt_hi(
      (uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, base));
}

// ---------------------------------------------------------------------------
// Inverse-CDF sampling: x = min{k in 1..kH : T[k] >= U} (the ">=" rule of
// the paper's sampler).  U = m 2^-53 with m = (w >> 11) | 1 an odd 53-bit
// integer, and the LDS copy of the table holds TI[k] = floor(T[k] 2^53), so
// T[k] >= U exactly when TI[k] >= m, and U is never formed.  The guide brackets
// the answer in [g[b], g[b+1]]; most brackets are one or two values wide, decided
// by one comparison of first words (fast_offsets).  Wider brackets, equal words
// and U > T[kH] (the tail) are deferred and resolved 64 at a time.
// ---------------------------------------------------------------------------
__device__ __forceinline__ uint64_t m53(uint32_t hi, uint32_t lo) {
  return ((((uint64_t)hi) << 32 | (uint64_t)lo) >> 11) | 1ull;
}

// ---------------------------------------------------------------------------
// KS distance (eq. 3) over the distinct values of one replicate, in
// ascending order.  With C the count of draws <= t and Z(t) = zeta(a, t+1)
// (so F(t) = 1 - Z(t)/zeta(a)), each distinct value v contributes
// |Z(v)/zeta - (n - C(v))/n| and |Z(v-1)/zeta - (n - C(v-1))/n|: between
// sample values S_n is flat and F rises, so the sup over all t is reached at
// a sample value or one below it.  Values <= 16 use the precomputed head
// suf[]; for larger ones Z(v) comes from the Euler-Maclaurin tail and
// Z(v-1) = Z(v) + v^-a.  Src yields the distinct values: small(v) returns
// the count of v for v = 1..16 in order, then next_large() returns the
// remaining (value, count) pairs ascending.  Every kernel evaluates the terms
// by these expressions, in whatever order and for whichever values can reach
// the maximum, so all give the same D bit for bit.
//
// KS distance (eq. 3) under the truncated law on 1..K.  Where its sums go by
// Euler-Maclaurin (trunc_em), as described, with the survival sums of
// trunc_tail.  Else (K < 161) F(t) = P(t)/Z with P(t) = sum_{k<=t} k^-a
// accumulated in ascending k as the distinct values are visited, and Z the K
// terms from K down.  The terms are |F(v) - C(v)/n| and |F(v-1) - C(v-1)/n|
// per distinct v either way.
template <class Src>
__device__ __forceinline__ double ks_distance_trunc(Src& src, double a, uint32_t K, int64_t n,
                                                    const double* __restrict__ ln) {
  const double idn = 1.0 / (double)n;
  int64_t C = 0;
  double D = 0.0;
  if (trunc_em(a, K)) {
    const EmCoef E = em_coef(a);
    const TruncEnd te = trunc_end(E, K, ln);
    double suf[17];
    survival_head_trunc(E, te, ln, suf);
    const double iz = 1.0 / suf[0];
    auto term = [&](double zv, double zv1, uint32_t c) {
      const double t2 = fabs(fma(zv1, iz, -(double)(n - C) * idn));
      C += c;
      const double t1 = fabs(fma(zv, iz, -(double)(n - C) * idn));
      D = fmax(D, fmax(t1, t2));
    };
#pragma unroll
    for (int v = 1; v <= 16; ++v) {
      const uint32_t c = src.small(v);
      if (c) term(suf[v], suf[v - 1], c);
    }
    double zprev = suf[16];
    int64_t vprev = 16, v;
    uint32_t c;
    while (src.next_large(v, c)) {
      const double zv = trunc_tail(E, te, v, ln[v + 1]);  // v <= K <= kH
      term(zv, v - 1 == vprev ? zprev : zv + pow_neg(a, ln[v]), c);
      zprev = zv;
      vprev = v;
    }
    return D;
  }
  const double iz = 1.0 / zeta3_trunc(a, K, ln).z0;  // the normaliser Z_K(a)
  double pw[kDirect + 1];
  direct_powers(a, K, ln, pw);
  double P = 0.0;  // P(k - 1), then P(k)
  auto term = [&](double Pl, double Pv, uint32_t c) {
    const double t2 = fabs(fma(Pl, iz, -(double)C * idn));
    C += c;
    const double t1 = fabs(fma(Pv, iz, -(double)C * idn));
    D = fmax(D, fmax(t1, t2));
  };
#pragma unroll
  for (int k = 1; k <= kDirect; ++k) {
    const double Pk = P + pw[k];
    const uint32_t ck = src.small(k);
    if (ck) term(P, Pk, ck);
    P = Pk;
  }
  int64_t v;
  uint32_t c;
  bool have = src.next_large(v, c);
  int64_t k = kDirect;  // P = P(k)
  while (have) {
    while (k < v - 1) {
      ++k;
      P += pow_neg(a, ln[k]);
    }
    ++k;
    const double Pk = P + pow_neg(a, ln[k]);
    term(P, Pk, c);
    P = Pk;
    have = src.next_large(v, c);
  }
  return D;
}

// The MLE's start table, behind the logarithms and their fixed-point form in
// the context's constants (k_ln_table, k_mle_guess).
__device__ __forceinline__ const double* mle_guess_table(const double* ln) {
  return ln + 2 * (kH + 2);
}

// ln x 2^53 as an integer, from the context's table behind the logarithms.
__device__ __forceinline__ const uint64_t* ln_fixed_table(const double* ln) {
  return reinterpret_cast<const uint64_t*>(ln + kH + 2);
}
__device__ __forceinline__ uint64_t ln_fixed_at(int64_t v, const double* __restrict__ ln) {
  return v <= (int64_t)(kH + 1) ? ln_fixed_table(ln)[v] : (uint64_t)(log((double)v) * 0x1p53);
}

// Distances closer than this to the largest one found are always evaluated:
// far above the rounding of a bound (a few 2^-53), far below any distance.
constexpr double kPruneMargin = 1e-12;

// S (with the paper's all-ones rule), alpha_hat (eq. 2) and D (eq. 3) for the
// truncated law on 1..K, by one lane.
template <class Src>
__device__ __forceinline__ void finish_truncated(Src& src, const U128& S, int64_t n, uint32_t fl,
                                                 const double* __restrict__ ln, uint32_t K,
                                                 double& ahat, double& D, uint32_t& flags) {
  double Sd;
  if (S.lo == 0 && S.hi == 0) {  // every draw was 1: S := ln 2
    Sd = ln[2];
    fl |= kFlagAllOnes;
  } else {
    Sd = u128_to_S(S);
  }
  ahat = mle_alpha_trunc(Sd / (double)n, K, ln, &fl);
  D = ks_distance_trunc(src, ahat, K, n, ln);
  flags = fl;
}

__device__ __forceinline__ void write_outputs(const Outputs& o, int64_t idx, double D,
                                              double a, uint32_t fl, uint64_t fp) {
  if (o.D) o.D[idx] = D;
  if (o.ahat) o.ahat[idx] = a;
  if (o.flags) o.flags[idx] = fl;
  if (o.fp) o.fp[idx] = fp;
}

// ---------------------------------------------------------------------------
// Distinct-value sources.
// ---------------------------------------------------------------------------
// LDS words as such (address space 3) for functions that are called, not
// inlined: through a generic pointer their LDS accesses would be flat ones,
// which are not ordered with the callers' LDS instructions.
typedef __attribute__((address_space(3))) uint32_t LdsU32;
// Lane mode: a per-lane column of packed 16-bit counters for values 1..kHLB
// (dword b holds values 2b+1 and 2b+2) and a sorted per-lane overflow list.
struct LaneSrc {
  const LdsU32* hist;    // element (b, lane) at hist[b * 64]
  const int64_t* ov;     // element (p, lane) at ov[p * 64]
  int oc;
  int bin;  // next value to inspect in 17..kHLB
  int p;    // next overflow index
  __device__ __forceinline__ uint32_t count(int v) const {
    const uint32_t w = hist[((v - 1) >> 1) * 64];
    return ((v - 1) & 1) ? (w >> 16) : (w & 0xffffu);
  }
  __device__ __forceinline__ uint32_t small(int v) { return count(v); }
  __device__ __forceinline__ bool next_large(int64_t& v, uint32_t& c) {
    while (bin <= kHLB) {
      const int b = bin++;
      const uint32_t k = count(b);
      if (k) {
        v = b;
        c = k;
        return true;
      }
    }
    if (p < oc) {
      const int64_t x = ov[p * 64];
      uint32_t k = 0;
      while (p < oc && ov[p * 64] == x) {
        ++p;
        ++k;
      }
      v = x;
      c = k;
      return true;
    }
    return false;
  }
};

__device__ __forceinline__ double wave_max_f64(double v) {
#pragma unroll
  for (int m = 32; m > 0; m >>= 1) {
    const uint64_t b = shfl_xor_u64((uint64_t)__double_as_longlong(v), m);
    v = fmax(v, __longlong_as_double((long long)b));
  }
  return v;
}

// ---------------------------------------------------------------------------
// Wave-cooperative helpers.
// ---------------------------------------------------------------------------
// Ordering of one wave's global-memory stores before its later loads.
__device__ __forceinline__ void wave_sync_global() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
}

__device__ __forceinline__ int next_pow2(int v) {
  int p = 1;
  while (p < v) p <<= 1;
  return p;
}

// Ring of deferred draws (lane form), by number and lane.  Before an
// iteration's appends (at most 64 lanes x 4 draws) it holds fewer than 64
// entries, so it never overflows; a power of two for its places.
constexpr int kRing = 512;

// ---------------------------------------------------------------------------
// A wave's LDS in the lane form.
// ---------------------------------------------------------------------------
static_assert(kHLB % 2 == 0, "two 16-bit counters per dword; value kHLB + 1 maps to the pad row");
struct alignas(16) LaneRegion {
  // dword b of lane l at hist[b * 64 + l]; row kHLB / 2 is a pad that takes
  // the draw loop's no-op counts (never read)
  uint32_t hist[(kHLB / 2 + 1) * 64];
  uint32_t ring[kRing];          // deferred draws
  uint32_t ovc[64];  // values the drains added to a lane's list (may exceed its room)
  uint32_t fl[64];   // flags per lane
};

// Out of line: inlined into the persistent kernels' cell switch it takes
// registers from their hot loops.
static __device__ __noinline__ uint32_t guide_pack_dev(const uint16_t* g, int b, int sh,
                                                       uint64_t timax) {
  return guide_pack(as_global(g), b, sh, timax);
}

// Stages the cell's table, as the words of the integers floor(F(k) 2^53)
// (threshold_hi, then threshold_lo), and packed guide (guide_offsets) into LDS.
__device__ __forceinline__ void load_cell_tables(uint32_t* T, uint32_t* guide,
                                                 const double* __restrict__ Tg,
                                                 const uint16_t* __restrict__ g,
                                                 const DevCell& c, int tid, int nthreads) {
  for (int k = tid; k < kH; k += nthreads) {
    const uint64_t t = table_int(Tg[k]);
    T[k] = threshold_hi(t);
    T[kH + k] = threshold_lo(t);
  }
  const uint64_t timax = table_int(c.tmax);
  const int sh = (int)c.gsh;
  for (int b = tid; b < kGuide; b += nthreads)
    guide[b] = guide_offsets(guide_pack_dev(g, b, sh, timax));
}

// ---------------------------------------------------------------------------
// Lane form: one replicate per lane.
// ---------------------------------------------------------------------------
// Buckets of a lane's values above the column, eight per octave: 48.., 52..,
// 56.., 60.., 64.., 72.., ..., the last one (11264..) open.
constexpr int kLaneBuckets = 64;
__device__ __forceinline__ int lane_bucket(uint64_t v) {
  const int e = 63 - __clzll((long long)v);
  const int b = 8 * (e - 5) + (int)((v >> (e - 3)) & 7u) - 4;
  return b < kLaneBuckets - 1 ? b : kLaneBuckets - 1;
}
__device__ __forceinline__ uint64_t lane_bucket_start(int b) {
  return (uint64_t)(8 + ((b + 4) & 7)) << (2 + ((b + 4) >> 3));
}

// Lanes with up to this many such values do without the buckets, whose edges take
// up to 63 survival sums a lane: 100,000 replicates of 10 draws at alpha = 1.2 took
// 271 us with them, 201 without.
constexpr int kLaneFew = 12;
// Lanes with up to this many occupied buckets look at the edges of those only (at
// most two sums for each, of 63 in all): 180,000 replicates of 30 draws at alpha =
// 1.2 took 359 us over all edges, 318 so; a wave with more goes over all in turn.
constexpr int kLaneSparse = 24;
// The finish's use of the wave's LDS region once the columns are read.
typedef __attribute__((address_space(3))) uint8_t LdsU8;
typedef __attribute__((address_space(3))) uint64_t LdsU64;
constexpr int kLanePairs =
    ((int)sizeof(LaneRegion) - 64 * kLaneBuckets - 64 * 4 - 64 * 8) / 8;  // gathered values
static_assert(kLanePairs >= kLaneCap, "one lane's values always fit");

// S, MLE and KS distance of one replicate per lane (called, not inlined: the
// draw loop keeps its registers); every lane of the wave takes part, ok marks
// those with a replicate.  region: the wave's LDS, the lane's packed counts at
// dword b * 64 + lane; slots: its values above them, unsorted (the first myc
// slots and the last od of kLaneCap), with as many free ones behind.
// The KS needs no sort: past 16, past kHLB and between the edges of each
// bucket both distributions are bounded by their values at the edges, and only
// a bucket whose bound reaches the largest distance found has its values
// looked at.  Those of all lanes are gathered into LDS and evaluated 64 at a
// time whichever lane they belong to (a few lanes have most of them), each
// ranked among its own lane's.  A rank sort of every value above the column
// instead took 2.0 of 5.1 ns per replicate at alpha = 1.75, n = 1,000.
struct LaneOut {
  double a, D;
  uint64_t fp;
  uint32_t flags;
};
template <bool kTruncLaw>
static __device__ __noinline__ LaneOut lane_finish(LdsU32* region, int64_t* slots_, int myc, int od,
                                                   bool ok, int64_t n, uint32_t fl, uint32_t K,
                                                   bool want_fp, const double* ln_) {
  int64_t* slots = as_global(slots_);
  const double* __restrict__ ln = as_global(ln_);
  LaneOut o;
  o.fp = 0;
  const int lane = lane_id();
  const LdsU32* column = region + lane;
  const int oc = myc + od;
  int64_t* more = slots + 64 * kLaneCap;
  auto ov = [&](int q) -> int64_t {
    return slots[(q < myc ? q : kLaneCap - od + (q - myc)) * 64];
  };
  // exact sums of the low and high words of ln v 2^53
  uint64_t slo = 0, shi = 0;
#pragma unroll 4
  for (int q = 0; q < oc; ++q) {
    const int64_t v = ov(q);
    const uint64_t lf = ln_fixed_at(v, ln);
    slo += (uint32_t)lf;
    shi += lf >> 32;
    if (want_fp) o.fp += mix64((uint64_t)v);
  }
  for (int b = 0; b < kHLB / 2; ++b) {
    const uint32_t wv = column[b * 64];
#pragma unroll
    for (int half = 0; half < 2; ++half) {
      const uint32_t k = half ? (wv >> 16) : (wv & 0xffffu);
      const int64_t v = 2 * b + half + 1;
      const uint64_t lf = ln_fixed_table(ln)[v];
      slo += (uint64_t)k * (uint32_t)lf;
      shi += (uint64_t)k * (uint32_t)(lf >> 32);
      if (want_fp) o.fp += (uint64_t)k * mix64((uint64_t)v);
    }
  }
  const uint64_t s1 = slo + (shi << 32);
  const U128 S{s1, (shi >> 32) + (s1 < slo ? 1u : 0u)};
  o.flags = fl;
  double Sd;
  if (S.lo == 0 && S.hi == 0) {  // every draw was 1: S := ln 2
    Sd = ln[2];
    o.flags |= kFlagAllOnes;
  } else {
    Sd = u128_to_S(S);
  }
  // sum of k^-a over k > v (v >= 16)
  auto survival = [&](const EmCoef& e, const TruncEnd& t, int64_t v) -> double {
    if constexpr (kTruncLaw) return trunc_tail(e, t, v, ln[v <= (int64_t)kH ? v + 1 : 0]);
    return survival_next(e, v, ln);
  };
  if constexpr (kTruncLaw)
    o.a = mle_alpha_trunc(Sd / (double)n, K, ln, &o.flags);
  else
    o.a = mle_alpha_start(Sd / (double)n, ln, mle_guess_table(ln), &o.flags);
  const EmCoef E = em_coef(o.a);
  TruncEnd te = {};
  if constexpr (kTruncLaw) te = trunc_end(E, K, ln);
  const double idn = 1.0 / (double)n;
  const uint32_t nu = (uint32_t)n;  // lane form: n <= 65535
  double D = 0.0, iz, zprev;
  uint32_t C = 0;
  {
    double suf[17];
    if constexpr (kTruncLaw)
      survival_head_trunc(E, te, ln, suf);
    else
      survival_head(E, ln, suf);
    iz = 1.0 / suf[0];
#pragma unroll
    for (int v = 1; v <= 16; ++v) {
      const uint32_t wv = column[((v - 1) >> 1) * 64];
      const uint32_t c = (v & 1) ? (wv & 0xffffu) : (wv >> 16);
      if (c) {
        const double t2 = fabs(fma(suf[v - 1], iz, -(double)(nu - C) * idn));
        C += c;
        const double t1 = fabs(fma(suf[v], iz, -(double)(nu - C) * idn));
        D = fmax(D, fmax(t1, t2));
      }
    }
    zprev = suf[16];
  }
  bool live = ok && fmax(zprev * iz, (double)(nu - C) * idn) > D - kPruneMargin;
  bool prev = true;  // zprev is the survival sum past v - 1
  if (live) {
    for (int v = 17; v <= kHLB; ++v) {
      const uint32_t wv = column[((v - 1) >> 1) * 64];
      const uint32_t c = (v & 1) ? (wv & 0xffffu) : (wv >> 16);
      if (c) {
        const double zv = survival(E, te, v);
        const double zv1 = prev ? zprev : zv + pow_neg(E.s, ln[v]);
        const double t2 = fabs(fma(zv1, iz, -(double)(nu - C) * idn));
        C += c;
        const double t1 = fabs(fma(zv, iz, -(double)(nu - C) * idn));
        D = fmax(D, fmax(t1, t2));
        zprev = zv;
      }
      prev = c != 0u;
    }
    if (!prev) zprev = survival(E, te, kHLB);
    live = oc > 0 && fmax(zprev * iz, (double)oc * idn) > D - kPruneMargin;
  }
  if (__ballot(live) == 0ull) {
    o.D = D;
    return o;
  }
  // the lane's bucket counts, then in their place the counts below each bucket
  wave_sync();  // every column has been read
  LdsU8* cum = (LdsU8*)region;  // bucket b of lane l at cum[b * 64 + l]
  LdsU32* ends = region + 16 * kLaneBuckets;       // 64 inclusive counts
  LdsU64* dmax = (LdsU64*)(ends + 64);             // 64 distances
  LdsU64* pairs = dmax + 64;                       // kLanePairs values
  // few values in every lane: all are in reach of one bucket from kHLB + 1 on
  const bool few = __ballot(live && oc > kLaneFew) == 0ull;
  uint64_t um = few && live ? ~0ull : 0ull;  // buckets in reach
  if (!few) {
#pragma unroll 4
    for (int k = lane; k < 16 * kLaneBuckets; k += 64) region[k] = 0u;
    wave_sync();
  }
  uint64_t occupied = 0ull;
  if (live && !few) {
    for (int q = 0; q < oc; ++q) {
      const int b = lane_bucket((uint64_t)ov(q));
      LdsU8* c = cum + 64 * b + lane;
      *c = (uint8_t)(*c + 1u);
      occupied |= 1ull << b;
    }
  }
  // each bucket's bound, kept in scratch, and the largest distance at an edge: of
  // the occupied buckets, or where they are many in some lane of all in turn (the
  // right edge of one is the next one's left)
  const bool all = __ballot(__popcll(occupied) > kLaneSparse) != 0ull;
  if (occupied != 0ull) {
    uint32_t lower = 0;
    double zl = zprev * iz, Dlow = D;
    int next = 0;  // the bucket whose left edge zl is
    uint64_t todo = all ? ~0ull : occupied, seen = 0ull;
    while (todo != 0ull) {
      const int nb = __ffsll((long long)todo) - 1;
      todo &= todo - 1ull;
      seen |= 1ull << nb;
      const uint32_t c = cum[64 * nb + lane];
      cum[64 * nb + lane] = (uint8_t)lower;
      const double sl = (double)((uint32_t)oc - lower) * idn;
      lower += c;
      const double sr = (double)((uint32_t)oc - lower) * idn;
      if (nb != next) {
        zl = iz * survival(E, te, (int64_t)lane_bucket_start(nb) - 1);
        Dlow = fmax(Dlow, fabs(zl - sl));
      }
      const double zr = nb < kLaneBuckets - 1
                            ? iz * survival(E, te, (int64_t)lane_bucket_start(nb + 1) - 1)
                            : 0.0;
      more[64 * nb] = __double_as_longlong(c ? fmax(zl - sr, sl - zr) : 0.0);
      Dlow = fmax(Dlow, fabs(zr - sr));
      if (fmax(zr, sr) <= Dlow - kPruneMargin) todo = 0ull;
      zl = zr;
      next = nb + 1;
    }
    for (uint64_t m = seen & occupied; m != 0ull; m &= m - 1ull) {
      const int b = __ffsll((long long)m) - 1;
      if (__longlong_as_double(more[64 * b]) > Dlow - kPruneMargin) um |= 1ull << b;
    }
  }
  uint64_t pm = 0ull;  // buckets whose first value's predecessor was drawn
  uint32_t cnt = few && live ? (uint32_t)oc : 0u;
  if (um != 0ull && !few) {
#pragma unroll 4
    for (int q = 0; q < oc; ++q) {
      const uint64_t v = (uint64_t)ov(q);
      const int b = lane_bucket(v), b1 = lane_bucket(v + 1u);
      cnt += (uint32_t)((um >> b) & 1ull);
      if (b1 != b) pm |= 1ull << b1;
    }
  }
  uint32_t incl = cnt;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const uint32_t u = (uint32_t)__shfl_up((int)incl, d, 64);
    if (lane >= d) incl += u;
  }
  ends[lane] = incl;
  dmax[lane] = (uint64_t)__double_as_longlong(D);
  const uint32_t total = (uint32_t)__shfl((int)incl, 63, 64);
  const uint32_t info = (uint32_t)oc | (prev ? 0x10000u : 0u);
  for (uint32_t done = 0; done < total;) {  // windows of whole lanes that fit
    const bool mine = cnt != 0u && incl - cnt >= done && incl - done <= (uint32_t)kLanePairs;
    uint32_t p = incl - cnt - done;
    if (mine) {
#pragma unroll 4
      for (int q = 0; q < oc; ++q) {
        const int64_t v = ov(q);
        if ((um >> lane_bucket((uint64_t)v)) & 1ull) pairs[p++] = (uint64_t)v;
      }
    }
    // the last lane of the window (lanes in order: the prefix counts ascend)
    const uint64_t in = __ballot(mine);
    const uint32_t next = (uint32_t)__shfl((int)incl, 63 - __clzll((long long)in), 64);
    wave_sync();
    for (uint32_t f0 = done; f0 < next; f0 += 64u) {
      const uint32_t f = f0 + (uint32_t)lane;
      const bool valid = f < next;
      int owner = 0;  // the first lane whose inclusive count exceeds f
#pragma unroll
      for (int step = 32; step > 0; step >>= 1)
        if (ends[owner + step - 1] <= f) owner += step;
      owner = valid ? owner : 0;
      const uint32_t e1 = ends[owner], e0 = owner > 0 ? ends[owner - 1] : 0u;
      auto from = [&](uint64_t x) {
        const uint32_t lo = (uint32_t)__shfl((int)(uint32_t)x, owner, 64);
        const uint32_t hi = (uint32_t)__shfl((int)(uint32_t)(x >> 32), owner, 64);
        return ((uint64_t)hi << 32) | lo;
      };
      const double as = __longlong_as_double((long long)from((uint64_t)__double_as_longlong(o.a)));
      const double izo = __longlong_as_double((long long)from((uint64_t)__double_as_longlong(iz)));
      const uint64_t pmo = from(pm);
      const uint32_t io = (uint32_t)__shfl((int)info, owner, 64);
      if (valid) {
        const int64_t v = (int64_t)pairs[f - done];
        const int b = few ? 0 : lane_bucket((uint64_t)v);
        const int64_t start = few ? kHLB + 1 : (int64_t)lane_bucket_start(b);
        uint32_t lt = 0, eq = 0;
        bool pres = v == kHLB + 1 ? (io >> 16) != 0u : (v == start && ((pmo >> b) & 1ull) != 0ull);
        for (uint32_t k = e0 - done; k < e1 - done; ++k) {
          const int64_t x = (int64_t)pairs[k];
          lt += x < v && x >= start ? 1u : 0u;
          eq += x == v ? 1u : 0u;
          pres = pres || (x == v - 1 && x >= start);
        }
        const uint32_t Cb = nu - (io & 0xffffu) + (few ? 0u : (uint32_t)cum[64 * b + owner]) + lt;
        const EmCoef Eo = em_coef(as);
        TruncEnd to = {};
        if constexpr (kTruncLaw) to = trunc_end(Eo, K, ln);
        const double zv = survival(Eo, to, v);
        const double zv1 =
            pres ? survival(Eo, to, v - 1) : zv + pow_neg(as, ln_value(v, ln));
        const double t2 = fabs(fma(zv1, izo, -(double)(nu - Cb) * idn));
        const double t1 = fabs(fma(zv, izo, -(double)(nu - Cb - eq) * idn));
        __hip_atomic_fetch_max(&dmax[owner], (uint64_t)__double_as_longlong(fmax(t1, t2)),
                               __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
      }
    }
    wave_sync();
    done = next;
  }
  o.D = __longlong_as_double((long long)dmax[lane]);
  return o;
}

// The same under the truncated law, each lane by itself: its values above the
// column (few: they are rare under the planner's rule) sorted by rank.
static __device__ __noinline__ LaneOut lane_finish_trunc(const LdsU32* column, int64_t* slots_,
                                                         int myc, int od, int64_t n, uint32_t fl,
                                                         uint32_t K, bool want_fp,
                                                         const double* ln_) {
  int64_t* slots = as_global(slots_);
  const double* __restrict__ ln = as_global(ln_);
  LaneOut o;
  o.fp = 0;
  const int oc = myc + od;
  int64_t* more = slots + 64 * kLaneCap;
  auto ov = [&](int q) -> int64_t {
    return slots[(q < myc ? q : kLaneCap - od + (q - myc)) * 64];
  };
  U128 S = {0, 0};
  for (int i = 0; i < oc; ++i) {
    const int64_t v = ov(i);
    int rank = 0;  // values below it, plus equal ones stored before it
    for (int j = 0; j < oc; ++j) {
      const int64_t x = ov(j);
      rank += x < v || (x == v && j < i) ? 1 : 0;
    }
    more[rank * 64] = v;
    u128_add(S, ln_fixed(v, ln), 0);
    if (want_fp) o.fp += mix64((uint64_t)v);
  }
  for (int b = 0; b < kHLB / 2; ++b) {
    const uint32_t wv = column[b * 64];
#pragma unroll
    for (int half = 0; half < 2; ++half) {
      const uint32_t k = half ? (wv >> 16) : (wv & 0xffffu);
      const int64_t v = 2 * b + half + 1;
      u128_add_mul(S, k, ln_fixed(v, ln));
      if (want_fp) o.fp += (uint64_t)k * mix64((uint64_t)v);
    }
  }
  LaneSrc src{column, more, oc, 17, 0};
  finish_truncated(src, S, n, fl, ln, K, o.a, o.D, o.flags);
  return o;
}

// The whole tail draw of a deferred entry (called: rare, and long).
struct TailDraw {
  int64_t X;
  uint32_t fl;
};
static __device__ __noinline__ TailDraw tail_draw_call(double beta, double gm, uint32_t k0,
                                                       uint32_t k1, uint32_t i, uint32_t rep,
                                                       uint32_t stream) {
  TailDraw t;
  t.fl = 0;
  t.X = tail_draw(beta, gm, k0, k1, i, rep, stream, &t.fl);
  return t;
}

__device__ __forceinline__ void lds_inc(LdsU32* p) {
  __hip_atomic_fetch_add(p, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}
__device__ __forceinline__ void lds_add(LdsU32* p, uint32_t v) {
  __hip_atomic_fetch_add(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}
__device__ __forceinline__ void lds_or(LdsU32* p, uint32_t v) {
  __hip_atomic_fetch_or(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}
__device__ __forceinline__ int64_t uniform64(int64_t v) {
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)v);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(v >> 32));
  return (int64_t)(((uint64_t)hi << 32) | lo);
}
__device__ __forceinline__ uint32_t uniform32(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_readfirstlane((int)v);
}
// Full search of a deferred body draw in the staged tables.
__device__ __forceinline__ int lds_search(uint64_t m, const LdsU32* T, const LdsU32* guide,
                                          int sh) {
  const uint32_t g = guide[guide_index(m, sh)];
  int lo = (int)(g & 0xffffu) >> 2, hi = (int)((g >> 16) & (kDeferred - 1)) >> 2;
  while (lo < hi) {
    const int mid = (lo + hi) >> 1;
    if (threshold(T[mid], T[kH + mid]) >= m)
      hi = mid;
    else
      lo = mid + 1;
  }
  return lo + 1;
}

// The fast path of four draws in 32-bit steps: z is the offset 4 (x - 1) of a
// draw that it decides, else kDeferred or more: a draw to search in full (a
// wide bracket, a tail uniform, a first word that equals the threshold's or
// whose bin needs more bits).  A counter's place is then a minimum away, with
// no look at what a draw is; the loops look when the largest z says so.
constexpr uint32_t kNoDraw = 0xffffu;  // z of a draw that does not exist
__device__ __forceinline__ void fast_offsets(const uint32_t (&w0)[4], const uint32_t (&gg)[4],
                                             const uint32_t (&t)[4], const GuideRule& rule,
                                             uint32_t (&z)[4]) {
  const uint32_t wm = max(max(w0[0], w0[1]), max(w0[2], w0[3]));
  bool odd = wm > rule.last;
#pragma unroll
  for (int d = 0; d < 4; ++d) {
    z[d] = w0[d] < t[d] ? (gg[d] & 0xffffu) : (gg[d] >> 16);
    odd = odd || w0[d] == t[d];
  }
  if (__ballot(odd) != 0ull) {
#pragma unroll
    for (int d = 0; d < 4; ++d)
      if (w0[d] == t[d] || w0[d] > rule.last) z[d] = (uint32_t)kDeferred;
  }
}
__device__ __forceinline__ bool deferred(uint32_t z) {
  return z >= (uint32_t)kDeferred && z != kNoDraw;
}

// Draw blocks per iteration of the lane form's loop (two draws each).
constexpr int kLaneBlocks = 2;  // four draws per lane and iteration
static_assert(kLaneBlocks == 2, "the draw loop keeps four table reads in flight");

// The draws of replicates rep0 + lane, lane < count (called, so that the loop's
// registers are its own): fast-path draws go straight into the lane's column,
// deferred draws of all lanes wait in a ring (head qh, qn entries) and are
// resolved 64 at a time by whichever lane picks them up, into the owner's
// column or slots.  Values above the column take kLaneCap slots of the wave's
// scratch, slot s of lane l at spill[s * 64 + l]: the lane's own draws fill
// slots 0, 1, ... (the count returned), the resolved ones slots kLaneCap - 1,
// kLaneCap - 2, ... (counted in L.ovc; either may exceed the room).
static __device__ __noinline__ int lane_draws(const DevCell* cell, int64_t rep0_, int count_,
                                              LdsU32* region, int64_t* spill_, const LdsU32* T,
                                              const LdsU32* guide) {
  const int lane = lane_id();
  const DevCell& c = *as_global(reinterpret_cast<const DevCell*>(uniform64((int64_t)cell)));
  const uint32_t rep0 = uniform32((uint32_t)rep0_);
  const bool active = lane < count_;
  const bool idle = __builtin_amdgcn_readfirstlane(count_) < 64;
  int64_t* __restrict__ spill = as_global(reinterpret_cast<int64_t*>(uniform64((int64_t)spill_)));
  LdsU32* hist = region + lane;
  const uint32_t column = (uint32_t)(uintptr_t)hist;
  LdsU32* ring = region + offsetof(LaneRegion, ring) / 4;
  LdsU32* ovc = region + offsetof(LaneRegion, ovc) / 4;
  LdsU32* lfl = region + offsetof(LaneRegion, fl) / 4;
#pragma unroll
  for (int b = 0; b < kHLB / 2; ++b) hist[b * 64] = 0u;
  ovc[lane] = 0u;
  lfl[lane] = 0u;
  wave_sync();
  const uint32_t n32 = uniform32((uint32_t)c.n);  // lane form: n <= 65535
  const uint32_t nblk = (n32 + 1) >> 1;
  const uint32_t r = rep0 + (uint32_t)lane;
  const uint64_t timax = (uint64_t)uniform64((int64_t)table_int(c.tmax));
  const int sh = (int)uniform32(c.gsh);
  const uint32_t ck0 = uniform32(c.k0), ck1 = uniform32(c.k1), cs = uniform32(c.stream);
  const double beta = c.beta, gm = c.gm;
  uint32_t qh = 0, qn = 0;
  int myc = 0;  // the lane's own values above the column
  // The loop is software-pipelined: an iteration issues the guide reads of
  // its uniforms, generates the next iteration's uniforms while they are in
  // flight, issues the table reads, and computes the next guide indexes while
  // those are in flight (one extra block of uniforms is generated at the end).
  auto gen = [&](uint32_t j, uint32_t (&ho)[4]) {  // the uniforms' first words
    // the round keys are recomputed per block with scalar adds rather than
    // kept live across the loop (where they would be spilled)
    uint32_t k0 = ck0, k1 = ck1;
    asm volatile("" : "+s"(k0), "+s"(k1));
#pragma unroll
    for (int b = 0; b < kLaneBlocks; ++b) {
      const Words4 w = philox4x32_10(j + (uint32_t)b, r, cs, 0u, k0, k1);
      ho[2 * b] = w.w0;
      ho[2 * b + 1] = w.w2;
    }
  };
  const GuideRule rule = guide_rule(sh);
  uint32_t wh[4];
  int gi[4];  // their guide bins
  gen(0u, wh);
#pragma unroll
  for (int d = 0; d < 4; ++d) gi[d] = guide_index32(wh[d], rule);
  for (uint32_t j = 0;;) {
    uint32_t gg[4];
#pragma unroll
    for (int d = 0; d < 4; ++d) gg[d] = guide[gi[d]];
    uint32_t nh[4];
    gen(j + (uint32_t)kLaneBlocks, nh);
    asm volatile("" : "+v"(nh[0]), "+v"(nh[1]), "+v"(nh[2]), "+v"(nh[3]));  // made here
    uint32_t t[4];
#pragma unroll
    for (int d = 0; d < 4; ++d) t[d] = T[(gg[d] & 0xffffu) >> 2];
    __builtin_amdgcn_sched_barrier(0);  // the table reads issue before the index math
#pragma unroll
    for (int d = 0; d < 4; ++d) gi[d] = guide_index32(nh[d], rule);
    asm volatile("" : "+v"(gi[0]), "+v"(gi[1]), "+v"(gi[2]), "+v"(gi[3]));  // made here
    asm volatile("" : "+v"(t[0]), "+v"(t[1]), "+v"(t[2]), "+v"(t[3]));  // reads stay unconditional
    uint32_t z[4];
    fast_offsets(wh, gg, t, rule, z);
    if (2u * j + 4u > n32 || idle) {
#pragma unroll
      for (int d = 0; d < 4; ++d)
        if (!active || 2u * j + (uint32_t)d >= n32) z[d] = kNoDraw;
    }
#pragma unroll
    for (int d = 0; d < 4; ++d) {
      // own column, no branch: what is above 1..kHLB counts into the pad row
      const uint32_t v = min(z[d], 4u * (uint32_t)kHLB);
      uint32_t at;
      asm("v_lshl_add_u32 %0, %1, 5, %2" : "=v"(at) : "v"(v & ~7u), "v"(column));
      lds_add((LdsU32*)(uintptr_t)at, 1u << ((v << 2) & 31u));
    }
    if (__ballot(max(max(z[0], z[1]), max(z[2], z[3])) >= 4u * (uint32_t)kHLB) != 0ull) {
#pragma unroll
      for (int d = 0; d < 4; ++d) {
        // values above the column, into the lane's own slots
        if (z[d] >= 4u * (uint32_t)kHLB && z[d] < (uint32_t)kDeferred) {
          if (myc < kLaneCap) spill[myc * 64 + lane] = (int64_t)(z[d] >> 2) + 1;
          ++myc;
        }
        // deferred draws into the ring, by number and lane (their uniform is
        // drawn again when they are resolved)
        const uint64_t md = __ballot(deferred(z[d]));
        const uint32_t pos = place_below(md, qh + qn) & (uint32_t)(kRing - 1);
        if ((md >> lane) & 1ull) ring[pos] = (2u * j + (uint32_t)d) * 64u + (uint32_t)lane;
        qn += (uint32_t)__popcll(md);
      }
    }
    j += (uint32_t)kLaneBlocks;
    const bool more = j < nblk;
    while (qn >= 64u || (!more && qn != 0u)) {
      const uint32_t m = min(qn, 64u);
      wave_sync();
      if ((uint32_t)lane < m) {
        const uint32_t e = ring[(qh + (uint32_t)lane) & (uint32_t)(kRing - 1)];
        const uint32_t owner = e & 63u, i = e >> 6;
        const Words4 w = philox4x32_10(i >> 1, rep0 + owner, cs, 0u, ck0, ck1);
        const uint64_t mu = (i & 1u) ? m53(w.w2, w.w3) : m53(w.w0, w.w1);
        int64_t v;
        if (mu > timax) {
          const TailDraw td = tail_draw_call(beta, gm, ck0, ck1, i, rep0 + owner, cs);
          v = td.X;
          if (td.fl) lds_or(&lfl[owner], td.fl);
        } else {
          v = (int64_t)lds_search(mu, T, guide, sh);
        }
        if (v <= kHLB) {
          const uint32_t b = (uint32_t)v - 1u;
          lds_add(&region[(b >> 1) * 64 + owner], 1u << ((b & 1u) * 16u));
        } else {
          const uint32_t s = __hip_atomic_fetch_add(&ovc[owner], 1u, __ATOMIC_RELAXED,
                                                    __HIP_MEMORY_SCOPE_WORKGROUP);
          if (s < (uint32_t)kLaneCap)
            spill[(kLaneCap - 1 - (int)s) * 64 + (int)owner] = v;
        }
      }
      qh += m;
      qn -= m;
    }
    if (!more) break;
#pragma unroll
    for (int d = 0; d < 4; ++d) wh[d] = nh[d];
  }
  wave_sync_global();  // other lanes wrote to this lane's slots
  return myc;
}

__device__ __forceinline__ void lane_wave(const DevCell* cells, int32_t cell_id, int64_t rep0,
                                          int count, LaneRegion* L, int lane, const uint32_t* T,
                                          const uint32_t* guide, const double* __restrict__ ln,
                                          const Outputs& out, uint64_t* esc_list,
                                          uint32_t* esc_count, uint32_t esc_cap, uint32_t* err,
                                          int64_t* spill) {
  const DevCell& c = cells[cell_id];
  LdsU32* region = (LdsU32*)L->hist;
  int myc = lane_draws(&c, rep0, count, region, spill, (const LdsU32*)T, (const LdsU32*)guide);
  int od = (int)L->ovc[lane];
  const uint32_t fl = L->fl[lane];
  bool ok = lane < count;
  if (ok && myc + od > kLaneCap) {
    const uint32_t slot = atomicAdd(esc_count, 1u);
    if (slot < esc_cap)
      esc_list[slot] = ((uint64_t)(uint32_t)cell_id << 32) | (uint32_t)(rep0 + lane);
    else
      atomicOr(err, kErrEscOverflow);
    ok = false;
  }
  if (!ok) myc = od = 0;
  const bool want_fp = out.fp != nullptr;
  LaneOut o;
  if (c.K >= kTruncEmK) {
    o = lane_finish<true>(region, spill + lane, myc, od, ok, c.n, fl, c.K, want_fp, ln);
  } else if (c.K) {
    if (ok)
      o = lane_finish_trunc(region + lane, spill + lane, myc, od, c.n, fl, c.K, want_fp, ln);
  } else {
    o = lane_finish<false>(region, spill + lane, myc, od, ok, c.n, fl, 0u, want_fp, ln);
  }
  if (ok) write_outputs(out, c.out_off + rep0 + lane, o.D, o.a, o.flags, o.fp);
}

}  // namespace zpl

#include "zpl_batch.hpp"
#include "zpl_fit.hpp"

namespace zpl {

// ---------------------------------------------------------------------------
// Table build: T[k] = F(k; alpha) = 1 - zeta(alpha, k+1)/zeta(alpha), the
// CDF of eq. (1), for k = 1..kH; then the guide table and per-cell constants.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_table(const DevCell* __restrict__ cells,
                                              double* __restrict__ tables,
                                              const double* __restrict__ ln,
                                              uint32_t* __restrict__ zero, int n_zero) {
  // the first block also clears the simulation's counters (one launch fewer)
  if (blockIdx.x == 0 && blockIdx.y == 0)
    for (int i = (int)threadIdx.x; i < n_zero; i += (int)blockDim.x) zero[i] = 0u;
  const int cell = (int)blockIdx.y;
  const int k = (int)(blockIdx.x * blockDim.x + threadIdx.x) + 1;
  if (k > kH || cells[cell].K != 0u) return;
  const double a = cells[cell].alpha;
  double suf[17];
  const int64_t xmin = cells[cell].xmin;
  if (xmin > 1) {  // T[k-1] = F(xmin + k - 1) = 1 - zeta(a, xmin + k)/zeta(a, xmin)
    const EmCoef E = em_coef(a);
    survival_head_cut(E, ln, suf);
    // zeta(a, q), q >= 2 (static indices into suf: no scratch); above a
    // cutoff of 17 every value relative to xmin^-a (survival_rel)
    auto zq = [&](int64_t q) {
      double z = 0.0;
#pragma unroll
      for (int t = 1; t <= 16; ++t)
        if (q - 1 == t) z = suf[t];
      if (xmin > 17) return survival_rel(E, q - 1, xmin);
      return q <= 17 ? z : survival_next_cut(E, q - 1, ln);
    };
    tables[(size_t)cell * kH + (k - 1)] = 1.0 - zq(xmin + k) / zq(xmin);
    return;
  }
  survival_head(a, ln, suf);
  double zk = suf[16];
#pragma unroll
  for (int t = 1; t < 16; ++t)
    if (k == t) zk = suf[t];
  if (k > 16) zk = survival_next(a, (int64_t)k, ln);
  tables[(size_t)cell * kH + (k - 1)] = 1.0 - zk / suf[0];
}

// Table of the truncated law on 1..K (Sect. 1 with a finite upper limit):
// T[k] = F(k) = 1 - Z(k)/Z(0) with Z(t) = sum_{j=t+1..K} j^-a, and T[k] = 1
// for k >= K, so a uniform never reaches the tail sampler.  The terms are
// computed in parallel; one thread forms the suffix sums from K down, in
// the order of the definition.  One workgroup per cell (pure-law cells exit).
__global__ __launch_bounds__(1024) void k_table_trunc(const DevCell* __restrict__ cells,
                                                     double* __restrict__ tables,
                                                     const double* __restrict__ ln) {
  const int cell = (int)blockIdx.x;
  const uint32_t K = cells[cell].K;
  if (K == 0u) return;
  __shared__ double w[kH + 2];  // w[j] = j^-a; then w[t + 1] = Z(t)
  const double a = cells[cell].alpha;
  const int tid = (int)threadIdx.x;
  for (int j = tid + 1; j <= (int)K; j += (int)blockDim.x) w[j] = j == 1 ? 1.0 : pow_neg(a, ln[j]);
  __syncthreads();
  if (tid == 0) {
    double z = 0.0;  // Z(K) = 0
    for (int t = (int)K - 1; t >= 0; --t) {
      const double wt = w[t + 1];
      w[t + 2] = z;  // Z(t + 1)
      z += wt;       // Z(t)
    }
    w[1] = z;
  }
  __syncthreads();
  const double z0 = w[1];
  double* T = tables + (size_t)cell * kH;
  for (int k = tid + 1; k <= kH; k += (int)blockDim.x)
    T[k - 1] = k >= (int)K ? 1.0 : 1.0 - w[k + 1] / z0;
}

// Guide entry b: the smallest k that a uniform in bin b can map to.  Bins
// b < kGA hold U in [b/(2 kGA), (b+1)/(2 kGA)); the others hold U with
// e = 1 - U in one (octave, sub-bin) cell, i.e. U in (1 - e_hi, 1 - e_lo].
// Entry kGuide is the sentinel kH.
// Guide entry b: 1 + the first index k with floor(T[k] 2^53) >= the smallest
// m of bin b (kH when none), the smallest value a uniform of the bin maps to;
// the cell's layout from its table (guide_layout).
__global__ __launch_bounds__(256) void k_guide(DevCell* __restrict__ cells,
                                              const double* __restrict__ tables,
                                              uint16_t* __restrict__ guides) {
  const int cell = (int)blockIdx.y;
  const int b = (int)(blockIdx.x * blockDim.x + threadIdx.x);
  if (b > kGuide) return;
  const double* T = tables + (size_t)cell * kH;
  const int sh = guide_layout(T);
  int g = kH;
  if (b < kGuide) {
    const uint64_t mmin = guide_bin_min(b, sh);
    int lo = 0, hi = kH;
    while (lo < hi) {
      const int mid = (lo + hi) >> 1;
      if (table_int(T[mid]) >= mmin)
        hi = mid;
      else
        lo = mid + 1;
    }
    g = lo < kH ? lo + 1 : kH;
  }
  guides[(size_t)cell * (kGuide + 1) + b] = (uint16_t)g;
  if (b == 0) {
    DevCell& c = cells[cell];
    c.tmax = T[kH - 1];
    c.beta = c.alpha - 1.0;
    c.gm = tail_g(c.beta, (double)(c.xmin + kH));
    c.gsh = (uint32_t)sh;
  }
}

// ln k for k = 0..kH+1 (ln 0 unused, set to 0), then ln k 2^53 as integers.
__global__ void k_ln_table(double* ln) {
  const int k = (int)(blockIdx.x * blockDim.x + threadIdx.x);
  if (k > kH + 1) return;
  const double l = k == 0 ? 0.0 : log((double)k);
  ln[k] = l;
  reinterpret_cast<uint64_t*>(ln + kH + 2)[k] = (uint64_t)(l * 0x1p53);
}

// The MLE's start table.
__global__ __launch_bounds__(64) void k_mle_guess(const double* __restrict__ ln,
                                                  double* __restrict__ guess) {
  const int i = (int)(blockIdx.x * blockDim.x + threadIdx.x);
  if (i < kGuessN) mle_guess_entry(i, ln, guess + 2 * i);
}

__global__ void k_fill_u32(uint32_t* p, int n, uint32_t v) {
  const int i = (int)(blockIdx.x * blockDim.x + threadIdx.x);
  if (i < n) p[i] = v;
}

// ---------------------------------------------------------------------------
// Order statistics per cell: the element of rank k = floor(R num/den) in the
// ascending D values (the annex's index rule).  D >= 0, so comparing the FP64
// bit patterns as unsigned integers orders the values.  Up to kSelQ quantiles
// at a time, in three launches:
//   1. k_sel_bracket (a workgroup per cell): a sample of kSelSample values at
//      fixed positions; each quantile brackets the sample values 5 standard
//      deviations of the sample rank around its expected position.  Instead of
//      sorting the sample, a histogram of the 11 bits below the sample's common
//      high bits (with each bin's smallest and largest value) locates the bins
//      of those two ranks; the bracket [lo, hi] runs from the smallest value of
//      the lower bin to the largest of the upper (it contains the two sample
//      values, and is a single value when one value fills the bin);
//   2. k_sel_gather (many workgroups per cell, each a slice of D): counts the
//      values below each bracket and gathers the values inside it into global
//      scratch, through per-(cell, quantile) counters;
//   3. k_sel_finish (a workgroup per cell): the rank k - below is selected
//      exactly among the gathered values by radix selection (11-bit digits),
//      the quantiles side by side, each from registers when its gathered
//      values fit (kSelRegs per thread), else re-read from scratch per digit.
// If rank k falls outside its bracket, or the bracket overflows its scratch,
// the radix selection runs over all of D instead.  Both give the same element.
// ---------------------------------------------------------------------------
constexpr int kSelSample = 4096;
constexpr int kSelUnroll = 8;
constexpr int kSelRegs = 24;  // gathered values per thread of a quantile group held in registers
static_assert(kHW % 256 == 0, "sum_replicate reads 256 bins per step");

__device__ __forceinline__ uint32_t wave_incl_scan_u32(uint32_t v, int lane) {
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const uint32_t o = (uint32_t)__shfl_up((int)v, d, 64);
    if (lane >= d) v += o;
  }
  return v;
}

// The bin of a 2048-bin histogram that holds rank kk (0-based: the first bin
// whose running count exceeds kk), found by one whole wave.  `sum` is the
// lane's total of bins 32 lane .. 32 lane + 31 and `incl` the inclusive scan
// of those totals across the wave.  The lane owning the rank is found from a
// ballot; its 32 bins are then scanned across lanes 0..31 (one LDS read per
// lane instead of a walk of up to 32 dependent reads).  Returns the bin, and
// in rem the rank inside it, identical on every lane; -1 when kk is not below
// the histogram's total (then rem is kk).
__device__ __forceinline__ int rank_bin(const uint32_t* hist, uint32_t incl, uint32_t sum,
                                        int64_t kk, int lane, int64_t& rem,
                                        uint32_t* bin_count = nullptr) {
  rem = kk;
  const uint64_t hit = __ballot((int64_t)incl > kk);
  if (hit == 0ull) return -1;
  const int owner = __ffsll((long long)hit) - 1;
  const int64_t base = (int64_t)(uint32_t)__shfl((int)(incl - sum), owner, 64);
  const uint32_t h = lane < 32 ? hist[owner * 32 + lane] : 0u;
  const uint32_t s = wave_incl_scan_u32(h, lane);  // lanes 32..63 add zeros
  const uint64_t hit2 = __ballot(lane < 32 && base + (int64_t)s > kk);
  const int j = __ffsll((long long)hit2) - 1;
  rem = kk - base - (int64_t)(uint32_t)__shfl((int)(s - h), j, 64);
  if (bin_count) *bin_count = (uint32_t)__shfl((int)h, j, 64);
  return owner * 32 + j;
}

struct SelLds {
  struct {
    uint32_t hist[kSelQ][2048];  // one per quantile group; the block-wide select uses [0]
  } u;
  uint64_t prefix, mask;
  int64_t krem;
  uint64_t gprefix[kSelQ], gmask[kSelQ];
  int64_t gkrem[kSelQ];
  int gstate[kSelQ];  // per group: 0 digits to select, 1 a single value left, 2 done
};

// Exact radix selection (11-bit digits) of rank k of bits[0..R), block-wide.
// All values share the bits above `top` (the caller's bracket), which are
// given in `common`; digits of 11 bits run from bit `top` down to bit 0.
__device__ uint64_t radix_select(SelLds& L, const uint64_t* __restrict__ bits, int64_t R,
                                 int64_t k, int top, uint64_t common) {
  const int tid = (int)threadIdx.x, lane = tid & 63, wave = tid >> 6;
  if (tid == 0) {
    const uint64_t m = top >= 63 ? 0ull : (~0ull << (top + 1));
    L.prefix = common & m;
    L.mask = m;
    L.krem = k;
  }
  __syncthreads();
  for (int hi_bit = top; hi_bit >= 0; hi_bit -= 11) {
    const int width = hi_bit + 1 < 11 ? hi_bit + 1 : 11;
    const int sh = hi_bit + 1 - width;
    const uint32_t dm = (1u << width) - 1u;
    for (int b = tid; b < 2048; b += (int)blockDim.x) L.u.hist[0][b] = 0u;
    __syncthreads();
    const uint64_t pre = L.prefix, msk = L.mask;
    const int64_t nt = (int64_t)blockDim.x;
    for (int64_t i0 = 0; i0 < R; i0 += nt * kSelUnroll) {
      uint64_t bv[kSelUnroll];
#pragma unroll
      for (int u = 0; u < kSelUnroll; ++u) {
        const int64_t i = i0 + u * nt + tid;
        bv[u] = i < R ? bits[i] : 0ull;
      }
#pragma unroll
      for (int u = 0; u < kSelUnroll; ++u) {
        const int64_t i = i0 + u * nt + tid;
        if (i < R && (bv[u] & msk) == pre) atomicAdd(&L.u.hist[0][(bv[u] >> sh) & dm], 1u);
      }
    }
    __syncthreads();
    if (wave == 0) {
      uint32_t sum = 0;
      for (int t = 0; t < 32; ++t) sum += L.u.hist[0][lane * 32 + t];
      const uint32_t incl = wave_incl_scan_u32(sum, lane);
      int64_t kk;
      const int d = rank_bin(L.u.hist[0], incl, sum, L.krem, lane, kk);
      if (lane == 0 && d >= 0) {
        L.krem = kk;
        L.prefix = pre | ((uint64_t)d << sh);
        L.mask = msk | ((uint64_t)dm << sh);
      }
    }
    __syncthreads();
  }
  return L.prefix;
}

// radix_select for up to kSelQ quantiles at once: group g (threads
// 256g..256g+255 of the 1024-thread block) selects rank k[g] of its own
// array a[g][0..n[g]), whose values share the bits above top[g] with
// common[g]; groups with act[g] false idle.  Same digits, same result as
// radix_select, with the quantiles' passes running side by side.  When the
// bin holding the rank has a single value and digits remain, the next pass
// instead finds that value (the only one matching the prefix so far) and the
// group is done.  Every barrier is reached by the whole block: the loop runs
// until no group has a pass left, finished groups idling.
__device__ void radix_select_groups(SelLds& L, const uint64_t* const (&a)[kSelQ],
                                    const int64_t (&n)[kSelQ], const int64_t (&k)[kSelQ],
                                    const int (&top)[kSelQ], const uint64_t (&common)[kSelQ],
                                    const bool (&act)[kSelQ], uint64_t (&res)[kSelQ]) {
  static_assert(kSelQ * 256 == 1024, "one 256-thread group per quantile");
  const int tid = (int)threadIdx.x, g = tid >> 8, gt = tid & 255, lane = tid & 63;
  const bool scanner = ((tid >> 6) & 3) == 0;  // the group's first wave
  // this group's parameters (static indices: the arrays stay in registers)
  const uint64_t* src = nullptr;
  int64_t cnt = 0, kg = 0;
  int topg = 0;
  uint64_t comg = 0ull;
  bool actg = false;
  int maxtop = -1;
#pragma unroll
  for (int q = 0; q < kSelQ; ++q) {
    if (q == g) {
      src = a[q];
      cnt = n[q];
      kg = k[q];
      topg = top[q];
      comg = common[q];
      actg = act[q];
    }
    if (act[q] && top[q] > maxtop) maxtop = top[q];
  }
  if (gt == 0) {
    const uint64_t m = topg >= 63 ? 0ull : (~0ull << (topg + 1));
    L.gprefix[g] = comg & m;
    L.gmask[g] = m;
    L.gkrem[g] = kg;
    L.gstate[g] = actg ? 0 : 2;
  }
  // the group's values in registers when they fit (loaded once for all digits)
  const bool inreg = actg && cnt <= (int64_t)256 * kSelRegs;
  uint64_t rv[kSelRegs];
#pragma unroll
  for (int u = 0; u < kSelRegs; ++u) {
    const int64_t i = (int64_t)u * 256 + gt;
    rv[u] = inreg && i < cnt ? src[i] : 0ull;
  }
  __syncthreads();
  uint32_t* hist = L.u.hist[g];
  for (int p = 0; maxtop - 11 * p >= 0; ++p) {
    const int hb = topg - 11 * p;
    const int st = L.gstate[g];
    const bool on = actg && hb >= 0 && st == 0;
    const bool find = actg && st == 1;
    const int width = hb + 1 < 11 ? hb + 1 : 11;
    const int sh = hb + 1 - width;
    const uint32_t dm = on ? (1u << width) - 1u : 0u;
    if (on)
      for (int b = gt; b < 2048; b += 256) hist[b] = 0u;
    __syncthreads();
    if (on && inreg) {
      const uint64_t pre = L.gprefix[g], msk = L.gmask[g];
#pragma unroll
      for (int u = 0; u < kSelRegs; ++u) {
        const int64_t i = (int64_t)u * 256 + gt;
        if (i < cnt && (rv[u] & msk) == pre) atomicAdd(&hist[(rv[u] >> sh) & dm], 1u);
      }
    } else if (on) {
      const uint64_t pre = L.gprefix[g], msk = L.gmask[g];
      for (int64_t i0 = 0; i0 < cnt; i0 += 256 * kSelUnroll) {
        uint64_t bv[kSelUnroll];
#pragma unroll
        for (int u = 0; u < kSelUnroll; ++u) {
          const int64_t i = i0 + u * 256 + gt;
          bv[u] = i < cnt ? src[i] : 0ull;
        }
#pragma unroll
        for (int u = 0; u < kSelUnroll; ++u) {
          const int64_t i = i0 + u * 256 + gt;
          if (i < cnt && (bv[u] & msk) == pre) atomicAdd(&hist[(bv[u] >> sh) & dm], 1u);
        }
      }
    } else if (find) {  // exactly one value matches: it is the result
      const uint64_t pre = L.gprefix[g], msk = L.gmask[g];
      if (inreg) {
#pragma unroll
        for (int u = 0; u < kSelRegs; ++u) {
          const int64_t i = (int64_t)u * 256 + gt;
          if (i < cnt && (rv[u] & msk) == pre) L.gprefix[g] = rv[u];
        }
      } else {
        for (int64_t i = gt; i < cnt; i += 256) {
          const uint64_t v = src[i];
          if ((v & msk) == pre) L.gprefix[g] = v;
        }
      }
    }
    __syncthreads();
    if (on && scanner) {
      uint32_t sum = 0;
      for (int t = 0; t < 32; ++t) sum += hist[lane * 32 + t];
      const uint32_t incl = wave_incl_scan_u32(sum, lane);
      int64_t kk;
      uint32_t nbin = 0;
      const int d = rank_bin(hist, incl, sum, L.gkrem[g], lane, kk, &nbin);
      if (lane == 0 && d >= 0) {
        L.gkrem[g] = kk;
        L.gprefix[g] = L.gprefix[g] | ((uint64_t)d << sh);
        L.gmask[g] = L.gmask[g] | ((uint64_t)dm << sh);
        if (nbin == 1u && sh > 0) L.gstate[g] = 1;
      }
    }
    if (find && gt == 0) {
      L.gmask[g] = ~0ull;
      L.gstate[g] = 2;
    }
    __syncthreads();
    // another pass only while some group has digits or its single value left
    bool more = false;
#pragma unroll
    for (int q = 0; q < kSelQ; ++q)
      if (act[q] && (L.gstate[q] == 1 || (L.gstate[q] == 0 && top[q] - 11 * (p + 1) >= 0)))
        more = true;
    if (!more) break;
  }
#pragma unroll
  for (int q = 0; q < kSelQ; ++q) res[q] = L.gprefix[q];
  __syncthreads();
}

// Per (cell, quantile) state between the three launches.
struct SelMeta {
  uint64_t lo, hi;           // bracket (FP64 bit patterns)
  unsigned long long below;  // values below lo
  uint32_t nb;               // values gathered in [lo, hi]
  uint32_t pad;
};

__global__ __launch_bounds__(1024) void k_sel_bracket(const double* __restrict__ D,
                                                     const DevCell* __restrict__ cells, int q0,
                                                     int nq, const uint32_t* __restrict__ qnum,
                                                     const uint32_t* __restrict__ qden,
                                                     SelMeta* __restrict__ meta) {
  constexpr int kSpt = kSelSample / 1024;  // sample values per thread
  __shared__ uint32_t cnt[2048];
  __shared__ unsigned long long bmin[2048], bmax[2048];
  __shared__ uint64_t wor[16], wand[16];
  __shared__ int bin_of[2 * kSelQ];
  __shared__ int64_t rank_ab[2 * kSelQ];  // sample ranks a, b of each quantile
  __shared__ uint64_t sample[kSelSample];  // for the exact order statistics (rare case)
  __shared__ SelLds L;
  const int cell = (int)blockIdx.x;
  const int tid = (int)threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const DevCell c = cells[cell];
  const uint64_t* bits = reinterpret_cast<const uint64_t*>(D + c.out_off);
  const int64_t R = c.R;
  // sample ranks a = p - dl and b = p + dl of each quantile, as in the sorted
  // sample (published by the first barrier below)
  if (tid < nq) {
    const int64_t k = (int64_t)(((uint64_t)R * qnum[q0 + tid]) / qden[q0 + tid]);
    const double qf = (double)k / (double)R;
    const int64_t p = (int64_t)(qf * kSelSample);
    const int64_t dl = (int64_t)(5.0 * sqrt((double)kSelSample * qf * (1.0 - qf))) + 8;
    rank_ab[2 * tid] = p - dl;
    rank_ab[2 * tid + 1] = p + dl;
  }
  uint64_t x[kSpt];
  uint64_t o = 0ull, an = ~0ull;
#pragma unroll
  for (int t = 0; t < kSpt; ++t) {
    const uint64_t pos = (uint64_t)(tid + 1024 * t);
    x[t] = bits[(int64_t)((pos * (uint64_t)R) / kSelSample)];
    sample[pos] = x[t];
    o |= x[t];
    an &= x[t];
  }
#pragma unroll
  for (int m = 32; m > 0; m >>= 1) {
    o |= shfl_xor_u64(o, m);
    an &= shfl_xor_u64(an, m);
  }
  if (lane == 0) {
    wor[wave] = o;
    wand[wave] = an;
  }
  for (int b = tid; b < 2048; b += 1024) {
    cnt[b] = 0u;
    bmin[b] = ~0ull;
    bmax[b] = 0ull;
  }
  __syncthreads();
  o = 0ull;
  an = ~0ull;
#pragma unroll
  for (int w = 0; w < 16; ++w) {
    o |= wor[w];
    an &= wand[w];
  }
  // the sample's common high bits, then an 11-bit digit below them
  const uint64_t diff = o ^ an;
  const int top = diff ? 63 - __clzll((long long)diff) : 0;
  const int sh = top > 10 ? top - 10 : 0;
#pragma unroll
  for (int t = 0; t < kSpt; ++t) {
    const int d = (int)((x[t] >> sh) & 2047u);
    atomicAdd(&cnt[d], 1u);
    atomicMin(&bmin[d], (unsigned long long)x[t]);
    atomicMax(&bmax[d], (unsigned long long)x[t]);
  }
  __syncthreads();
  // the bin holding sample rank r is the first whose running count exceeds r
  if (wave == 0) {
    uint32_t sum = 0;
    for (int t = 0; t < 32; ++t) sum += cnt[lane * 32 + t];
    const uint32_t incl = wave_incl_scan_u32(sum, lane);
    for (int r = 0; r < 2 * nq; ++r) {
      int64_t rk = rank_ab[r];
      rk = rk < 0 ? 0 : (rk > kSelSample - 1 ? kSelSample - 1 : rk);
      int64_t kk;
      const int d = rank_bin(cnt, incl, sum, rk, lane, kk);  // the sample holds 4096 > rk
      if (lane == 0) bin_of[r] = d;
    }
  }
  __syncthreads();
  // The bracket holds [sample[a], sample[b]]: the smallest value of a's bin
  // and the largest of b's.  When both ranks fall in one bin that holds more
  // than one value, sample[a] and sample[b] themselves are selected (radix
  // selection over the sample), so that a value filling ranks a..b (an atom
  // of D) still gives lo = hi.
  for (int q = 0; q < nq; ++q) {
    const int64_t a = rank_ab[2 * q], b = rank_ab[2 * q + 1];
    const int ba = bin_of[2 * q], bb = bin_of[2 * q + 1];
    uint64_t lo = a <= 0 ? 0ull : (uint64_t)bmin[ba];
    uint64_t hi = b >= kSelSample - 1 ? ~0ull : (uint64_t)bmax[bb];
    if (a > 0 && b < kSelSample - 1 && ba == bb && bmin[ba] != bmax[ba]) {
      lo = radix_select(L, sample, kSelSample, a, 63, 0ull);
      hi = radix_select(L, sample, kSelSample, b, 63, 0ull);
    }
    if (tid == 0) {
      SelMeta m;
      m.lo = lo;
      m.hi = hi;
      m.below = 0ull;
      m.nb = 0u;
      m.pad = 0u;
      meta[(size_t)cell * kSelQ + q] = m;
    }
  }
}

// Slice `slice` of cell `cell` (blocks laid out cell-major, `slices` per
// cell): values below each bracket are counted, values inside are appended
// to the quantile's gather area.  Per step of 256 x kSelUnroll values the
// workgroup takes its slots with one atomic per quantile (a wave scan of the
// threads' counts, then the four waves' totals), not one per wave and value.
__global__ __launch_bounds__(256) void k_sel_gather(const double* __restrict__ D,
                                                   const DevCell* __restrict__ cells, int nq,
                                                   int slices, int64_t chunk,
                                                   SelMeta* __restrict__ meta,
                                                   uint64_t* __restrict__ gather, int64_t gcap) {
  __shared__ uint32_t wtot[4][kSelQ];   // per wave, in-bracket values of the step
  __shared__ uint32_t wbase[4][kSelQ];  // first slot of each wave's values
  const int cell = (int)(blockIdx.x / (unsigned)slices);
  const int slice = (int)(blockIdx.x % (unsigned)slices);
  const int tid = (int)threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const DevCell c = cells[cell];
  const int64_t R = c.R;
  const int64_t ib = (int64_t)slice * chunk;
  if (ib >= R) return;  // the whole block
  const int64_t ie = ib + chunk < R ? ib + chunk : R;
  const uint64_t* bits = reinterpret_cast<const uint64_t*>(D + c.out_off);
  SelMeta* M = meta + (size_t)cell * kSelQ;
  uint64_t* G = gather + (size_t)cell * kSelQ * gcap;
  uint64_t lo[kSelQ], hi[kSelQ];
  uint32_t below[kSelQ];
#pragma unroll
  for (int qq = 0; qq < kSelQ; ++qq) {
    lo[qq] = qq < nq ? M[qq].lo : 0ull;
    hi[qq] = qq < nq ? M[qq].hi : 0ull;
    below[qq] = 0u;
  }
  for (int64_t i0 = ib; i0 < ie; i0 += 256 * kSelUnroll) {
    uint64_t bv[kSelUnroll];
#pragma unroll
    for (int u = 0; u < kSelUnroll; ++u) {
      const int64_t i = i0 + u * 256 + tid;
      bv[u] = i < ie ? bits[i] : 0ull;
    }
    uint32_t inm[kSelQ], incl[kSelQ], cnt[kSelQ];
#pragma unroll
    for (int qq = 0; qq < kSelQ; ++qq) {
      inm[qq] = 0u;
      cnt[qq] = 0u;
#pragma unroll
      for (int u = 0; u < kSelUnroll; ++u) {
        const bool valid = i0 + u * 256 + tid < ie;
        const uint64_t b = bv[u];
        const bool bl = qq < nq && valid && b < lo[qq];
        const bool in = qq < nq && valid && !bl && b <= hi[qq];
        below[qq] += bl ? 1u : 0u;
        inm[qq] |= in ? (1u << u) : 0u;
        cnt[qq] += in ? 1u : 0u;
      }
      incl[qq] = wave_incl_scan_u32(cnt[qq], lane);
      if (lane == 63) wtot[wave][qq] = incl[qq];
    }
    __syncthreads();
    if (tid < kSelQ) {
      uint32_t t = 0;
#pragma unroll
      for (int w = 0; w < 4; ++w) {
        wbase[w][tid] = t;
        t += wtot[w][tid];
      }
      const uint32_t b = (tid < nq && t) ? atomicAdd(&M[tid].nb, t) : 0u;
#pragma unroll
      for (int w = 0; w < 4; ++w) wbase[w][tid] += b;
    }
    __syncthreads();
#pragma unroll
    for (int qq = 0; qq < kSelQ; ++qq) {
      if (inm[qq]) {
        uint32_t slot = wbase[wave][qq] + incl[qq] - cnt[qq];
#pragma unroll
        for (int u = 0; u < kSelUnroll; ++u) {
          if (inm[qq] & (1u << u)) {
            if ((int64_t)slot < gcap) G[qq * gcap + slot] = bv[u];
            ++slot;
          }
        }
      }
    }
    __syncthreads();  // wtot and wbase are reused by the next step
  }
  // values below each bracket: one atomic per workgroup and quantile (a cell's
  // counters share a cache line, which every workgroup of the cell updates)
#pragma unroll
  for (int qq = 0; qq < kSelQ; ++qq) {
    const uint32_t w = wave_sum_u32(below[qq]);
    if (lane == 0) wtot[wave][qq] = w;
  }
  __syncthreads();
  if (tid < nq) {
    uint32_t t = 0;
#pragma unroll
    for (int w = 0; w < 4; ++w) t += wtot[w][tid];
    if (t) atomicAdd(&M[tid].below, (unsigned long long)t);
  }
}

__global__ __launch_bounds__(1024) void k_sel_finish(const double* __restrict__ D,
                                                    const DevCell* __restrict__ cells, int q0,
                                                    int nq, int n_q,
                                                    const uint32_t* __restrict__ qnum,
                                                    const uint32_t* __restrict__ qden,
                                                    const SelMeta* __restrict__ meta,
                                                    double* __restrict__ qout,
                                                    uint64_t* __restrict__ gather, int64_t gcap) {
  __shared__ SelLds L;
  const int cell = (int)blockIdx.x;
  const int tid = (int)threadIdx.x;
  const DevCell c = cells[cell];
  const uint64_t* bits = reinterpret_cast<const uint64_t*>(D + c.out_off);
  const uint64_t* G = gather + (size_t)cell * kSelQ * gcap;
  const SelMeta* M = meta + (size_t)cell * kSelQ;
  const int64_t R = c.R;
  const uint64_t* arr[kSelQ];
  int64_t cnt[kSelQ], rk[kSelQ];
  int tops[kSelQ];
  uint64_t com[kSelQ], res[kSelQ];
  bool grp[kSelQ], full[kSelQ];
#pragma unroll
  for (int qq = 0; qq < kSelQ; ++qq) {
    arr[qq] = G + qq * gcap;
    cnt[qq] = 0;
    rk[qq] = 0;
    tops[qq] = 0;
    com[qq] = 0ull;
    res[qq] = 0ull;
    grp[qq] = false;
    full[qq] = false;
    if (qq < nq) {
      const int64_t k = (int64_t)(((uint64_t)R * qnum[q0 + qq]) / qden[q0 + qq]);
      const SelMeta m = M[qq];
      const int64_t lo_rank = (int64_t)m.below;
      const int64_t nin = (int64_t)m.nb;
      rk[qq] = k;
      if (k >= lo_rank && k < lo_rank + nin && m.lo == m.hi) {
        res[qq] = m.lo;  // every value in the bracket equals lo (an atom of D)
      } else if (k >= lo_rank && k < lo_rank + nin && nin <= gcap) {
        const uint64_t x = m.lo ^ m.hi;
        tops[qq] = x ? 63 - __clzll((long long)x) : 0;
        com[qq] = m.lo;
        cnt[qq] = nin;
        rk[qq] = k - lo_rank;
        grp[qq] = true;
      } else {
        full[qq] = true;
      }
    }
  }
  uint64_t gres[kSelQ];
  radix_select_groups(L, arr, cnt, rk, tops, com, grp, gres);
#pragma unroll
  for (int qq = 0; qq < kSelQ; ++qq) {
    if (grp[qq]) res[qq] = gres[qq];
    if (full[qq]) res[qq] = radix_select(L, bits, R, rk[qq], 63, 0ull);
  }
  if (tid == 0) {
#pragma unroll
    for (int qq = 0; qq < kSelQ; ++qq)
      if (qq < nq) qout[cell * n_q + q0 + qq] = __longlong_as_double((long long)res[qq]);
  }
}

// The same order statistics by one workgroup per cell, for cells of up to
// kSelCellMax values: up to kSelQ quantiles side by side narrow an interval of
// bit patterns around their rank, by histograms of 2,048 equal parts over all
// values (from the cache after the first pass), until at most kSelCand are
// left; those are gathered into LDS and narrowed there until a wave ranks the
// last 64.  Bound by latency (about a dozen barriers); two reads of D for
// values without ties.  10,000 values: 12 us, in three launches 37; 36 cells of
// 50,000 with many ties: 42 and 235.
constexpr int64_t kSelCellMax = 131072;
constexpr int kSelCand = 2048;
struct SelCellLds {
  uint32_t hist[kSelQ][2048];
  uint64_t cand[kSelQ][kSelCand];
  uint64_t lo[kSelQ], hi[kSelQ];  // the values lo..hi hold the rank
  unsigned long long least[kSelQ], most[kSelQ];  // found in a pass
  int64_t k[kSelQ];               // the rank among them
  uint32_t n[kSelQ];              // their number
  uint32_t fill[kSelQ];           // gathered
};
// The first histogram: 64 parts per octave from 2^-32 to 1, the ends open.
constexpr int kSelFirstShift = 46;
constexpr int64_t kSelFirstBase = (int64_t)(1023 - 32) << 6;

// Counts part b of each active lane; the lanes that agree with the first of
// them add theirs at once (with ties most do).
__device__ __forceinline__ void sel_count(uint32_t* hist, int b, int lane) {
  const int b0 = __builtin_amdgcn_readfirstlane(b);
  const uint64_t same = __ballot(b == b0);
  if (b != b0)
    atomicAdd(&hist[b], 1u);
  else if ((same & lanes_below(lane)) == 0ull)
    atomicAdd(&hist[b], (uint32_t)__popcll(same));
}
// The first active lane's value.
__device__ __forceinline__ uint64_t uniform_u64(uint64_t v) {
  return (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)v) |
         (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(v >> 32)) << 32;
}

// Shift that splits lo..hi into at most 2,048 parts.
__device__ __forceinline__ int sel_shift(uint64_t lo, uint64_t hi) {
  const int bits = 64 - __clzll((long long)(hi - lo));  // lo < hi
  return bits > 11 ? bits - 11 : 0;
}
// One wave: quantile q's interval becomes part b of its 2^sh wide ones.
__device__ __forceinline__ void sel_narrow(SelCellLds& L, int q, int sh, bool first, int lane) {
  uint32_t sum = 0;
  for (int t = 0; t < 32; ++t) sum += L.hist[first ? 0 : q][lane * 32 + t];
  const uint32_t incl = wave_incl_scan_u32(sum, lane);
  int64_t k;
  uint32_t n = 0;
  const int b = rank_bin(L.hist[first ? 0 : q], incl, sum, L.k[q], lane, k, &n);
  if (lane == 0 && b >= 0) {
    if (first) {
      L.lo[q] = b == 0 ? 0ull : (uint64_t)(kSelFirstBase + b) << kSelFirstShift;
      L.hi[q] = b == 2047 ? ~0ull : ((uint64_t)(kSelFirstBase + b + 1) << kSelFirstShift) - 1ull;
    } else {
      const uint64_t lo = L.lo[q] + ((uint64_t)b << sh), end = lo + ((1ull << sh) - 1ull);
      L.lo[q] = lo;
      if (end < L.hi[q]) L.hi[q] = end;
    }
    L.k[q] = k;
    L.n[q] = n;
  }
}

__global__ __launch_bounds__(1024) void k_sel_cell(const double* __restrict__ D,
                                                  const DevCell* __restrict__ cells, int q0,
                                                  int nq, int n_q,
                                                  const uint32_t* __restrict__ qnum,
                                                  const uint32_t* __restrict__ qden,
                                                  double* __restrict__ qout) {
  __shared__ SelCellLds L;
  const int cell = (int)blockIdx.x;
  const int tid = (int)threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const uint64_t* bits = reinterpret_cast<const uint64_t*>(D + cells[cell].out_off);
  const int R = (int)cells[cell].R;
  if (tid < kSelQ) {
    L.lo[tid] = 0ull;
    L.hi[tid] = tid < nq ? ~0ull : 0ull;
    L.k[tid] = tid < nq ? (int64_t)(((uint64_t)R * qnum[q0 + tid]) / qden[q0 + tid]) : 0;
    L.n[tid] = tid < nq ? (uint32_t)R : 0u;
    L.fill[tid] = 0u;
  }
  auto each = [&](auto fn) {  // fn of every value, eight loads in flight
    constexpr int kUnroll = 8;
    int i = tid;
    for (; i + (kUnroll - 1) * 1024 < R; i += kUnroll * 1024) {
      uint64_t v[kUnroll];
#pragma unroll
      for (int u = 0; u < kUnroll; ++u) v[u] = bits[i + u * 1024];
#pragma unroll
      for (int u = 0; u < kUnroll; ++u) fn(v[u]);
    }
    for (; i < R; i += 1024) fn(bits[i]);
  };
  uint64_t lo[kSelQ], hi[kSelQ];
  bool on[kSelQ];
  for (bool first = true;; first = false) {
    for (int b = tid; b < kSelQ * 2048; b += 1024) L.hist[0][b] = 0u;
    if (tid < kSelQ) {
      L.least[tid] = ~0ull;
      L.most[tid] = 0ull;
    }
    __syncthreads();
    int sh[kSelQ];
    bool any = false;
#pragma unroll
    for (int q = 0; q < kSelQ; ++q) {
      lo[q] = L.lo[q];
      hi[q] = L.hi[q];
      on[q] = L.n[q] > (uint32_t)kSelCand && lo[q] < hi[q];
      sh[q] = lo[q] < hi[q] ? sel_shift(lo[q], hi[q]) : 0;
      any = any || on[q];
    }
    if (!any) break;
    if (first) {
      each([&](uint64_t v) {
        int64_t b = (int64_t)(v >> kSelFirstShift) - kSelFirstBase;
        sel_count(L.hist[0], b < 0 ? 0 : (b > 2047 ? 2047 : (int)b), lane);
      });
    } else {
      // an interval whose values are all equal (ties) is a result
      uint64_t mn[kSelQ], mx[kSelQ];
#pragma unroll
      for (int q = 0; q < kSelQ; ++q) {
        mn[q] = ~0ull;
        mx[q] = 0ull;
      }
      each([&](uint64_t v) {
#pragma unroll
        for (int q = 0; q < kSelQ; ++q)
          if (on[q] && v >= lo[q] && v <= hi[q]) {
            mn[q] = v < mn[q] ? v : mn[q];
            mx[q] = v > mx[q] ? v : mx[q];
            sel_count(L.hist[q], (int)((v - lo[q]) >> sh[q]), lane);
          }
      });
#pragma unroll
      for (int q = 0; q < kSelQ; ++q)
        if (mx[q] >= mn[q]) {
          const bool odd = mn[q] != uniform_u64(mn[q]) || mx[q] != uniform_u64(mx[q]);
          const uint64_t here = __ballot(true);
          if (__ballot(odd) != 0ull || (here & lanes_below(lane)) == 0ull) {
            atomicMin(&L.least[q], (unsigned long long)mn[q]);
            atomicMax(&L.most[q], (unsigned long long)mx[q]);
          }
        }
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < kSelQ; ++q)
      if (wave == q && on[q]) {
        sel_narrow(L, q, sh[q], first, lane);
        if (lane == 0 && L.least[q] == L.most[q]) L.lo[q] = L.hi[q] = L.least[q];
      }
    __syncthreads();
  }
  // at most kSelCand values (or copies of one) are left of each quantile
#pragma unroll
  for (int q = 0; q < kSelQ; ++q) on[q] = lo[q] < hi[q];
  each([&](uint64_t v) {
#pragma unroll
    for (int q = 0; q < kSelQ; ++q)
      if (on[q] && v >= lo[q] && v <= hi[q]) L.cand[q][atomicAdd(&L.fill[q], 1u)] = v;
  });
  __syncthreads();
  // 256 threads per quantile from here on
  const int q = wave >> 2, t = tid & 255;
  for (;;) {
    const uint64_t l = L.lo[q], h = L.hi[q];
    const bool more = L.n[q] > 64u && l < h;
    if (!__syncthreads_or(more ? 1 : 0)) break;
    const int sh = l < h ? sel_shift(l, h) : 0;
    const int m = (int)L.fill[q];
    for (int b = t; b < 2048; b += 256) L.hist[q][b] = 0u;
    __syncthreads();
    if (more)
      for (int i = t; i < m; i += 256) {
        const uint64_t v = L.cand[q][i];
        if (v >= l && v <= h) atomicAdd(&L.hist[q][(v - l) >> sh], 1u);
      }
    __syncthreads();
    if (more && (wave & 3) == 0) sel_narrow(L, q, sh, false, lane);
    __syncthreads();
  }
  if ((wave & 3) != 0 || q >= nq) return;
  const uint64_t l = L.lo[q], h = L.hi[q];
  uint64_t result = l;
  if (l < h) {  // at most 64 values: rank them
    uint64_t* list = reinterpret_cast<uint64_t*>(L.hist[q]);
    const int m = (int)L.fill[q];
    int n = 0;
    for (int i0 = 0; i0 < m; i0 += 64) {
      const int i = i0 + lane;
      const uint64_t v = i < m ? L.cand[q][i] : 0ull;
      const bool in = i < m && v >= l && v <= h;
      const uint64_t mask = __ballot(in);
      if (in) list[n + __popcll(mask & lanes_below(lane))] = v;
      n += __popcll(mask);
    }
    wave_sync();
    const uint64_t v = lane < n ? list[lane] : 0ull;
    int64_t less = 0, same = 0;
    for (int j = 0; j < n; ++j) {
      const uint64_t x = list[j];
      less += x < v ? 1 : 0;
      same += x == v ? 1 : 0;
    }
    const int64_t k = L.k[q];
    const uint64_t hit = __ballot(lane < n && less <= k && k < less + same);
    const int src = hit ? __ffsll((long long)hit) - 1 : 0;
    result = (uint64_t)(uint32_t)__shfl((int)(uint32_t)v, src, 64) |
             (uint64_t)(uint32_t)__shfl((int)(uint32_t)(v >> 32), src, 64) << 32;
  }
  if (lane == 0) qout[cell * n_q + q0 + q] = __longlong_as_double((long long)result);
}

// count of D_b >= D_obs over the bootstrap replicates.
__global__ __launch_bounds__(256) void k_count_ge(const double* __restrict__ Db, int64_t B,
                                                 const double* __restrict__ Dobs,
                                                 unsigned long long* __restrict__ count) {
  const double d = *Dobs;
  uint32_t local = 0;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < B;
       i += (int64_t)gridDim.x * blockDim.x)
    local += (Db[i] >= d) ? 1u : 0u;
  local = wave_sum_u32(local);
  if ((threadIdx.x & 63u) == 0u && local) atomicAdd(count, (unsigned long long)local);
}

// Per cell c: count of D[out_off + b] >= dobs[c], b < R (batched bootstrap).
__global__ __launch_bounds__(256) void k_count_cells(const double* __restrict__ D,
                                                    const DevCell* __restrict__ cells,
                                                    const double* __restrict__ dobs,
                                                    unsigned long long* __restrict__ counts) {
  const int cell = (int)blockIdx.y;
  const DevCell c = cells[cell];
  const double d = dobs[cell];
  uint32_t local = 0;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < c.R;
       i += (int64_t)gridDim.x * blockDim.x)
    local += (D[c.out_off + i] >= d) ? 1u : 0u;
  local = wave_sum_u32(local);
  if ((threadIdx.x & 63u) == 0u && local) atomicAdd(&counts[cell], (unsigned long long)local);
}

// Raw draws of replicates rep_lo.. in draw order (parity checks of the
// sampler), by the steps of the simulation: the fast path of four draws from
// their first words, the search in the staged tables, and a tail proposal at a
// time.  A thread takes four draws of a replicate.
__global__ __launch_bounds__(256) void k_draws(const DevCell* __restrict__ cells,
                                              const double* __restrict__ tables,
                                              const uint16_t* __restrict__ guides,
                                              int64_t rep_lo, int64_t count,
                                              int64_t* __restrict__ x,
                                              uint32_t* __restrict__ flags) {
  __shared__ uint32_t T[2 * kH];
  __shared__ uint32_t guide[kGuide];
  const DevCell c = cells[0];
  load_cell_tables(T, guide, tables, guides, c, (int)threadIdx.x, 256);
  __syncthreads();
  const uint64_t timax = table_int(c.tmax);
  const int sh = (int)c.gsh;
  const GuideRule rule = guide_rule(sh);
  const int64_t off = c.xmin - 1, quads = (c.n + 3) / 4, total = count * quads;
  for (int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; t < total;
       t += (int64_t)gridDim.x * blockDim.x) {
    const int64_t rr = t / quads;
    const uint32_t i0 = 4u * (uint32_t)(t - rr * quads);
    const uint32_t rep = (uint32_t)(rep_lo + rr);
    Words4 w[2];
    uint32_t wh[4], gg[4], th[4], z[4];
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      w[b] = philox4x32_10((i0 >> 1) + (uint32_t)b, rep, c.stream, 0u, c.k0, c.k1);
      wh[2 * b] = w[b].w0;
      wh[2 * b + 1] = w[b].w2;
    }
#pragma unroll
    for (int d = 0; d < 4; ++d) {
      gg[d] = guide[guide_index32(wh[d], rule)];
      th[d] = T[(gg[d] & 0xffffu) >> 2];
    }
    fast_offsets(wh, gg, th, rule, z);
    uint32_t fl = 0;
#pragma unroll
    for (int d = 0; d < 4; ++d) {
      const uint32_t i = i0 + (uint32_t)d;
      if ((int64_t)i >= c.n) continue;
      int64_t v = off + (int64_t)(z[d] >> 2) + 1;
      if (deferred(z[d])) {
        const Words4& p = w[d >> 1];
        const uint64_t m = (d & 1) ? m53(p.w2, p.w3) : m53(p.w0, p.w1);
        if (m <= timax) {
          v = off + lds_search(m, (const LdsU32*)T, (const LdsU32*)guide, sh);
        } else {
          const double m0 = (double)(c.xmin + kH);
          TailTry y{0, kTailFirst};
          for (uint32_t attempt = 0; y.code != kTailTaken; ++attempt) {
            y = tail_try(m0, c.beta, c.gm, c.k0, c.k1, i, rep, c.stream, attempt);
            if (y.code == kTailHard)
              y = tail_hard(m0, c.beta, c.gm, c.k0, c.k1, i, rep, c.stream, attempt);
            if (y.code == kTailCapped) fl |= kFlagTailCapped;
          }
          v = y.X;
        }
      }
      x[rr * c.n + i] = v;
    }
    if (fl) atomicOr(&flags[rr], fl);
  }
}

}  // namespace zpl

// ---------------------------------------------------------------------------
// Host-side launchers (called by the runtime in zpl_api.cpp).
// ---------------------------------------------------------------------------
namespace zpl {

hipError_t launch_ln_table(double* ln, hipStream_t s) {
  k_ln_table<<<(kH + 2 + 255) / 256, 256, 0, s>>>(ln);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  k_mle_guess<<<(kGuessN + 63) / 64, 64, 0, s>>>(ln, ln + 2 * (kH + 2));
  return hipGetLastError();
}

hipError_t launch_fill_u32(uint32_t* p, int n, uint32_t v, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  k_fill_u32<<<(n + 255) / 256, 256, 0, s>>>(p, n, v);
  return hipGetLastError();
}

hipError_t launch_tables(DevCell* cells, int n_cells, double* tables, uint16_t* guides,
                         const double* ln, hipStream_t s, bool any_trunc, uint32_t* zero,
                         int n_zero) {
  if (n_cells <= 0) return hipSuccess;
  k_table<<<dim3(kH / 256, n_cells), 256, 0, s>>>(cells, tables, ln, zero, n_zero);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  if (any_trunc) {
    k_table_trunc<<<n_cells, 1024, 0, s>>>(cells, tables, ln);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  k_guide<<<dim3((kGuide + 1 + 255) / 256, n_cells), 256, 0, s>>>(cells, tables, guides);
  return hipGetLastError();
}

static_assert(sizeof(WaveSlot) == kWaveSlotBytes, "WaveSlot layout");

hipError_t launch_simulate(const SimGrid& g, const DevCell* cells, const double* tables,
                           const uint16_t* guides, const double* ln, const Unit* lane_units,
                           int n_lane, const Unit* batch_units, int n_batch, uint32_t* lane_queue,
                           uint32_t* batch_queue, uint32_t* big_queue, Outputs out,
                           uint64_t* esc_list, uint32_t* esc_count, uint32_t esc_cap,
                           int64_t* scratch, uint32_t* err, hipStream_t s) {
  if (g.grid <= 0) return hipSuccess;
  k_simulate<<<g.grid, kBlock, 0, s>>>(g, cells, tables, guides, ln, lane_units, n_lane,
                                       batch_units, n_batch, lane_queue, batch_queue, big_queue,
                                       out, esc_list, esc_count, esc_cap, scratch, err);
  return hipGetLastError();
}

hipError_t launch_escalated(int grid, const DevCell* cells, const double* tables,
                            const uint16_t* guides, const double* ln, uint32_t* queue, Outputs out,
                            uint64_t* esc_list, uint32_t* esc_count, uint32_t esc_cap,
                            int64_t* scratch, int waves, int64_t stride, uint32_t* err,
                            hipStream_t s) {
  if (grid <= 0) return hipSuccess;
  k_escalated<<<grid, 64 * kEscWaves, 0, s>>>(cells, tables, guides, ln, queue, out, esc_list,
                                              esc_count, esc_cap, scratch, waves, stride, err);
  return hipGetLastError();
}

hipError_t launch_cutoff(int grid, const DevCell* cells, const double* tables,
                         const uint16_t* guides, const double* ln, const Unit* units, int n_units,
                         uint32_t* queue, Outputs out, uint64_t* esc_list, uint32_t* esc_count,
                         uint32_t esc_cap, int64_t* scratch, int waves, int64_t stride,
                         uint32_t* err, hipStream_t s) {
  if (n_units <= 0 || grid <= 0) return hipSuccess;
  k_cutoff<<<grid, 64 * kBatchWavesCut, 0, s>>>(cells, tables, guides, ln, units, n_units, queue,
                                                out, esc_list, esc_count, esc_cap, scratch, waves,
                                                stride, err);
  return hipGetLastError();
}

hipError_t launch_fit(int grid, const int64_t* const* xs, const int64_t* ns, int n_sets,
                      const double* ln, int64_t* scratch, int64_t stride, double* ahat,
                      double* D, uint32_t* flags, uint32_t* status, hipStream_t s) {
  if (n_sets <= 0) return hipSuccess;
  k_fit_block<false><<<grid, kFitThreads, 0, s>>>(xs, ns, n_sets, nullptr, 0, ln, scratch, stride,
                                                  ahat, D, flags, status, 0u);
  return hipGetLastError();
}

// Counts and sorts a dataset into fit_view(scratch, n, *groups).
static hipError_t launch_fit_prepare(const int64_t* x, int64_t n, uint32_t K, const double* ln,
                                     int64_t* scratch, int* groups, hipStream_t s) {
  if (n < kFitGridMin) {
    *groups = 0;
    k_fit_block<true><<<1, kFitThreads, 0, s>>>(nullptr, nullptr, 1, x, n, ln, scratch, 0, nullptr,
                                                nullptr, nullptr, nullptr, K);
    return hipGetLastError();
  }
  int64_t g = n / kFitChunkMin;
  if (g > kFitGroups) g = kFitGroups;
  const int64_t chunk = (n + g - 1) / g;
  g = (n + chunk - 1) / chunk;
  *groups = (int)g;
  k_fit_count<<<(int)g, kFitCountThreads, 0, s>>>(x, n, chunk, K, ln, scratch);
  const int64_t runs = (n + kFitRun - 1) / kFitRun;
  const int most = runs < kFitGroups ? (int)runs : kFitGroups;
  k_fit_merge<<<most < kFitBins / 64 ? kFitBins / 64 : most, kFitThreads, 0, s>>>(n, chunk, (int)g,
                                                                                 scratch);
  int pass = 0;
  if (K == 0u)  // (up to K <= kFitBins every value has its bin)
    for (int64_t run = kFitRun; run < n; run *= kFitFan)
      k_fit_runs<<<most, 256, 0, s>>>(n, (int)g, run, pass++, scratch);
  return hipGetLastError();
}

hipError_t launch_fit_one(const int64_t* x, int64_t n, const double* ln, int64_t* scratch,
                          double* ahat, double* D, uint32_t* flags, uint32_t* status, uint32_t K,
                          hipStream_t s) {
  if (n < kFitGridMin) {
    k_fit_block<false><<<1, kFitThreads, 0, s>>>(nullptr, nullptr, 1, x, n, ln, scratch, 0, ahat, D,
                                                 flags, status, K);
    return hipGetLastError();
  }
  int groups = 0;
  const hipError_t e = launch_fit_prepare(x, n, K, ln, scratch, &groups, s);
  if (e != hipSuccess) return e;
  k_fit_cand<false><<<kFitShares, kFitCandThreads, 0, s>>>(nullptr, n, groups, scratch, nullptr,
                                                           kFitShares, K, ln, ahat, D, nullptr,
                                                           flags, status);
  return hipGetLastError();
}

// Scratch of the allocation-free fit (a dataset's larger values and counts,
// fit_view), one copy per GPU for the life of the
// process.  Host code never passes this name to a kernel: it stands for the
// host-side shadow; the device address comes from noalloc_scratch_address.
static __device__ __align__(256) int64_t zpl_noalloc_scratch[kNoAllocStride];

hipError_t noalloc_scratch_address(int64_t** p) {
  return hipGetSymbolAddress((void**)p, HIP_SYMBOL(zpl_noalloc_scratch));
}

hipError_t launch_fit_scan(const int64_t* x, int64_t n, const int64_t* xmins, int n_cand,
                           const double* ln, int64_t* scratch, double* ahat, double* D,
                           int64_t* ntail, uint32_t* flags, uint32_t* status, hipStream_t s) {
  if (n_cand <= 0) return hipSuccess;
  if (n <= kFitSmall && n_cand <= kFitAlone) {
    k_fit_cand<true><<<n_cand, kFitThreads, 0, s>>>(x, n, 0, scratch, xmins, 1, 0u, ln, ahat, D,
                                                        ntail, flags, status);
    return hipGetLastError();
  }
  int groups = 0;
  const hipError_t e = launch_fit_prepare(x, n, 0u, ln, scratch, &groups, s);
  if (e != hipSuccess) return e;
  // few candidates: several workgroups share a distance (about one per compute
  // unit in all; a small dataset has no more to share than a few of them take)
  const int most = n < kFitGridMin ? 8 : kFitShares;
  int wgs = n_cand <= kFitAcc ? 256 / n_cand : 1;
  if (wgs > most) wgs = most;
  k_fit_cand<false><<<n_cand * wgs, kFitCandThreads, 0, s>>>(nullptr, n, groups, scratch, xmins, wgs,
                                                             0u, ln, ahat, D, ntail, flags, status);
  return hipGetLastError();
}

hipError_t launch_select(const double* D, const DevCell* cells, int n_cells, int n_q,
                         const uint32_t* qnum, const uint32_t* qden, double* qout,
                         uint64_t* gather, int64_t gcap, int64_t maxR, int n_cu, hipStream_t s) {
  if (n_cells <= 0 || n_q <= 0) return hipSuccess;
  // the per-(cell, quantile) state follows the gather areas
  SelMeta* meta = reinterpret_cast<SelMeta*>(gather + (size_t)n_cells * kSelQ * gcap);
  // slices of at least 2,048 values, about two workgroups per compute unit
  const int64_t unit = 256 * kSelUnroll;
  int64_t slices = (2 * (int64_t)n_cu + n_cells - 1) / n_cells;
  const int64_t most = (maxR + unit - 1) / unit;
  if (slices > most) slices = most;
  if (slices < 1) slices = 1;
  int64_t chunk = (maxR + slices - 1) / slices;
  chunk = (chunk + unit - 1) / unit * unit;
  for (int q0 = 0; q0 < n_q; q0 += kSelQ) {
    const int nq = (n_q - q0) < kSelQ ? (n_q - q0) : kSelQ;
    if (maxR <= kSelCellMax) {
      k_sel_cell<<<n_cells, 1024, 0, s>>>(D, cells, q0, nq, n_q, qnum, qden, qout);
      const hipError_t e = hipGetLastError();
      if (e != hipSuccess) return e;
      continue;
    }
    k_sel_bracket<<<n_cells, 1024, 0, s>>>(D, cells, q0, nq, qnum, qden, meta);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    k_sel_gather<<<(unsigned)(n_cells * slices), 256, 0, s>>>(D, cells, nq, (int)slices, chunk,
                                                              meta, gather, gcap);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    k_sel_finish<<<n_cells, 1024, 0, s>>>(D, cells, q0, nq, n_q, qnum, qden, meta, qout, gather,
                                          gcap);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

hipError_t launch_count_ge(const double* Db, int64_t B, const double* Dobs,
                           unsigned long long* count, hipStream_t s) {
  int grid = (int)((B + 255) / 256);
  if (grid > 1024) grid = 1024;
  if (grid < 1) grid = 1;
  k_count_ge<<<grid, 256, 0, s>>>(Db, B, Dobs, count);
  return hipGetLastError();
}

hipError_t launch_count_cells(const double* D, const DevCell* cells, int n_cells,
                              const double* dobs, unsigned long long* counts, int64_t maxR,
                              hipStream_t s) {
  if (n_cells <= 0) return hipSuccess;
  int gx = (int)((maxR + 255) / 256);
  if (gx > 64) gx = 64;
  if (gx < 1) gx = 1;
  k_count_cells<<<dim3(gx, n_cells), 256, 0, s>>>(D, cells, dobs, counts);
  return hipGetLastError();
}

hipError_t launch_draws(const DevCell* cell, const double* table, const uint16_t* guide,
                        int64_t rep_lo, int64_t count, int64_t* x, uint32_t* flags,
                        int64_t total, hipStream_t s) {
  if (total <= 0) return hipSuccess;
  int64_t g = (total + 1023) / 1024;  // four draws a thread
  int grid = (int)(g > 4096 ? 4096 : g);
  k_draws<<<grid, 256, 0, s>>>(cell, table, guide, rep_lo, count, x, flags);
  return hipGetLastError();
}

}  // namespace zpl
