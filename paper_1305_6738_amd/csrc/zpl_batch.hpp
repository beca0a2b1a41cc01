// zpl_batch.hpp -- replicates by whole waves in batches, without sorting.
//
// A wave draws a batch of replicates one after another.  Of each it keeps the
// exact sum of logarithms, the counts of the first 1,024 support values and
// the larger draws unsorted.  The MLE of the batch then runs one replicate
// per lane, and the KS distance (eq. 3) one replicate per wave, by bounds:
// between two points l < r of the support every |F - S_n| is at most
// max(F(r) - S_n(l), S_n(r) - F(l)), so an interval whose bound does not reach
// a distance already found elsewhere holds no maximum and its values are not
// looked at.  What remains is evaluated by the same expressions as everywhere
// (hence the same D bit for bit).
//
// Included by zpl_kernels.hip after the helpers it uses.
#pragma once

namespace zpl {

// Sums, maxima and scans over the wave by DPP lane moves, which stay in the
// vector ALU: a step takes its few issue cycles, where a shuffle through the
// LDS crossbar takes over a hundred (a wave's six-step sum measured about
// 0.35 us so, and a replicate's fit takes about ten of them).  Steps 1..8
// shift within rows of 16 lanes, the two broadcasts carry a row's last lane to
// the next row and the lower half's to the upper: an inclusive scan, lane 63
// holding the total.  Lanes without a source take 0, so 0 must be the
// operation's identity.  Every lane of the wave must be active.
template <int kCtrl, int kRows>
__device__ __forceinline__ uint32_t dpp0_u32(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, kCtrl, kRows, 0xf, false);
}
template <int kCtrl, int kRows>
__device__ __forceinline__ uint64_t dpp0_u64(uint64_t v) {
  return ((uint64_t)dpp0_u32<kCtrl, kRows>((uint32_t)(v >> 32)) << 32) |
         dpp0_u32<kCtrl, kRows>((uint32_t)v);
}
template <class T, class Op>
__device__ __forceinline__ T dpp_scan(T v, Op op) {
  if constexpr (sizeof(T) == 4) {
    v = op(v, dpp0_u32<0x111, 0xf>(v));
    v = op(v, dpp0_u32<0x112, 0xf>(v));
    v = op(v, dpp0_u32<0x114, 0xf>(v));
    v = op(v, dpp0_u32<0x118, 0xf>(v));
    v = op(v, dpp0_u32<0x142, 0xa>(v));
    v = op(v, dpp0_u32<0x143, 0xc>(v));
  } else {
    v = op(v, dpp0_u64<0x111, 0xf>(v));
    v = op(v, dpp0_u64<0x112, 0xf>(v));
    v = op(v, dpp0_u64<0x114, 0xf>(v));
    v = op(v, dpp0_u64<0x118, 0xf>(v));
    v = op(v, dpp0_u64<0x142, 0xa>(v));
    v = op(v, dpp0_u64<0x143, 0xc>(v));
  }
  return v;
}
__device__ __forceinline__ uint32_t lane63_u32(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_readlane((int)v, 63);
}
__device__ __forceinline__ uint64_t lane63_u64(uint64_t v) {
  return ((uint64_t)lane63_u32((uint32_t)(v >> 32)) << 32) | lane63_u32((uint32_t)v);
}
__device__ __forceinline__ uint32_t dpp_sum_u32(uint32_t v) {
  return lane63_u32(dpp_scan(v, [](uint32_t a, uint32_t b) { return a + b; }));
}
__device__ __forceinline__ uint32_t dpp_or_u32(uint32_t v) {
  return lane63_u32(dpp_scan(v, [](uint32_t a, uint32_t b) { return a | b; }));
}
__device__ __forceinline__ uint32_t dpp_max_u32(uint32_t v) {
  return lane63_u32(dpp_scan(v, [](uint32_t a, uint32_t b) { return a > b ? a : b; }));
}
__device__ __forceinline__ uint64_t dpp_sum_u64(uint64_t v) {
  return lane63_u64(dpp_scan(v, [](uint64_t a, uint64_t b) { return a + b; }));
}
// Largest of the wave's values, none of them negative.
__device__ __forceinline__ double dpp_max_f64(double v) {
  const uint64_t b = dpp_scan((uint64_t)__double_as_longlong(v), [](uint64_t x, uint64_t y) {
    return (uint64_t)__double_as_longlong(
        fmax(__longlong_as_double((long long)x), __longlong_as_double((long long)y)));
  });
  return __longlong_as_double((long long)lane63_u64(b));
}
__device__ __forceinline__ uint32_t dpp_incl_scan_u32(uint32_t v) {
  return dpp_scan(v, [](uint32_t a, uint32_t b) { return a + b; });
}

// Support values are handled as the table index j = v - (xmin - 1) (v itself
// without a cutoff): 1..kHW in the LDS histogram, larger ones in the wave's
// global scratch.
//
// Deferred draws wait by their number and are resolved 64 at a time: on two
// stacks that share an array, body draws to search in full and tail draws (by
// the first word; mixed, each pass ran both paths: heavy tails of 10,000 draws 4.56
// against 4.81 ms).  A tail draw makes one
// proposal per pass; a rejected one waits in a ring with its next attempt, one
// that needs a double-double floor in another, so that a wave runs that long
// path with all its lanes (at alpha = 1.2 one proposal in 80 needs it, which
// was half of all passes).  A pass over body draws draws their uniforms again:
// cheaper than keeping and composing them (an uneven batch, 256 cells: 66.9
// against 69.0 ms).  The stacks hold fewer than 64 entries each before an
// iteration's at most 256 in all.  A pass of one begins with fewer than 64 in
// each ring and adds at most 64 in all, a pass of a ring moves entries or
// removes them and takes no more than the other has room for: both hold at
// most 190 together, 128 each.
constexpr int kBatchRing = 512;
constexpr int kHardRing = 128;
// Histogram layout: bins of j = 1..kHW, a row of 64 of which the first word takes
// all lanes' no-op counts in the draw loop (never read), then three rows of
// per-lane counts of j = 1, 2 and 3 (most draws: a lane counting into its own slot
// never conflicts with another lane).  The KS keeps a byte per bin in the four rows.
constexpr int kWavePad = kHW;
constexpr int kWaveOwn = kHW + 64;
// Draw blocks per lane per iteration of the draw loop.
constexpr int kWaveBlocks = 2;
static_assert(kWaveBlocks == 2, "the draw loop keeps four table reads in flight");
struct alignas(16) BatchLds {
  // during the KS the bin table of the larger draws
  uint32_t hist[kHW + 64 + 3 * 64];
  uint32_t ring[kBatchRing];  // deferred draws; the gathered draws during the KS
  uint64_t retry[kHardRing];  // tail draws whose proposals so far were rejected
  uint64_t hard[kHardRing];   // tail proposals whose floor FP64 does not decide
};

// The larger draws are counted in tables of kHW bins: first 16 per octave of
// j (j >= kHW), then, for a bin in reach of the maximum that holds too many
// draws to gather, a power-of-two range of j in equal bins of 2^sh values.
constexpr int kBucketBits = 4;
constexpr int kBuckets = (63 - 10) << kBucketBits;  // octaves 10..62
static_assert(kHW == 1024 && kBuckets <= kHW, "the bin table takes the histogram's place");
// Draws gathered per pass (the ring's room, less the draws just below a bin),
// and the count from which a bin is split instead.
constexpr uint32_t kGather = 255;  // (places in bytes)
constexpr uint32_t kManyDraws = 255;
// A bin in reach keeps the number of larger draws below it (n <= 2^31), with
// the mark for a draw just below its first value.
constexpr uint32_t kNoBin = 0xffffffffu;
constexpr uint32_t kBelowDrawn = 0x80000000u;

struct Bins {
  uint64_t lo;  // first j
  int sh;       // negative: 16 per octave from kHW on
  __device__ __forceinline__ int of(uint64_t j) const {
    if (sh >= 0) return (int)((j - lo) >> sh);
    const int e = 63 - __clzll((long long)j);
    return ((e - 10) << kBucketBits) + (int)((j >> (e - kBucketBits)) & ((1u << kBucketBits) - 1u));
  }
  __device__ __forceinline__ uint64_t start(int b) const {
    if (sh >= 0) return lo + ((uint64_t)b << sh);
    const int e = 10 + (b >> kBucketBits);
    return ((uint64_t)(b & ((1 << kBucketBits) - 1)) + (1u << kBucketBits)) << (e - kBucketBits);
  }
  __device__ __forceinline__ int width_bits(int b) const {
    return sh >= 0 ? sh : 10 + (b >> kBucketBits) - kBucketBits;
  }
  __device__ __forceinline__ uint64_t end(int b) const {  // last j of bin b
    return start(b) + ((uint64_t)1 << width_bits(b)) - 1u;
  }
};

// The laws: the functions below are instantiated for each, so that one does
// not take the registers of another's sums.
enum Law { kPure = 0, kCutoff = 1, kTrunc = 2 };

// The law at alpha_hat as the KS needs it.
template <int kLaw>
struct KsLaw {
  EmCoef E;
  double iz;     // 1 / normaliser
  int64_t xmin;  // the cutoff (1 without)
  TruncEnd te;   // the truncated law's (trunc_em)
  // sum of k^-a over k > t (t >= 16), relative to xmin^-a for cutoffs above 17
  __device__ __forceinline__ double survival(int64_t t, const double* __restrict__ ln) const {
    if constexpr (kLaw == kCutoff)
      return xmin > 17 ? survival_rel(E, t, xmin) : survival_next_cut(E, t, ln);
    else if constexpr (kLaw == kTrunc)
      return trunc_tail(E, te, t, ln[t < (int64_t)kH ? t + 1 : 0]);
    else
      return survival_next(E, t, ln);
  }
  __device__ __forceinline__ double point(int64_t v, const double* __restrict__ ln) const {
    if constexpr (kLaw == kCutoff)
      if (xmin > 17) return pow_rel(E.s, v, xmin);
    return pow_neg(E.s, ln_value(v, ln));
  }
};

__device__ __forceinline__ double shfl_f64(double v, int src) {
  const uint64_t b = (uint64_t)__double_as_longlong(v);
  const uint32_t lo = (uint32_t)__shfl((int)(uint32_t)b, src, 64);
  const uint32_t hi = (uint32_t)__shfl((int)(uint32_t)(b >> 32), src, 64);
  return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}
__device__ __forceinline__ double readlane_f64(double v, int src) {
  const uint64_t b = (uint64_t)__double_as_longlong(v);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)b, src);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(b >> 32), src);
  return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}
// Inclusive sum within each group of 16 lanes.
__device__ __forceinline__ uint32_t row_incl_scan_u32(uint32_t v) {
  v += dpp0_u32<0x111, 0xf>(v);
  v += dpp0_u32<0x112, 0xf>(v);
  v += dpp0_u32<0x114, 0xf>(v);
  return v + dpp0_u32<0x118, 0xf>(v);
}
// The previous lane's value (0 in lane 0).
__device__ __forceinline__ uint32_t prev_lane_u32(uint32_t v) { return dpp0_u32<0x138, 0xf>(v); }
__device__ __forceinline__ double prev_lane_f64(double v) {
  return __longlong_as_double((long long)dpp0_u64<0x138, 0xf>((uint64_t)__double_as_longlong(v)));
}

// The stored counts of one replicate: 16-bit for n < 65536, else 32-bit.
struct CountView {
  const uint32_t* p;
  bool wide;
  __device__ __forceinline__ uint32_t at(int b) const {  // bin b = j - 1
    if (wide) return p[b];
    const uint32_t w = p[b >> 1];
    return (b & 1) ? (w >> 16) : (w & 0xffffu);
  }
  // Sum of bins 16 g .. 16 g + 15, and the last of them.
  __device__ __forceinline__ uint32_t sum16(int g, uint32_t& last) const {
    uint32_t s = 0;
    if (wide) {
      const uint4* q = reinterpret_cast<const uint4*>(p + 16 * g);
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const uint4 w = q[k];
        s += w.x + w.y + w.z + w.w;
        last = w.w;
      }
    } else {
      const uint4* q = reinterpret_cast<const uint4*>(p + 8 * g);
#pragma unroll
      for (int k = 0; k < 2; ++k) {
        const uint4 w = q[k];
        s += (w.x & 0xffffu) + (w.x >> 16) + (w.y & 0xffffu) + (w.y >> 16) + (w.z & 0xffffu) +
             (w.z >> 16) + (w.w & 0xffffu) + (w.w >> 16);
        last = w.w >> 16;
      }
    }
    return s;
  }
};

// D of one replicate by a whole wave, given D0, the largest term over the
// values up to 16 (taken from the head sums), and z16 = zeta(a, 17).  counts:
// those of j = 1..hi (hi a multiple of 256, zero above); ov[-1 - p], p < oc:
// the draws above kHW, in any order.  tab, list, level: the wave's LDS
// (kHW + 256 words, kBatchRing and kHardRing entries).
// kLarge: there can be such draws (without them the function saves fewer
// registers per call).
template <int kLaw, bool kLarge = true>
static __device__ __noinline__ double ks_rest(double a, double iz, int64_t xmin_, uint32_t K_,
                                              const uint32_t* counts, bool wide_, int hi_,
                                              const int64_t* ov_, uint32_t oc_, int64_t n_,
                                              double D0, double z16, LdsU32* tab, LdsU64* list,
                                              LdsU32* ends, LdsU64* level, const double* ln_) {
  // every argument is the wave's
  const int lane = lane_id();
  const uint32_t nu = (uint32_t)uniform64(n_);
  const double idn = 1.0 / (double)n_;
  const int hi = __builtin_amdgcn_readfirstlane(hi_);
  const uint32_t oc = (uint32_t)__builtin_amdgcn_readfirstlane((int)oc_);
  const int64_t* __restrict__ ov = as_global(reinterpret_cast<const int64_t*>(uniform64((int64_t)ov_)));
  const double* __restrict__ ln = as_global(reinterpret_cast<const double*>(uniform64((int64_t)ln_)));
  const CountView cv{as_global(reinterpret_cast<const uint32_t*>(uniform64((int64_t)counts))),
                     __builtin_amdgcn_readfirstlane((int)wide_) != 0};
  KsLaw<kLaw> w;
  w.E = em_coef(a);
  w.iz = iz;
  w.xmin = kLaw == kCutoff ? uniform64(xmin_) : 1;
  if constexpr (kLaw == kTrunc)
    w.te = trunc_end(w.E, (uint32_t)__builtin_amdgcn_readfirstlane((int)K_), ln);
  const int64_t off = w.xmin - 1;
  const int jh = off < 16 ? 16 - (int)off : 0;  // values up to 16
  double D = D0;  // the lane's largest term
  // the two terms of a sample value v: zv and zv1 the survival sums past v and
  // past v - 1, Cb draws below v, c equal to it
  auto terms = [&](double zv, double zv1, uint32_t Cb, uint32_t c) {
    const double t2 = fabs(fma(zv1, w.iz, -(double)(nu - Cb) * idn));
    const double t1 = fabs(fma(zv, w.iz, -(double)(nu - Cb - c) * idn));
    D = fmax(D, fmax(t1, t2));
  };
  // the next four set bits of mask, one for each 16 lanes (-1: none)
  auto next4 = [&](uint64_t& mask) {
    int p = -1;
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      const int q = mask != 0ull ? __ffsll((long long)mask) - 1 : -1;
      mask &= mask - 1ull;
      if ((lane >> 4) == g) p = q;
    }
    return p;
  };
  // 1. the histogram in 64 chunks of 16 values, one per lane
  uint32_t last = 0, sum = 0;
  if (16 * lane < hi) sum = cv.sum16(lane, last);
  const uint32_t Cr = dpp_incl_scan_u32(sum), Cl = Cr - sum;
  const double zr = w.survival(off + 16 * (lane + 1), ln);  // right edge of the chunk
  {
    const double z = zr * w.iz, s = (double)(nu - Cr) * idn;
    const double Dlow = fmax(D, dpp_max_f64(fabs(z - s)));
    double zl = prev_lane_f64(z), sl = (double)(nu - Cl) * idn;
    if (lane == 0) {
      zl = 1.0;
      sl = 1.0;
    }
    const double bound = fmax(zl - s, sl - z);
    const bool need = sum != 0u && 16 * (lane + 1) > jh && bound > Dlow - kPruneMargin;
    uint64_t mask = __ballot(need);
    // four chunks per round, one value per lane
    while (mask != 0ull) {
      const int p = next4(mask);
      const int pc = p < 0 ? 0 : p;
      const int b = 16 * pc + (lane & 15);
      const uint32_t cnt = p < 0 ? 0u : cv.at(b);
      const uint32_t Ca = (uint32_t)__shfl((int)Cl, pc, 64) + row_incl_scan_u32(cnt);
      const int64_t v = off + b + 1;
      // (values up to 16 are in D0: below a cutoff's direct sums)
      const double zv = w.survival(kLaw == kCutoff && v < 17 ? 17 : v, ln);
      double zp = prev_lane_f64(zv);
      uint32_t cp = prev_lane_u32(cnt);
      const double zq = shfl_f64(zr, pc > 0 ? pc - 1 : 0);
      const uint32_t cq = (uint32_t)__shfl((int)last, pc > 0 ? pc - 1 : 0, 64);
      if ((lane & 15) == 0) {
        zp = zq;
        cp = pc > 0 ? cq : 0u;
      }
      if (v == 17) {
        zp = z16;
        cp = 1u;
      }
      if (cnt != 0u && b >= jh) terms(zv, cp != 0u ? zp : zv + w.point(v, ln), Ca - cnt, cnt);
      // What a round found may rule out the rest.  Worth a maximum over the wave
      // only where the sums cost as much as with a cutoff (1,000 draws: 5.69
      // against 5.89 ms; the truncated law's K = 1,000 6.92 against 6.72).
      if constexpr (kLaw == kCutoff)
        if (mask != 0ull) mask &= __ballot(bound > dpp_max_f64(D) - kPruneMargin);
    }
    D = dpp_max_f64(D);
  }
  if constexpr (!kLarge) return D;
  // 2. the larger draws: none can matter when their whole mass is below D
  const double zE = readlane_f64(zr, 63);
  if (oc == 0u || fmax(zE * w.iz, (double)oc * idn) <= D - kPruneMargin) return D;
  const bool has_top = __builtin_amdgcn_readlane((int)last, 63) != 0;  // j = kHW was drawn
  const uint32_t nbody = nu - oc;
  // at most one per lane: every one is compared with all and evaluated, a third
  // of the tables' work (a call of 83,710 replicates of 34 draws, cutoff 798: 0.91
  // against 1.04 ms)
  if (oc <= 64u) {
    const bool valid = (uint32_t)lane < oc;
    const uint64_t j = valid ? (uint64_t)ov[-1 - (int64_t)lane] : 0ull;
    uint32_t lt = 0, eq = 0;
    bool pres = j == (uint64_t)kHW + 1u && has_top;
    for (int k = 0; k < (int)oc; ++k) {
      const uint64_t x =
          (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)j, k) |
          (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(j >> 32), k) << 32;
      lt += x < j ? 1u : 0u;
      eq += x == j ? 1u : 0u;
      pres = pres || x + 1u == j;
    }
    if (valid) {
      const int64_t v = off + (int64_t)j;
      const double zv = w.survival(v, ln);
      const double zv1 = pres ? w.survival(v - 1, ln) : zv + w.point(v, ln);
      terms(zv, zv1, nbody + lt, eq);
    }
    return dpp_max_f64(D);
  }
  LdsU8* many = (LdsU8*)(tab + kHW);  // counts of the bins in reach, up to kManyDraws
  int depth = 0, next = 0;
  Bins B{(uint64_t)kHW, -1};
  while (depth >= 0) {
    // the table of the range; draws below it; whether the value just below it
    // was drawn
    wave_sync();
    for (int k = lane; k < kHW; k += 64) tab[k] = 0u;
    wave_sync();
    const uint64_t bhi = B.sh >= 0 ? B.end(kHW - 1) : ~0ull;
    uint32_t lower = 0, edge = 0;
    for (uint32_t p = (uint32_t)lane; p < oc; p += 64u) {
      const uint64_t j = (uint64_t)ov[-1 - (int64_t)p];
      if (j >= B.lo && j <= bhi)
        lds_inc(&tab[B.of(j)]);
      else if (j < B.lo) {
        ++lower;
        edge |= j + 1u == B.lo ? 1u : 0u;
      }
    }
    wave_sync();
    if (B.sh >= 0) {
      lower = dpp_sum_u32(lower);
      edge = dpp_or_u32(edge);
    }
    // 16 bins per lane, then those of the lanes in reach, four lanes' bins per
    // round: a single value is evaluated, a wider bin kept when in reach
    uint32_t cs = 0;
#pragma unroll
    for (int k = 0; k < 16; ++k) cs += tab[16 * lane + k];
    const uint32_t cr = lower + dpp_incl_scan_u32(cs), cl = cr - cs;
    const bool real = B.sh >= 0 || lane < (kBuckets >> kBucketBits);
    auto right = [&](int b) {
      const uint64_t e = (uint64_t)off + B.end(b);
      return e < (uint64_t)INT64_MAX ? (int64_t)e : INT64_MAX;
    };
    const double zo = w.survival(right(real ? 16 * lane + 15 : 15), ln);
    const double zlo = B.sh >= 0 && B.lo > (uint64_t)kHW
                           ? w.survival(off + (int64_t)B.lo - 1, ln)
                           : zE;
    double Dlow = fmax(D, dpp_max_f64(real ? fabs(zo * w.iz - (double)(oc - cr) * idn) : 0.0));
    double zl = prev_lane_f64(zo);
    if (lane == 0) zl = zlo;
    const bool need = cs != 0u && fmax(zl * w.iz - (double)(oc - cr) * idn,
                                       (double)(oc - cl) * idn - zo * w.iz) > Dlow - kPruneMargin;
    if (!need && B.sh != 0) {
#pragma unroll
      for (int k = 0; k < 16; ++k) tab[16 * lane + k] = kNoBin;
    }
    uint64_t mask = __ballot(need);
    uint32_t small = 0, large = 0;
    while (mask != 0ull) {
      const int p = next4(mask);
      const int pc = p < 0 ? 0 : p;
      const int b = 16 * pc + (lane & 15);
      const uint32_t cnt = p < 0 ? 0u : tab[b];
      const uint32_t ca = (uint32_t)__shfl((int)cl, pc, 64) + row_incl_scan_u32(cnt);
      const int64_t t = right(b);
      const double zv = w.survival(t, ln);
      double zp = prev_lane_f64(zv);
      const double zq = shfl_f64(zl, pc);
      if ((lane & 15) == 0) zp = zq;
      if (B.sh == 0) {
        const bool pres = B.lo + (uint64_t)b == (uint64_t)kHW + 1u
                              ? has_top
                              : (b > 0 ? tab[b - 1] != 0u : edge != 0u);
        if (cnt != 0u) terms(zv, pres ? zp : zv + w.point(t, ln), nbody + ca - cnt, cnt);
      } else {
        const double sb = (double)(oc - ca) * idn;
        Dlow = fmax(Dlow, dpp_max_f64(p < 0 ? 0.0 : fabs(zv * w.iz - sb)));
        const bool in = cnt != 0u && fmax(zp * w.iz - sb, (double)(oc - (ca - cnt)) * idn -
                                                              zv * w.iz) > Dlow - kPruneMargin;
        if (p >= 0) {
          tab[b] = in ? ca - cnt : kNoBin;
          many[b] = (uint8_t)(cnt < kManyDraws ? cnt : kManyDraws);
        }
        small += in && cnt < kManyDraws ? cnt : 0u;
        large |= in && cnt >= kManyDraws ? 1u : 0u;
      }
    }
    if (B.sh != 0) {
      small = next == 0 ? dpp_sum_u32(small) : 0u;
      large = dpp_or_u32(large);
    }
    wave_sync();
    // 3. the draws of the smaller bins in reach, gathered into LDS: in one pass
    // when they fit, else a window of bins at a time.  A draw equal to the
    // value just below a bin marks the bin's entry (it decides a term).
    int wlo = 0;
    while (small != 0u && wlo < kHW) {
      int whi = kHW;
      if (small > kGather) {
        const int b = wlo + lane;
        uint32_t c = 0;
        if (b < kHW && tab[b] != kNoBin) c = many[b];
        c = c < kManyDraws ? c : 0u;
        const uint64_t fit = __ballot(dpp_incl_scan_u32(c) <= kGather);
        const int take = fit == ~0ull ? 64 : __ffsll((long long)~fit) - 1;  // at least one
        whi = wlo + take < kHW ? wlo + take : kHW;
        if (__ballot(c != 0u && lane < take) == 0ull) {
          wlo = whi;
          continue;
        }
      }
      auto wanted = [&](uint64_t j) {
        if (j < B.lo || j > bhi) return false;
        const int b = B.of(j);
        return b >= wlo && b < whi && tab[b] != kNoBin && many[b] < kManyDraws;
      };
      // The list is grouped by bin, so that a draw is compared with its bin's
      // only: each bin's first place, then (as its draws are placed) its end,
      // in bytes.
      uint32_t m = 0;  // draws of the window (wave-uniform)
      {
        auto count = [&](int b) {
          const uint32_t n = many[b];
          return b >= wlo && b < whi && tab[b] != kNoBin && n < kManyDraws ? n : 0u;
        };
        // (counted twice: kept, they would take registers from every call)
        uint32_t cs16 = 0;
#pragma unroll 1
        for (int k = 0; k < 16; ++k) cs16 += count(16 * lane + k);
        const uint32_t inc = dpp_incl_scan_u32(cs16);
        m = (uint32_t)__builtin_amdgcn_readlane((int)inc, 63);
        uint32_t at = inc - cs16;
#pragma unroll 1
        for (int k = 0; k < 4; ++k) {
          uint32_t places = 0;
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            places |= at << (8 * i);
            at += count(16 * lane + 4 * k + i);
          }
          ends[4 * lane + k] = places;
        }
        wave_sync();
      }
      for (uint32_t p0 = 0; p0 < oc; p0 += 64u) {
        const uint32_t p = p0 + (uint32_t)lane;
        bool take = false;
        uint64_t j = 0;
        if (p < oc) {
          j = (uint64_t)ov[-1 - (int64_t)p];
          take = wanted(j);
          if (wanted(j + 1u) && (j < B.lo || B.of(j) != B.of(j + 1u)))
            lds_or(&tab[B.of(j + 1u)], kBelowDrawn);
        }
        if (take) {
          const int b = B.of(j);
          const uint32_t old = __hip_atomic_fetch_add(&ends[b >> 2], 1u << (8 * (b & 3)),
                                                      __ATOMIC_RELAXED,
                                                      __HIP_MEMORY_SCOPE_WORKGROUP);
          list[(old >> (8 * (b & 3))) & 0xffu] = j;  // below m, at most kGather
        }
      }
      wave_sync();
      for (uint32_t i0 = 0; i0 < m; i0 += 64u) {
        const uint32_t i = i0 + (uint32_t)lane;
        const uint64_t j = i < m ? list[i] : 0ull;
        const bool valid = i < m;
        const int bj = valid ? B.of(j) : 0;
        const uint32_t entry = valid ? tab[bj] : 0u;
        const uint64_t jlo = valid ? B.start(bj) : 0ull;
        const uint32_t k1 = valid ? (ends[bj >> 2] >> (8 * (bj & 3))) & 0xffu : 0u;
        uint32_t lt = 0, eq = 0;
        uint32_t pres = j == (uint64_t)kHW + 1u ? (has_top ? 1u : 0u)
                                                 : (j == jlo ? entry >> 31 : 0u);
        for (uint32_t k = valid ? k1 - many[bj] : 0u; k < k1; ++k) {
          const uint64_t x = list[k];
          lt += x < j ? 1u : 0u;
          eq += x == j ? 1u : 0u;
          pres |= x + 1u == j ? 1u : 0u;
        }
        if (valid) {
          const int64_t v = off + (int64_t)j;
          const double zv = w.survival(v, ln);
          const double zv1 = pres ? w.survival(v - 1, ln) : zv + w.point(v, ln);
          terms(zv, zv1, nbody + (entry & ~kBelowDrawn) + lt, eq);
        }
      }
      wave_sync();
      wlo = whi;
    }
    D = dpp_max_f64(D);
    // 4. the bins with many draws, one after another, as ranges of their own
    int child = -1;
    if (large != 0u) {
      for (int b0 = next & ~63; b0 < kHW && child < 0; b0 += 64) {
        const int b = b0 + lane;
        const uint64_t hit =
            __ballot(b >= next && tab[b] != kNoBin && many[b] == (uint8_t)kManyDraws);
        if (hit != 0ull) child = b0 + __ffsll((long long)hit) - 1;
      }
    }
    if (child >= 0) {
      if (lane == 0) {
        level[3 * depth] = B.lo;
        level[3 * depth + 1] = (uint64_t)(int64_t)B.sh;
        level[3 * depth + 2] = (uint64_t)(child + 1);
      }
      const int bits = B.width_bits(child);
      B = Bins{B.start(child), bits > 10 ? bits - 10 : 0};
      next = 0;
      ++depth;
    } else {
      --depth;
      if (depth >= 0) {
        wave_sync();
        B.lo = (uint64_t)uniform64((int64_t)level[3 * depth]);
        B.sh = (int)uniform64((int64_t)level[3 * depth + 1]);
        next = (int)uniform64((int64_t)level[3 * depth + 2]);
      }
    }
  }
  return D;
}

// ks_rest's second part for a replicate with many larger draws.  Gathered window
// by window, every window of 255 reads them all again: of 20,000 draws above the
// histogram nearly all are in reach (D is about 0.005, a bin holds 0.003 of them),
// and 80 passes over them took 18 ms where the whole replicate had taken 7.4.
// Here the bins in reach are copied out in order once, those of up to 254 draws
// first; a window is then a piece of the copy, and a bin with more is a
// contiguous range with a table, a copy and bins of its own.
// D0: the largest term over the values of the histogram.  work, words: the
// scratch behind the batch's counts.  Negative: it does not hold the copies (the
// caller takes the windows over all draws instead).
template <int kLaw>
static __device__ __noinline__ double ks_many(double a, double iz, int64_t xmin_, uint32_t K_,
                                              bool has_top_, const int64_t* ov_, uint32_t oc_,
                                              int64_t* work_, int64_t words_, int64_t n_, double D0,
                                              LdsU32* tab, LdsU64* list, LdsU64* level,
                                              const double* ln_) {
  // every argument is the wave's
  const int lane = lane_id();
  const uint32_t nu = (uint32_t)uniform64(n_);
  const double idn = 1.0 / (double)n_;
  const uint32_t oc = uniform32(oc_);
  const bool has_top = uniform32(has_top_) != 0u;
  int64_t* work = as_global(reinterpret_cast<int64_t*>(uniform64((int64_t)work_)));
  const int64_t words = uniform64(words_);
  const double* __restrict__ ln = as_global(reinterpret_cast<const double*>(uniform64((int64_t)ln_)));
  KsLaw<kLaw> w;
  w.E = em_coef(a);
  w.iz = iz;
  w.xmin = kLaw == kCutoff ? uniform64(xmin_) : 1;
  if constexpr (kLaw == kTrunc) w.te = trunc_end(w.E, uniform32(K_), ln);
  const int64_t off = w.xmin - 1;
  double D = D0;
  const double zE = w.survival(off + kHW, ln);
  if (fmax(zE * w.iz, (double)oc * idn) <= D - kPruneMargin) return D;
  const uint32_t nbody = nu - oc;
  auto terms = [&](double zv, double zv1, uint32_t Cb, uint32_t c) {
    const double t2 = fabs(fma(zv1, w.iz, -(double)(nu - Cb) * idn));
    const double t1 = fabs(fma(zv, w.iz, -(double)(nu - Cb - c) * idn));
    D = fmax(D, fmax(t1, t2));
  };
  LdsU8* many = (LdsU8*)(tab + kHW);  // counts of the bins in reach, up to kManyDraws
  // the range at hand: its bins and how many of them are in it, its draws, the
  // larger draws below it, whether the value just below it was drawn, and the
  // words of `work` in use
  Bins B{(uint64_t)kHW, -1};
  int nbins = kBuckets;
  const int64_t* src = as_global(reinterpret_cast<const int64_t*>(uniform64((int64_t)ov_))) - oc;
  uint32_t len = oc, lower = 0;
  bool edge = false;
  int64_t used = 0;
  int depth = 0;
  for (;;) {
    if (B.sh != 0 && used + kPartLevel > words) return -1.0;
    // of each bin in reach: its draws, its first place in the copy, the larger
    // draws below it (with kBelowDrawn)
    uint32_t* cnts = reinterpret_cast<uint32_t*>(work + used);
    uint32_t* firsts = cnts + kHW;
    uint32_t* belows = firsts + kHW;
    int64_t* part = work + used + kPartLevel;
    auto each = [&](auto fn) {  // fn of every draw, four loads in flight
      uint32_t p = (uint32_t)lane;
      for (; p + 192u < len; p += 256u) {
        uint64_t j[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) j[k] = (uint64_t)src[p + 64u * k];
#pragma unroll
        for (int k = 0; k < 4; ++k) fn(j[k]);
      }
      for (; p < len; p += 64u) fn((uint64_t)src[p]);
    };
    wave_sync();
    for (int k = lane; k < kHW; k += 64) tab[k] = 0u;
    wave_sync();
    each([&](uint64_t j) { lds_inc(&tab[B.of(j)]); });
    wave_sync();
    uint32_t cs = 0;
#pragma unroll
    for (int k = 0; k < 16; ++k) cs += tab[16 * lane + k];
    const uint32_t cr = lower + dpp_incl_scan_u32(cs), cl = cr - cs;
    auto right = [&](int b) {
      const uint64_t e = (uint64_t)off + B.end(b);
      return e < (uint64_t)INT64_MAX ? (int64_t)e : INT64_MAX;
    };
    // (S_n is known at the edges of the range's own bins only)
    const bool real = 16 * lane + 15 < nbins;
    const double zo = w.survival(right(16 * lane < kBuckets || B.sh >= 0 ? 16 * lane + 15 : 15), ln);
    const double zlo = B.sh >= 0 ? w.survival(off + (int64_t)B.lo - 1, ln) : zE;
    double Dlow = fmax(D, dpp_max_f64(real ? fabs(zo * w.iz - (double)(oc - cr) * idn) : 0.0));
    double zl = prev_lane_f64(zo);
    if (lane == 0) zl = zlo;
    const bool need = cs != 0u && fmax(zl * w.iz - (double)(oc - cr) * idn,
                                       (double)(oc - cl) * idn - zo * w.iz) > Dlow - kPruneMargin;
    if (!need && B.sh != 0) {
#pragma unroll
      for (int k = 0; k < 16; ++k) tab[16 * lane + k] = kNoBin;
#pragma unroll
      for (int k = 0; k < 4; ++k)
        reinterpret_cast<uint4*>(cnts + 16 * lane)[k] = uint4{0u, 0u, 0u, 0u};
    }
    uint64_t mask = __ballot(need);
    uint32_t small = 0, large = 0;
    while (mask != 0ull) {  // 16 bins of four lanes per round
      int p = -1;
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const int q = mask != 0ull ? __ffsll((long long)mask) - 1 : -1;
        mask &= mask - 1ull;
        if ((lane >> 4) == g) p = q;
      }
      const int pc = p < 0 ? 0 : p;
      const int b = 16 * pc + (lane & 15);
      const uint32_t cnt = p < 0 ? 0u : tab[b];
      const uint32_t ca = (uint32_t)__shfl((int)cl, pc, 64) + row_incl_scan_u32(cnt);
      const int64_t t = right(b);
      const double zv = w.survival(t, ln);
      double zp = prev_lane_f64(zv);
      const double zq = shfl_f64(zl, pc);
      if ((lane & 15) == 0) zp = zq;
      if (B.sh == 0) {  // single values
        const bool pres = B.lo + (uint64_t)b == (uint64_t)kHW + 1u
                              ? has_top
                              : (b > 0 ? tab[b - 1] != 0u : edge);
        if (cnt != 0u) terms(zv, pres ? zp : zv + w.point(t, ln), nbody + ca - cnt, cnt);
      } else {
        const double sb = (double)(oc - ca) * idn;
        Dlow = fmax(Dlow, dpp_max_f64(p < 0 ? 0.0 : fabs(zv * w.iz - sb)));
        const bool in = cnt != 0u && fmax(zp * w.iz - sb, (double)(oc - (ca - cnt)) * idn -
                                                              zv * w.iz) > Dlow - kPruneMargin;
        if (p >= 0) {
          tab[b] = in ? ca - cnt : kNoBin;
          cnts[b] = in ? cnt : 0u;
          many[b] = (uint8_t)(cnt < kManyDraws ? cnt : kManyDraws);
        }
        small += in && cnt < kManyDraws ? cnt : 0u;
        large += in && cnt >= kManyDraws ? cnt : 0u;
      }
    }
    small = dpp_sum_u32(small);
    large = dpp_sum_u32(large);
    const uint32_t m = small + large;
    if (m != 0u) {
      if (used + kPartLevel + (int64_t)m > words) return -1.0;
      wave_sync_global();
      // the places, 16 bins per lane; the table then counts them up
      {
        uint32_t c1 = 0, c2 = 0;
#pragma unroll 4
        for (int k = 0; k < 16; ++k) {
          const int b = 16 * lane + k;
          const uint32_t c = cnts[b];
          c1 += c < kManyDraws ? c : 0u;
          c2 += c < kManyDraws ? 0u : c;
        }
        uint32_t p1 = dpp_incl_scan_u32(c1) - c1, p2 = small + dpp_incl_scan_u32(c2) - c2;
#pragma unroll 4
        for (int k = 0; k < 16; ++k) {
          const int b = 16 * lane + k;
          const uint32_t c = cnts[b];
          if (c == 0u) continue;
          const uint32_t at = c < kManyDraws ? p1 : p2;
          firsts[b] = at;
          belows[b] = tab[b];
          tab[b] = at | (b == 0 && edge ? kBelowDrawn : 0u);
          p1 += c < kManyDraws ? c : 0u;
          p2 += c < kManyDraws ? 0u : c;
        }
        wave_sync();
      }
      // a draw equal to the value just below another bin marks that bin's entry
      const uint64_t last = B.sh >= 0 ? B.end(kHW - 1) : ~0ull;
      each([&](uint64_t j) {
        const int b = B.of(j);
        if (tab[b] != kNoBin) {
          const uint32_t at = __hip_atomic_fetch_add(&tab[b], 1u, __ATOMIC_RELAXED,
                                                     __HIP_MEMORY_SCOPE_WORKGROUP);
          part[at & ~kBelowDrawn] = (int64_t)j;
        }
        if (j < last) {
          const int b1 = B.of(j + 1u);
          if (b1 != b && tab[b1] != kNoBin) lds_or(&tab[b1], kBelowDrawn);
        }
      });
      wave_sync();
#pragma unroll 4
      for (int k = 0; k < 16; ++k) {  // marks, kept for the ranges of their own
        const int b = 16 * lane + k;
        if (tab[b] != kNoBin && (tab[b] & kBelowDrawn) != 0u) belows[b] |= kBelowDrawn;
      }
      wave_sync_global();
      // the bins of up to 254 draws, whole bins of at most kGather draws at a time
      uint32_t w0 = 0;
      for (int lo = 0; w0 < small && lo < kHW;) {
        const int b = lo + lane;
        uint32_t c = 0;
        if (b < kHW && tab[b] != kNoBin) c = many[b];
        c = c < kManyDraws ? c : 0u;
        const uint32_t inc = dpp_incl_scan_u32(c);
        const uint64_t fit = __ballot(inc <= kGather);
        const int take = fit == ~0ull ? 64 : __ffsll((long long)~fit) - 1;  // at least one
        const uint32_t wn = (uint32_t)__builtin_amdgcn_readlane((int)inc, take - 1);
        lo += take;
        for (uint32_t i = (uint32_t)lane; i < wn; i += 64u) list[i] = (uint64_t)part[w0 + i];
        wave_sync();
        for (uint32_t i = (uint32_t)lane; i < wn; i += 64u) {
          const uint64_t j = list[i];
          const int bj = B.of(j);
          const uint32_t entry = tab[bj];
          const uint32_t k1 = (entry & ~kBelowDrawn) - w0;  // past the bin's last
          uint32_t lt = 0, eq = 0;
          uint32_t pres = j == (uint64_t)kHW + 1u ? (has_top ? 1u : 0u)
                                                   : (j == B.start(bj) ? entry >> 31 : 0u);
          for (uint32_t k = k1 - many[bj]; k < k1; ++k) {
            const uint64_t x = list[k];
            lt += x < j ? 1u : 0u;
            eq += x == j ? 1u : 0u;
            pres |= x + 1u == j ? 1u : 0u;
          }
          const int64_t v = off + (int64_t)j;
          const double zv = w.survival(v, ln);
          const double zv1 = pres ? w.survival(v - 1, ln) : zv + w.point(v, ln);
          terms(zv, zv1, nbody + (belows[bj] & ~kBelowDrawn) + lt, eq);
        }
        wave_sync();
        w0 += wn;
      }
    }
    D = dpp_max_f64(D);
    // the bins with more, one after another
    if (large != 0u) {
      if (lane == 0) {
        level[5 * depth] = B.lo;
        level[5 * depth + 1] = (uint64_t)(int64_t)B.sh;
        level[5 * depth + 2] = (uint64_t)used;
        level[5 * depth + 3] = (uint64_t)((m + 1u) & ~1u);  // (16-byte alignment)
        level[5 * depth + 4] = 0u;
      }
      ++depth;
    }
    wave_sync();
    for (;;) {
      if (depth == 0) return D;
      LdsU64* r = level + 5 * (depth - 1);
      const Bins P{(uint64_t)uniform64((int64_t)r[0]), (int)uniform64((int64_t)r[1])};
      const int64_t base = uniform64((int64_t)r[2]);
      const int next = (int)uniform64((int64_t)r[4]);
      const uint32_t* pc = reinterpret_cast<const uint32_t*>(work + base);
      int child = -1;
      for (int b0 = next & ~63; b0 < kHW && child < 0; b0 += 64) {
        const uint64_t hit = __ballot(b0 + lane >= next && pc[b0 + lane] >= kManyDraws);
        if (hit != 0ull) child = b0 + __ffsll((long long)hit) - 1;
      }
      if (child < 0) {
        --depth;
        continue;
      }
      used = base + kPartLevel + uniform64((int64_t)r[3]);
      wave_sync();
      if (lane == 0) r[4] = (uint64_t)(child + 1);
      len = uniform32(pc[child]);
      src = work + base + kPartLevel + uniform32(pc[kHW + child]);
      const uint32_t bl = uniform32(pc[2 * kHW + child]);
      lower = bl & ~kBelowDrawn;
      edge = (bl & kBelowDrawn) != 0u;
      const int bits = P.width_bits(child);
      B = Bins{P.start(child), bits > 10 ? bits - 10 : 0};
      nbins = 1 << (bits > 10 ? 10 : bits);
      break;
    }
  }
}

// Record of one replicate of a batch.
struct WaveSlot {
  U128 S;
  uint64_t fp;
  int64_t top;  // its larger draws lie below this offset of the scratch
  uint32_t hi, len, flags, esc;
};

// The places of a wave's scratch: records, counts of each replicate, then free
// space and the draws above kHW from the end.
constexpr int64_t kBatchRecords = 64 * (int64_t)kWaveSlotBytes / 8;
__device__ __forceinline__ int64_t count_words(int64_t n) {  // int64 per replicate's counts
  return n >= 65536 ? kHW / 2 : kHW / 4;
}

// ks_rest for the replicates of a batch that have many larger draws (bits of
// `left`; a, iz, D and z16 are each lane's own replicate's, D comes back), the
// batch's q replicates in scratch, their draws from `top` on.  One call outside the
// loop over the others, with few arguments: in the batch's own body it took
// registers from every replicate (six cutoff cells of 1,000 draws: 5.91 against
// 5.78 ms).
template <int kLaw>
static __device__ __noinline__ double ks_parted(uint64_t left, double a, double iz, double D,
                                                double z16, const DevCell* cell,
                                                int64_t* scratch_, int q, int64_t top_,
                                                LdsU32* lds, const double* ln) {
  const int lane = lane_id();
  const DevCell& c = *as_global(reinterpret_cast<const DevCell*>(uniform64((int64_t)cell)));
  int64_t* scratch = as_global(reinterpret_cast<int64_t*>(uniform64((int64_t)scratch_)));
  const int64_t n = uniform64(c.n), cw = count_words(n);
  const bool wide = n >= 65536;
  int64_t* counts = scratch + kBatchRecords;
  int64_t* work = counts + uniform32((uint32_t)q) * cw;
  const int64_t words = scratch + uniform64(top_) - work;
  LdsU64* list = (LdsU64*)(lds + offsetof(BatchLds, ring) / 4);
  LdsU32* ends = lds + offsetof(BatchLds, retry) / 4;
  LdsU64* level = (LdsU64*)(lds + offsetof(BatchLds, hard) / 4);
  left = (uint64_t)uniform64((int64_t)left);
  while (left != 0ull) {
    const int i = __ffsll((long long)left) - 1;
    left &= left - 1ull;
    const WaveSlot& sl = reinterpret_cast<const WaveSlot*>(scratch)[i];
    const int hi = (int)uniform32(sl.hi);
    const uint32_t oc = uniform32(sl.len);
    const int64_t* ov = scratch + uniform64(sl.top);
    const CountView cv{reinterpret_cast<const uint32_t*>(counts + i * cw), wide};
    const double ai = readlane_f64(a, i), izi = readlane_f64(iz, i);
    // the histogram alone (as without larger draws), then those by bin or, where
    // their copies do not fit, in windows
    double Di = readlane_f64(D, i);
    for (uint32_t large = 0u;; large = oc) {
      Di = ks_rest<kLaw>(ai, izi, c.xmin, c.K, cv.p, wide, hi, ov, large, n, Di,
                         readlane_f64(z16, i), lds, list, ends, level, ln);
      if (large != 0u) break;
      const double r = ks_many<kLaw>(ai, izi, c.xmin, c.K, hi == kHW && cv.at(kHW - 1) != 0u, ov,
                                     oc, work, words, n, Di, lds, list, level, ln);
      if (r >= 0.0) {
        Di = r;
        break;
      }
    }
    if (lane == i) D = Di;
  }
  return D;
}

// One proposal of the tail sampler (tail_draw_from): taken (X), rejected,
// rejected above 2^63, or undecided in FP64 (tail_hard repeats it with the
// floor in double-double).  The last attempt that an entry can hold is taken
// as the sampler's last resort is (never reached: it would follow 2^21
// rejections).
constexpr uint32_t kTailAttempts = (1u << 21) - 1u;
constexpr uint32_t kTailTaken = 0, kTailRejected = 1, kTailCapped = 2, kTailHard = 3,
                   kTailFirst = 4;  // (no proposal made yet)
struct TailTry {
  int64_t X;
  uint32_t code;
};
static __device__ __noinline__ TailTry tail_try(double m0, double beta, double gm, uint32_t k0,
                                                uint32_t k1, uint32_t i, uint32_t rep,
                                                uint32_t stream, uint32_t attempt) {
  const Words4 w = philox4x32_10(i, rep, stream, kTailDomain | attempt, k0, k1);
  if (attempt == kTailAttempts) return TailTry{(int64_t)m0, kTailTaken};
  const double V = u53(w.w0, w.w1);
  const double W = u53(w.w2, w.w3);
  const double z = -log(V) / beta;
  const double y = m0 * exp(z);
  if (y >= 0x1p63 * (1.0 + 0x1p-40)) return TailTry{0, kTailCapped};
  const double fy = floor(y);
  const double tol = y * 0x1p-44;
  if (!(y < 0x1p52 && (y - fy) > tol && (fy + 1.0 - y) > tol)) return TailTry{0, kTailHard};
  const double wg = W * gm;
  const bool take = wg * beta <= 1.0 - 0x1p-39 || wg <= tail_g(beta, fy);
  return TailTry{(int64_t)fy, take ? kTailTaken : kTailRejected};
}
static __device__ __noinline__ TailTry tail_hard(double m0, double beta, double gm, uint32_t k0,
                                                 uint32_t k1, uint32_t i, uint32_t rep,
                                                 uint32_t stream, uint32_t attempt) {
  const Words4 w = philox4x32_10(i, rep, stream, kTailDomain | attempt, k0, k1);
  int64_t X;
  if (!tail_floor_dd(u53(w.w0, w.w1), beta, m0, &X)) return TailTry{0, kTailCapped};
  const double wg = u53(w.w2, w.w3) * gm;
  const bool take = wg * beta <= 1.0 - 0x1p-39 || wg <= tail_g(beta, (double)X);
  return TailTry{X, take ? kTailTaken : kTailRejected};
}

// The draws of replicate rep of a cell by one wave (a loop pipelined as the
// lane form's): counts of j <= kHW into the histogram (the rows of 1..3 added
// in at the end), larger ones to top[-1 - p], p < ovn, as far as `room` reaches
// (ovn counts them all).  On entry bins [0, hi) may be nonzero and are cleared;
// on return hi covers the bins that may be nonzero.  Called, like the stages
// after it: in one body the persistent kernel keeps all their constants in
// registers and the draw loop spills.
struct DrawOut {
  uint32_t fl, ovn;
  int hi;
};
// The first words of the two blocks' uniforms (w0 and w2 of each).  The blocks'
// rounds are kept side by side: one block is two dependent chains, and three
// waves need about four to fill the vector ALU's issue slots (an uneven batch,
// 256 cells: 61.4 against 63.3 ms one block after the other; heavy tails 4.81
// against 4.88).  The lane form keeps them apart: its slice of 9 cells gains 2 %,
// but the truncated law's short replicates at K = 20 lose as much.
__device__ __forceinline__ void philox_pair(uint32_t a0, uint32_t b0, uint32_t c1, uint32_t c2,
                                            uint32_t k0, uint32_t k1, uint32_t (&w)[4]) {
  uint32_t a1 = c1, a2 = c2, a3 = 0u, b1 = c1, b2 = c2, b3 = 0u;
#pragma unroll
  for (int r = 0; r < 10; ++r) {
    const uint64_t pa0 = (uint64_t)0xD2511F53u * a0, pb0 = (uint64_t)0xD2511F53u * b0;
    const uint64_t pa1 = (uint64_t)0xCD9E8D57u * a2, pb1 = (uint64_t)0xCD9E8D57u * b2;
    a0 = xor3((uint32_t)(pa1 >> 32), a1, k0);
    b0 = xor3((uint32_t)(pb1 >> 32), b1, k0);
    a2 = xor3((uint32_t)(pa0 >> 32), a3, k1);
    b2 = xor3((uint32_t)(pb0 >> 32), b3, k1);
    a1 = (uint32_t)pa1;
    b1 = (uint32_t)pb1;
    a3 = (uint32_t)pa0;
    b3 = (uint32_t)pb0;
    k0 += 0x9E3779B9u;
    k1 += 0xBB67AE85u;
    __builtin_amdgcn_sched_barrier(0);  // a round of both at a time
  }
  w[0] = a0;
  w[1] = a2;
  w[2] = b0;
  w[3] = b2;
}

// (kKernel only tells the kernels' copies apart: each then has its own tables'
// LDS addresses as constants.)
template <bool kCut, int kKernel>
static __device__ __noinline__ DrawOut draw_replicate(const DevCell* cell, uint32_t rep_,
                                                      LdsU32* hist, LdsU32* ring, LdsU64* retry,
                                                      LdsU64* hard,
                                                      int64_t* top_, uint32_t room_,
                                                      const LdsU32* T, const LdsU32* guide,
                                                      int hi_) {
  const int lane = lane_id();
  const DevCell& c = *as_global(reinterpret_cast<const DevCell*>(uniform64((int64_t)cell)));
  const uint32_t rep = (uint32_t)__builtin_amdgcn_readfirstlane((int)rep_);
  const uint32_t room = (uint32_t)__builtin_amdgcn_readfirstlane((int)room_);
  int64_t* __restrict__ top = as_global(reinterpret_cast<int64_t*>(uniform64((int64_t)top_)));
  const int hi0 = __builtin_amdgcn_readfirstlane(hi_);
  for (int k = lane; k < hi0; k += 64) hist[k] = 0u;
#pragma unroll
  for (int k = 0; k < 3; ++k) hist[kWaveOwn + k * 64 + lane] = 0u;
  wave_sync();
  const uint32_t n32 = (uint32_t)uniform64(c.n);
  const uint32_t nblk = (n32 >> 1) + (n32 & 1u);
  const uint64_t timax = (uint64_t)uniform64((int64_t)table_int(c.tmax));
  const int sh = __builtin_amdgcn_readfirstlane((int)c.gsh);
  const uint32_t ck0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)c.k0);
  const uint32_t ck1 = (uint32_t)__builtin_amdgcn_readfirstlane((int)c.k1);
  const uint32_t cs = (uint32_t)__builtin_amdgcn_readfirstlane((int)c.stream);
  const double m0 = kCut ? (double)(c.xmin + kH) : kTailM;
  const double beta = c.beta, gm = c.gm;
  const int64_t off = kCut ? uniform64(c.xmin) - 1 : 0;
  // LDS addresses of the bins and of the lane's own counters
  const uint32_t bins = (uint32_t)(uintptr_t)hist;
  const uint32_t own = bins + 4u * (uint32_t)(kWaveOwn + lane);
  uint32_t xm = 0;  // largest offset drawn (16 bits), values above kHW included
  uint32_t fl = 0, ovn = 0;
  // lengths of the stacks; first places and lengths of the rings (wave-uniform)
  uint32_t qn = 0, tn = 0, rh = 0, rn = 0, hh = 0, hn = 0;
  const uint32_t tailw = threshold_hi(timax);  // larger first words: tail uniforms
  // larger draws (j > kHW) of the lanes that have one, in converged code
  auto put_big = [&](int64_t j) {
    const uint64_t mb = __ballot(j > kHW);
    if (mb != 0ull) {
      const uint32_t pos = ovn + place_below(mb);
      if (j > kHW && pos < room) top[-1 - (int64_t)pos] = j;
      ovn += (uint32_t)__popcll(mb);
    }
  };
  // the uniforms' first words
  auto gen = [&](uint32_t j0, uint32_t (&ho)[4]) {
    uint32_t k0 = ck0, k1 = ck1;  // round keys per pair (see lane_draws)
    asm volatile("" : "+s"(k0), "+s"(k1));
    philox_pair(j0 + (uint32_t)lane, j0 + 64u + (uint32_t)lane, rep, cs, k0, k1, ho);
  };
  const GuideRule rule = guide_rule(sh);
  uint32_t wh[4];
  int gi[4];
  gen(0u, wh);
#pragma unroll
  for (int d = 0; d < 4; ++d) gi[d] = guide_index32(wh[d], rule);
  for (uint32_t j0 = 0;;) {
    uint32_t gg[4];
#pragma unroll
    for (int d = 0; d < 4; ++d) gg[d] = guide[gi[d]];
    uint32_t nh[4];
#pragma unroll
    for (int d = 0; d < 4; ++d) asm volatile("" : "=v"(nh[d]));  // any (see more)
    const bool more = j0 + 64u * kWaveBlocks < nblk;
    if (more) gen(j0 + 64u * kWaveBlocks, nh);  // none past the end
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
    if (n32 - 2u * j0 < 4u * 64u) {  // the last ones
      // draw d of the lane is number 2 lane + (d & 1) of the wave's 128 from
      // 2 j0 + 128 (d >> 1) on
      const int left = (int)(n32 - 2u * j0);
#pragma unroll
      for (int d = 0; d < 4; ++d)
        if (2 * lane >= left - 128 * (d >> 1) - (d & 1)) z[d] = kNoDraw;
    }
#pragma unroll
    for (int d = 0; d < 4; ++d) {
      // values 1..3 into the lane's own counters, what is above 1..kHW into the
      // pad
      const uint32_t at = z[d] < 12u ? (z[d] << 6) + own : min(z[d], 4u * (uint32_t)kWavePad) + bins;
      lds_inc((LdsU32*)(uintptr_t)at);
      // the largest offset, marks left out: they are negative in 16 bits
      asm("v_max_i16 %0, %0, %1" : "+v"(xm) : "v"(z[d]));
    }
    if (__ballot(max(max(z[0], z[1]), max(z[2], z[3])) >= 4u * (uint32_t)kHW) != 0ull) {
#pragma unroll
      for (int d = 0; d < 4; ++d) {
        const bool bg = z[d] >= 4u * (uint32_t)kHW && z[d] < (uint32_t)kDeferred;
        const uint64_t mb = __ballot(bg);
        if (mb != 0ull) {
          const uint32_t at = ovn + place_below(mb);
          if (bg && at < room) top[-1 - (int64_t)at] = (int64_t)((z[d] >> 2) + 1u);
          ovn += (uint32_t)__popcll(mb);
        }
        // deferred draws onto the stacks, by their number (their uniform is drawn
        // again when they are resolved): tail draws from the end
        const uint64_t md = __ballot(deferred(z[d])), mt = md & __ballot(wh[d] > tailw);
        if (md != 0ull) {
          const bool tl = wh[d] > tailw;
          const uint32_t pos = tl ? (uint32_t)kBatchRing - 1u - place_below(mt, tn)
                                  : place_below(md & ~mt, qn);
          if ((md >> lane) & 1ull)
            ring[pos] = 2u * (j0 + 64u * (uint32_t)(d >> 1)) + (uint32_t)(d & 1) + 2u * (uint32_t)lane;
          tn += (uint32_t)__popcll(mt);
          qn += (uint32_t)__popcll(md & ~mt);
        }
      }
    }
    // resolve 64 entries (one per lane) at a time, at the end the rest
    while (qn >= 64u || tn >= 64u || rn >= 64u || hn >= 64u ||
           (!more && (qn | tn | rn | hn) != 0u)) {
      // (whole passes first; hard ones last, as they are few and long)
      const int which = hn >= 64u || rn >= 64u ? (hn > rn ? 2 : 1)
                        : tn >= 64u            ? 3
                        : qn != 0u             ? 0
                        : tn != 0u             ? 3
                        : rn != 0u             ? 1
                                               : 2;
      const uint32_t m = which == 0   ? min(qn, 64u)
                         : which == 3 ? min(tn, 64u)
                         : which == 1 ? min(min(rn, 64u), (uint32_t)kHardRing - hn)
                                      : min(min(hn, 64u), (uint32_t)kHardRing - rn);
      wave_sync();
      int64_t j = 0;
      uint32_t code = kTailTaken;
      uint64_t e = 0;  // the draw's number, the attempt from bit 32 on
      if ((uint32_t)lane < m) {
        bool tail = true;
        uint64_t mu = 0;
        if (which == 0) {
          const uint32_t i = ring[qn - 1u - (uint32_t)lane];
          const Words4 w = philox4x32_10(i >> 1, rep, cs, 0u, ck0, ck1);
          mu = (i & 1u) ? m53(w.w2, w.w3) : m53(w.w0, w.w1);
          tail = false;
          e = i;
        } else if (which == 3) {
          e = ring[(uint32_t)kBatchRing - tn + (uint32_t)lane];
        } else {
          const uint32_t p = ((which == 2 ? hh : rh) + (uint32_t)lane) & (uint32_t)(kHardRing - 1);
          e = which == 2 ? hard[p] : retry[p];
        }
        if (tail) {
          const uint32_t attempt = (uint32_t)(e >> 32);
          const TailTry t = which == 2
                                ? tail_hard(m0, beta, gm, ck0, ck1, (uint32_t)e, rep, cs, attempt)
                                : tail_try(m0, beta, gm, ck0, ck1, (uint32_t)e, rep, cs, attempt);
          code = t.code;
          j = t.X - off;
          if (code == kTailCapped) fl |= kFlagTailCapped;
        } else if (mu > timax) {
          // its first word is the last threshold's: a tail draw after all
          code = kTailFirst;
        } else {
          j = (int64_t)lds_search(mu, T, guide, sh);
        }
      }
      if (which == 2) {
        hh += m;
        hn -= m;
      } else if (which == 1) {
        rh += m;
        rn -= m;
      } else if (which == 3) {
        tn -= m;
      } else {
        qn -= m;
      }
      const uint64_t mr =
          __ballot(code == kTailRejected || code == kTailCapped || code == kTailFirst);
      if (mr != 0ull) {
        const uint32_t p = place_below(mr, rh + rn) & (uint32_t)(kHardRing - 1);
        if ((mr >> lane) & 1ull) retry[p] = code == kTailFirst ? e : e + (1ull << 32);
        rn += (uint32_t)__popcll(mr);
      }
      const uint64_t mh = __ballot(code == kTailHard);
      if (mh != 0ull) {
        const uint32_t p = place_below(mh, hh + hn) & (uint32_t)(kHardRing - 1);
        if (code == kTailHard) hard[p] = e;
        hn += (uint32_t)__popcll(mh);
      }
      if (code != kTailTaken) j = 0;
      if (j >= 1 && j <= kHW) {
        lds_inc(&hist[j - 1]);
        xm = max(xm, 4u * (uint32_t)j - 4u);
      }
      put_big(j);
    }
    if (!more) break;
    j0 += 64u * kWaveBlocks;
#pragma unroll
    for (int d = 0; d < 4; ++d) wh[d] = nh[d];
  }
  DrawOut o;
  o.fl = dpp_or_u32(fl);
  o.ovn = ovn;
  const int hi = ((int)min((dpp_max_u32(xm) >> 2) + 1u, (uint32_t)kHW) + 255) & ~255;
  o.hi = hi < 256 ? 256 : hi;
  wave_sync();
  const uint32_t c1 = dpp_sum_u32(hist[kWaveOwn + lane]);
  const uint32_t c2 = dpp_sum_u32(hist[kWaveOwn + 64 + lane]);
  const uint32_t c3 = dpp_sum_u32(hist[kWaveOwn + 128 + lane]);
  if (lane == 0) {
    hist[0] += c1;  // the rings' draws count 1..3 into the bins themselves
    hist[1] += c2;
    hist[2] += c3;
  }
  wave_sync();
  return o;
}

// Counts of one replicate to scratch, and the exact sum of ln v 2^53 over its
// draws (as sums of the low and the high words) with, when want_fp, the
// multiset fingerprint.
struct SumOut {
  uint64_t lo, hi, fp;
};
static __device__ __noinline__ SumOut sum_replicate(const LdsU32* hist, int hi_, uint32_t* cp_,
                                                    bool wide_, const int64_t* ov_, uint32_t oc_,
                                                    int64_t off_, bool want_fp_,
                                                    const double* ln_) {
  const int lane = lane_id();
  const int hi = __builtin_amdgcn_readfirstlane(hi_);
  const uint32_t oc = (uint32_t)__builtin_amdgcn_readfirstlane((int)oc_);
  const int64_t off = uniform64(off_);
  const bool wide = __builtin_amdgcn_readfirstlane((int)wide_) != 0;
  const bool want_fp = __builtin_amdgcn_readfirstlane((int)want_fp_) != 0;
  uint32_t* __restrict__ cp = as_global(reinterpret_cast<uint32_t*>(uniform64((int64_t)cp_)));
  const int64_t* __restrict__ ov = as_global(reinterpret_cast<const int64_t*>(uniform64((int64_t)ov_)));
  const double* __restrict__ ln = as_global(reinterpret_cast<const double*>(uniform64((int64_t)ln_)));
  uint64_t slo = 0, shi = 0, fp = 0;
  for (int b0 = 0; b0 < hi; b0 += 256) {
    uint32_t cs[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) cs[k] = hist[b0 + 4 * lane + k];
    if (wide)
      *reinterpret_cast<uint4*>(cp + b0 + 4 * lane) = uint4{cs[0], cs[1], cs[2], cs[3]};
    else
      *reinterpret_cast<uint2*>(cp + (b0 >> 1) + 2 * lane) =
          uint2{cs[0] | (cs[1] << 16), cs[2] | (cs[3] << 16)};
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int64_t v = off + b0 + 4 * lane + k + 1;
      if (__ballot(cs[k] != 0u) != 0ull) {
        const uint64_t lf = ln_fixed_at(v, ln);
        slo += (uint64_t)cs[k] * (uint32_t)lf;
        shi += (uint64_t)cs[k] * (uint32_t)(lf >> 32);
        if (want_fp) fp += (uint64_t)cs[k] * mix64((uint64_t)v);
      }
    }
  }
  if (oc != 0u) wave_sync_global();  // read back by other lanes than the writers
  for (uint32_t p = (uint32_t)lane; p < oc; p += 64u) {
    const int64_t v = off + ov[-1 - (int64_t)p];
    const uint64_t lf = ln_fixed_at(v, ln);
    slo += (uint32_t)lf;
    shi += lf >> 32;
    if (want_fp) fp += mix64((uint64_t)v);
  }
  SumOut o;
  o.lo = dpp_sum_u64(slo);
  o.hi = dpp_sum_u64(shi);
  o.fp = want_fp ? dpp_sum_u64(fp) : 0ull;
  return o;
}

// MLE and the values up to 16 of the KS, one replicate per lane: alpha_hat,
// 1 / normaliser, zeta(a, 17) and the largest term over those values.  D is
// final (done) where no larger value can reach it, and under the truncated law
// below trunc_em's range (K < 161) or on a short support, whose whole KS runs here.
struct HeadOut {
  double a, iz, z16, D;
  uint32_t flags, done;
};
// The distinct values of stored counts 1..K, K <= kHW, as ks_distance_trunc takes
// them.  Read 16 bytes at a time: the lanes' replicates lie 2 KiB apart, and a
// load for every value took longer than the terms.
struct CountSrc {
  CountView cv;
  uint32_t K;
  uint32_t v;      // next value above 16
  uint64_t lo, hi;  // counts of v and up, as far as they are read
  __device__ __forceinline__ void load(int b) {  // from bin b, a multiple of 8
    const uint4 w = *reinterpret_cast<const uint4*>(cv.wide ? cv.p + b : cv.p + (b >> 1));
    lo = (uint64_t)w.y << 32 | w.x;
    hi = (uint64_t)w.w << 32 | w.z;
  }
  __device__ __forceinline__ uint32_t small(int x) {  // x = 1..16 in order
    if (cv.wide) return (uint32_t)x <= K ? cv.at(x - 1) : 0u;
    if ((x & 7) == 1) load(x - 1);
    const uint32_t c = (uint32_t)((((x - 1) & 4) ? hi : lo) >> (16 * ((x - 1) & 3))) & 0xffffu;
    return (uint32_t)x <= K ? c : 0u;
  }
  __device__ __forceinline__ bool next_large(int64_t& x, uint32_t& c) {
    const int bits = cv.wide ? 32 : 16;
    while (v <= K) {
      if (((v - 1u) & (cv.wide ? 3u : 7u)) == 0u) load((int)v - 1);
      c = cv.wide ? (uint32_t)lo : (uint32_t)lo & 0xffffu;
      lo = lo >> bits | hi << (64 - bits);
      hi >>= bits;
      x = (int64_t)v++;
      if (c) return true;
    }
    return false;
  }
};
template <int kLaw>
static __device__ __noinline__ HeadOut head_lane(U128 S, int64_t n, int64_t xmin, uint32_t K,
                                                 const uint32_t* counts_, bool wide,
                                                 uint32_t flags, const double* ln_) {
  const uint32_t* counts = as_global(counts_);
  const double* __restrict__ ln = as_global(ln_);
  HeadOut o;
  o.flags = flags;
  o.done = 0u;
  const CountView cv{counts, wide};
  double suf[17];
  if constexpr (kLaw == kCutoff) {
    U128 Sx = {0, 0};
    u128_add_mul(Sx, (uint64_t)n, ln_fixed(xmin, ln));
    if (S.lo == Sx.lo && S.hi == Sx.hi) {  // every value at the cutoff: one counts as xmin + 1
      S = U128{0, 0};
      u128_add_mul(S, (uint64_t)(n - 1), ln_fixed(xmin, ln));
      u128_add(S, ln_fixed(xmin + 1, ln), 0);
      o.flags |= kFlagAllOnes;
    }
    o.a = mle_alpha_hz(u128_to_S(S) / (double)n, xmin, ln, &o.flags);
    const EmCoef E = em_coef(o.a);
    survival_head_cut(E, ln, suf);
    double zx = 0.0;
#pragma unroll
    for (int t = 1; t <= 16; ++t)
      if (xmin - 1 == t) zx = suf[t];
    if (xmin > 17) zx = survival_rel(E, xmin - 1, xmin);
    o.iz = 1.0 / zx;
  } else {
    double Sd;
    if (S.lo == 0 && S.hi == 0) {  // every draw was 1: S := ln 2
      Sd = ln[2];
      o.flags |= kFlagAllOnes;
    } else {
      Sd = u128_to_S(S);
    }
    if constexpr (kLaw == kTrunc) {
      o.a = mle_alpha_trunc(Sd / (double)n, K, ln, &o.flags);
      // (many lanes at once: their walks over a short support cost less than a
      // wave for each replicate.  12 exponents of 50,000 replicates, K = 100, n = 50:
      // 1,213 and 1,314 us; K = 160, n = 100: 1,929 and 1,692.)
      if (!trunc_em(o.a, K) || (K <= kTruncLaneK && __popcll(__ballot(true)) >= 16)) {
        CountSrc src{cv, K, 17, 0, 0};
        o.D = ks_distance_trunc(src, o.a, K, n, ln);
        o.iz = 1.0;
        o.z16 = 0.0;
        o.done = 1u;
        return o;
      }
      const EmCoef E = em_coef(o.a);
      survival_head_trunc(E, trunc_end(E, K, ln), ln, suf);
    } else {
      o.a = mle_alpha_start(Sd / (double)n, ln, mle_guess_table(ln), &o.flags);
      survival_head(em_coef(o.a), ln, suf);
    }
    o.iz = 1.0 / suf[0];
  }
  o.z16 = suf[16];
  const double idn = 1.0 / (double)n;
  const int off = kLaw == kCutoff ? (int)(xmin < 17 ? xmin - 1 : 16) : 0;
  uint32_t c16[16];  // read ahead of the terms' branches
#pragma unroll
  for (int v = 1; v <= 16; ++v) {
    const uint32_t t = cv.at(v > off ? v - 1 - off : 0);
    c16[v - 1] = v > off ? t : 0u;
  }
  int64_t C = 0;
  double D = 0.0;
#pragma unroll
  for (int v = 1; v <= 16; ++v) {
    const uint32_t cn = c16[v - 1];
    if (cn) {
      const double t2 = fabs(fma(suf[v - 1], o.iz, -(double)(n - C) * idn));
      C += cn;
      const double t1 = fabs(fma(suf[v], o.iz, -(double)(n - C) * idn));
      D = fmax(D, fmax(t1, t2));
    }
  }
  o.D = D;
  // past 16 both distributions lie between their values there and 1
  if (fmax(o.z16 * o.iz, (double)(n - C) * idn) <= D - kPruneMargin) o.done = 1u;
  return o;
}

// Replicates r0 .. r0 + nrep - 1 of a cell by one wave, in batches that fill
// its scratch (`stride` int64): 64 records, then the counts of each replicate
// from below and the draws above kHW from the end.  A replicate is begun while
// c.room of those still fit (all n of them, or what the cell's replicates
// hardly ever exceed); one that exceeds the rest after all is drawn again as
// the first of the next batch, or goes to the escalation list if it was.
template <bool kCut, int kKernel>
__device__ __forceinline__ void replicate_batch(const DevCell* cells, int32_t cell_id,
                                                int64_t r0, int nrep, BatchLds* L, int64_t* scratch,
                                                int64_t stride, int lane,
                                                const uint32_t* __restrict__ T,
                                                const uint32_t* __restrict__ guide,
                                                const double* __restrict__ ln, const Outputs& out,
                                                uint64_t* esc_list, uint32_t* esc_count,
                                                uint32_t esc_cap, uint32_t* err) {
  const DevCell& c = cells[cell_id];
  const int64_t n = c.n;
  const bool wide = n >= 65536;
  const int64_t cw = count_words(n);
  constexpr int64_t kRecords = kBatchRecords;
  WaveSlot* slots = reinterpret_cast<WaveSlot*>(scratch);
  int64_t* counts = scratch + kRecords;
  const int64_t off = kCut ? c.xmin - 1 : 0;
  const bool want_fp = out.fp != nullptr;
  const int64_t want = (int64_t)c.room + part_words(c.room);
  int hi = kHW;  // the region's LDS held other data
  int done = 0;
  while (done < nrep) {
    int q = 0;
    bool full = false;
    int64_t top = stride;  // the larger draws of the next replicate lie below it
    while (done + q < nrep && q < 64 && !full &&
           (q == 0 || top - (kRecords + (q + 1) * cw) >= want)) {
      const uint32_t rep = (uint32_t)(r0 + done + q);
      const uint32_t room = (uint32_t)min(top - (kRecords + (q + 1) * cw), n);
      const DrawOut dr = draw_replicate<kCut, kKernel>(&c, rep, (LdsU32*)L->hist, (LdsU32*)L->ring,
                                              (LdsU64*)L->retry, (LdsU64*)L->hard, scratch + top, room,
                                              (const LdsU32*)T, (const LdsU32*)guide, hi);
      hi = dr.hi;
      full = dr.ovn > room;
      if (full && q > 0) break;
      const uint32_t no = full ? 0u : dr.ovn;
      const SumOut su = sum_replicate((const LdsU32*)L->hist, hi,
                                      reinterpret_cast<uint32_t*>(counts + q * cw), wide,
                                      scratch + top, no, off, want_fp, ln);
      if (lane == 0) {
        WaveSlot sl;
        sl.S = U128{su.lo + (su.hi << 32),
                    (su.hi >> 32) + (su.lo + (su.hi << 32) < su.lo ? 1u : 0u)};
        sl.fp = su.fp;
        sl.top = top;
        sl.hi = (uint32_t)hi;
        sl.len = no;
        sl.flags = dr.fl;
        sl.esc = full ? 1u : 0u;
        slots[q] = sl;
      }
      top -= no;
      ++q;
    }
    wave_sync_global();  // the batch's records, counts and draws, before they are read back
    HeadOut h = {2.0, 1.0, 0.0, 0.0, 0u, 1u};
    uint32_t esc = 0, oc = 0, hib = 256;
    uint64_t fp = 0;
    int64_t ovtop = 0;
    if (lane < q) {
      const WaveSlot sl = slots[lane];
      esc = sl.esc;
      oc = sl.len;
      hib = sl.hi;
      fp = sl.fp;
      ovtop = sl.top;
      const uint32_t* cnt = reinterpret_cast<const uint32_t*>(counts + lane * cw);
      if (esc == 0u) {
        if constexpr (kCut)
          h = head_lane<kCutoff>(sl.S, n, c.xmin, 0u, cnt, wide, sl.flags, ln);
        else if (c.K)
          h = head_lane<kTrunc>(sl.S, n, 1, c.K, cnt, wide, sl.flags, ln);
        else
          h = head_lane<kPure>(sl.S, n, 1, 0u, cnt, wide, sl.flags, ln);
      }
    }
    // the rest of the KS, one replicate per wave
    const bool part = oc > (uint32_t)kPartMin;
    const uint64_t parted = __ballot(h.done == 0u && part);
    if (parted != 0ull) {
      auto many = [&](auto fn) {
        return fn(parted, h.a, h.iz, h.D, h.z16, &c, scratch, q, top, (LdsU32*)L->hist, ln);
      };
      if constexpr (kCut)
        h.D = many([](auto... x) { return ks_parted<kCutoff>(x...); });
      else if (c.K)
        h.D = many([](auto... x) { return ks_parted<kTrunc>(x...); });
      else
        h.D = many([](auto... x) { return ks_parted<kPure>(x...); });
    }
    uint64_t left = __ballot(h.done == 0u && !part);
    while (left != 0ull) {
      const int i = __ffsll((long long)left) - 1;
      left &= left - 1ull;
      const int64_t tp =
          ((int64_t)__builtin_amdgcn_readlane((int)(ovtop >> 32), i) << 32) |
          (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)ovtop, i);
      auto rest = [&](auto fn) {
        return fn(readlane_f64(h.a, i), readlane_f64(h.iz, i), c.xmin, c.K,
                  reinterpret_cast<const uint32_t*>(counts + i * cw), wide,
                  __builtin_amdgcn_readlane((int)hib, i), scratch + tp,
                  (uint32_t)__builtin_amdgcn_readlane((int)oc, i), n, readlane_f64(h.D, i),
                  readlane_f64(h.z16, i), (LdsU32*)L->hist, (LdsU64*)L->ring, (LdsU32*)L->retry,
                  (LdsU64*)L->hard, ln);
      };
      double Di;
      if constexpr (kCut)
        Di = rest([](auto... x) { return ks_rest<kCutoff>(x...); });
      else if (c.K)
        Di = c.K <= (uint32_t)kHW ? rest([](auto... x) { return ks_rest<kTrunc, false>(x...); })
                                  : rest([](auto... x) { return ks_rest<kTrunc>(x...); });
      else
        Di = rest([](auto... x) { return ks_rest<kPure>(x...); });
      if (lane == i) h.D = Di;
    }
    // the bin tables of larger draws went through the histogram
    if (__ballot(h.done == 0u && oc != 0u) != 0ull) hi = kHW;
    if (lane < q) {
      const int64_t rep = r0 + done + lane;
      if (esc != 0u) {
        const uint32_t slot = atomicAdd(esc_count, 1u);
        if (slot < esc_cap)
          esc_list[slot] = ((uint64_t)(uint32_t)cell_id << 32) | (uint32_t)rep;
        else
          atomicOr(err, kErrEscOverflow);
      } else {
        write_outputs(out, c.out_off + rep, h.D, h.a, h.flags, fp);
      }
    }
    wave_sync_global();  // the next batch overwrites the records
    done += q;
  }
}

// The cell's table and guide, and a region per wave.
template <class Region, int kWavesPer>
struct KernelLds {
  alignas(16) uint32_t T[2 * kH];  // floor(F(k) 2^53): threshold_hi, then threshold_lo
  uint32_t guide[kGuide];
  Region w[kWavesPer];
  int unit;
};
union SimRegion {
  LaneRegion lane;
  BatchLds batch;
};
static_assert(sizeof(KernelLds<SimRegion, kWaves>) <= 160 * 1024, "one workgroup per compute unit");

// Takes the next unit of a queue for the whole workgroup and stages its cell's
// table when that changes; false when the queue is empty.
template <class Lds>
__device__ __forceinline__ bool next_unit(Lds& L, uint32_t* queue, const Unit* __restrict__ units,
                                          int n_units, const DevCell* __restrict__ cells,
                                          const double* __restrict__ tables,
                                          const uint16_t* __restrict__ guides, int& loaded,
                                          Unit& un, int nthreads) {
  const int tid = (int)threadIdx.x;
  __syncthreads();  // the previous unit's table is no longer read
  if (tid == 0) L.unit = (int)atomicAdd(queue, 1u);
  __syncthreads();
  const int u = L.unit;
  if (u >= n_units) return false;
  un = units[u];
  if (un.cell != loaded) {
    load_cell_tables(L.T, L.guide, tables + (size_t)un.cell * kH,
                     guides + (size_t)un.cell * (kGuide + 1), cells[un.cell], tid, nthreads);
    loaded = un.cell;
    __syncthreads();
  }
  return true;
}

// Persistent simulation kernel: workgroups pull units from two queues, first
// those of the lane form (up to kBlock replicates of a cell, one per lane;
// workgroups 0 .. lane_wgs - 1), then those of the wave and heavy forms (each
// wave a contiguous share; the last batch_wgs workgroups, see SimGrid).  Both kinds in one
// launch: one after the other each would end on a device that runs dry.
// Three waves per SIMD: the twelve waves' LDS regions and the shared table
// fit one workgroup per compute unit, and the register budget is 168 per lane.
static_assert(kBlock == 64 * kWaves && kWaves == kBatchWaves, "twelve waves per workgroup");
__global__ __launch_bounds__(kBlock, 3) void k_simulate(
    SimGrid g, const DevCell* __restrict__ cells, const double* __restrict__ tables,
    const uint16_t* __restrict__ guides, const double* __restrict__ ln,
    const Unit* __restrict__ lane_units, int n_lane, const Unit* __restrict__ batch_units,
    int n_batch, uint32_t* lane_queue, uint32_t* batch_queue, uint32_t* big_queue, Outputs out,
    uint64_t* esc_list, uint32_t* esc_count, uint32_t esc_cap, int64_t* scratch, uint32_t* err) {
  __shared__ KernelLds<SimRegion, kWaves> L;
  const int wave = (int)threadIdx.x >> 6;
  const int lane = lane_id();
  int loaded = -1;
  Unit un;
  if ((int)blockIdx.x < g.lane_wgs) {
    int64_t* mine = scratch + (int64_t)blockIdx.x * g.lane_area + (int64_t)wave * kLaneScratch;
    while (next_unit(L, lane_queue, lane_units, n_lane, cells, tables, guides, loaded, un,
                     kBlock)) {
      const int first = wave * 64;
      if (first < un.count)
        lane_wave(cells, un.cell, un.r0 + first, un.count - first < 64 ? un.count - first : 64,
                  &L.w[wave].lane, lane, L.T, L.guide, ln, out, esc_list, esc_count, esc_cap, err,
                  mine);
    }
  }
  const int b = (int)blockIdx.x - (g.grid - g.batch_wgs);
  if (b < 0) return;
  // workgroups with scratch for the longest replicates take those first
  bool big = b < g.big_wgs;
  const int waves = big ? g.big_waves : g.waves;
  const int64_t stride = big ? g.big_stride : g.stride;
  int64_t* mine = scratch + wave * stride +
                  (big ? g.big_area + (int64_t)b * waves * stride
                       : g.rest + (int64_t)(b - g.big_wgs) * g.area);
  for (;;) {
    if (!next_unit(L, big ? big_queue : batch_queue, big ? batch_units : batch_units + g.n_big,
                   big ? g.n_big : n_batch - g.n_big, cells, tables, guides, loaded, un, kBlock)) {
      if (!big) return;
      big = false;
      continue;
    }
    const int share = (un.count + waves - 1) / waves;
    const int first = wave * share;
    if (wave < waves && first < un.count)
      replicate_batch<false, 0>(cells, un.cell, un.r0 + first,
                             un.count - first < share ? un.count - first : share,
                             &L.w[wave].batch, mine, stride, lane, L.T, L.guide, ln, out,
                             esc_list, esc_count, esc_cap, err);
  }
}

// The cells with a lower cutoff (heavy form).
__global__ __launch_bounds__(64 * kBatchWavesCut, kBatchWavesCut / 4) void k_cutoff(
    const DevCell* __restrict__ cells, const double* __restrict__ tables,
    const uint16_t* __restrict__ guides, const double* __restrict__ ln,
    const Unit* __restrict__ units, int n_units, uint32_t* queue, Outputs out,
    uint64_t* esc_list, uint32_t* esc_count, uint32_t esc_cap, int64_t* scratch, int waves,
    int64_t stride, uint32_t* err) {
  __shared__ KernelLds<BatchLds, kBatchWavesCut> L;
  const int wave = (int)threadIdx.x >> 6;
  const int lane = lane_id();
  int64_t* mine = scratch + ((int64_t)blockIdx.x * waves + wave) * stride;
  int loaded = -1;
  Unit un;
  while (next_unit(L, queue, units, n_units, cells, tables, guides, loaded, un,
                   64 * kBatchWavesCut)) {
    const int share = (un.count + waves - 1) / waves;
    const int first = wave * share;
    if (wave < waves && first < un.count)
      replicate_batch<true, 1>(cells, un.cell, un.r0 + first,
                            un.count - first < share ? un.count - first : share, &L.w[wave], mine,
                            stride, lane, L.T, L.guide, ln, out, esc_list, esc_count, esc_cap, err);
  }
}

// The replicates on the escalation list, with scratch for a replicate's every
// draw: a workgroup takes `waves` of them at a time (at most kEscWaves), those of
// the same cell side by side.
__global__ __launch_bounds__(64 * kEscWaves, kEscWaves / 4) void k_escalated(
    const DevCell* __restrict__ cells, const double* __restrict__ tables,
    const uint16_t* __restrict__ guides, const double* __restrict__ ln, uint32_t* queue,
    Outputs out, uint64_t* esc_list, uint32_t* esc_count, uint32_t esc_cap, int64_t* scratch,
    int waves, int64_t stride, uint32_t* err) {
  __shared__ KernelLds<BatchLds, kEscWaves> L;
  const int tid = (int)threadIdx.x;
  const int wave = tid >> 6;
  const int lane = tid & 63;
  int64_t* mine = scratch + ((int64_t)blockIdx.x * waves + wave) * stride;
  const uint32_t ne = *esc_count < esc_cap ? *esc_count : esc_cap;
  int loaded = -1;
  for (;;) {
    if (tid == 0) L.unit = (int)atomicAdd(queue, (uint32_t)waves);
    __syncthreads();
    const uint32_t e0 = (uint32_t)L.unit;
    if (e0 >= ne) break;
    const uint32_t e1 = e0 + (uint32_t)waves < ne ? e0 + (uint32_t)waves : ne;
    for (uint32_t e = e0; e < e1;) {
      const int cell = (int)(esc_list[e] >> 32);
      uint32_t same = 1;
      while (e + same < e1 && (int)(esc_list[e + same] >> 32) == cell) ++same;
      const DevCell c = cells[cell];
      if (cell != loaded) {
        __syncthreads();
        load_cell_tables(L.T, L.guide, tables + (size_t)cell * kH,
                         guides + (size_t)cell * (kGuide + 1), c, tid, 64 * kEscWaves);
        loaded = cell;
        __syncthreads();
      }
      if ((uint32_t)wave < same) {
        const int64_t r0 = (int64_t)(uint32_t)esc_list[e + (uint32_t)wave];
        if (c.xmin > 1)
          replicate_batch<true, 2>(cells, cell, r0, 1, &L.w[wave], mine, stride, lane, L.T, L.guide,
                                   ln, out, esc_list, esc_count, 0u, err);
        else
          replicate_batch<false, 2>(cells, cell, r0, 1, &L.w[wave], mine, stride, lane, L.T,
                                    L.guide, ln, out, esc_list, esc_count, 0u, err);
      }
      e += same;
    }
    __syncthreads();
  }
}

}  // namespace zpl
