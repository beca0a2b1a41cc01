// zpl_batch.hpp -- replicates by whole waves in batches, without sorting.
//
// A wave draws a batch of replicates one after another.  Of each it keeps the
// exact sum of logarithms, the counts of the first 1,024 support values and
// the larger draws unsorted.  The MLE of the batch then runs one replicate
// per lane, and the KS distance (eq. 3) one replicate per wave, by bounds:
// between two points l < r of the support every |F - S_n| is at most
// max(F(r) - S_n(l), S_n(r) - F(l)), so an interval whose bound does not reach
// a distance already found elsewhere holds no maximum and its values are not
// looked at.  What remains is evaluated exactly as the list walk of
// ks_distance does (the same terms, hence the same D bit for bit).
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
// for the pure law): 1..kHW in the LDS histogram, larger ones in the wave's
// global scratch.
//
// Deferred draws wait in two rings and are resolved 64 at a time.  A tail draw
// makes one proposal per pass; a rejected one goes back into the ring with its
// next attempt, one that needs a double-double floor into the second ring, so
// that a wave runs that long path with all its lanes (at alpha = 1.2 one
// proposal in 80 needs it, which was half of all passes).  The first ring
// holds fewer than 64 entries before an iteration's at most 256, and a pass
// of either ring puts back at most what it takes out, but for at most 64 that
// come from the second: 384.
constexpr int kBatchRing = 384;
constexpr int kHardRing = 128;
struct alignas(16) BatchLds {
  // bins j = 1..kHW, a pad slot per lane, three rows of per-lane counts of
  // j = 1..3 (the wave form's layout); the bucket table of the larger draws
  // during the KS
  uint32_t hist[kHW + 64 + 3 * 64];
  uint64_t ring[kBatchRing];  // deferred draws; the gathered draws during the KS
  uint64_t hard[kHardRing];   // tail proposals whose floor FP64 does not decide
};

// LDS words as such (address space 3): the functions below are called, not
// inlined, so that their registers and constants do not crowd the draw loops
// around the calls, and through a generic pointer their LDS accesses would be
// flat ones, which are not ordered with the callers' LDS instructions.
typedef __attribute__((address_space(3))) uint32_t LdsU32;
typedef __attribute__((address_space(3))) uint64_t LdsU64;
__device__ __forceinline__ void lds_inc(LdsU32* p) {
  __hip_atomic_fetch_add(p, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}
__device__ __forceinline__ int64_t uniform64(int64_t v) {
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)v);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(v >> 32));
  return (int64_t)(((uint64_t)hi << 32) | lo);
}

// The larger draws' buckets: 16 per octave of j, j >= kHW.
constexpr int kBucketBits = 4;
constexpr int kBuckets = (63 - 10) << kBucketBits;  // octaves 10..62
static_assert(kHW == 1024 && kBuckets <= kHW, "the bucket table takes the histogram's place");
// Gathered draws per pass (the ring's room, less ghosts) and the largest count
// of one bucket; a replicate with a larger bucket in reach of the maximum goes
// to the heavy kernel.
constexpr int kGather = 256;

__device__ __forceinline__ int bucket_of(uint64_t j) {
  const int e = 63 - __clzll((long long)j);
  return ((e - 10) << kBucketBits) + (int)((j >> (e - kBucketBits)) & ((1u << kBucketBits) - 1u));
}
// Largest j of bucket b (up to 2^63 - 1).
__device__ __forceinline__ uint64_t bucket_end(int b) {
  const int e = 10 + (b >> kBucketBits);
  const uint64_t m = (uint64_t)(b & ((1 << kBucketBits) - 1)) + (1u << kBucketBits) + 1u;
  return (m << (e - kBucketBits)) - 1u;
}

// A flagged bucket's entry: bit 31, its count (9 bits, saturated), and the
// larger draws below it (22 bits).
constexpr int64_t kBatchMaxN = (int64_t)1 << 20;
__device__ __forceinline__ uint32_t bucket_entry(uint32_t count, uint32_t below) {
  return 0x80000000u | ((count > 511u ? 511u : count) << 22) | below;
}

// The law at alpha_hat as the KS needs it.
template <bool kCut>
struct KsLaw {
  EmCoef E;
  double iz;     // 1 / normaliser
  int64_t xmin;  // kCut: the cutoff
  // sum of k^-a over k > t (t >= 16), relative to xmin^-a for cutoffs above 17
  __device__ __forceinline__ double survival(int64_t t, const double* __restrict__ ln) const {
    if constexpr (kCut)
      return xmin > 17 ? survival_rel(E, t, xmin) : survival_next_cut(E, t, ln);
    else
      return survival_next(E, t, ln);
  }
  __device__ __forceinline__ double point(int64_t v, const double* __restrict__ ln) const {
    if constexpr (kCut)
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

// Distances closer than this to the largest one found are always evaluated:
// far above the rounding of a bound (a few 2^-53), far below any distance.
constexpr double kPruneMargin = 1e-12;

// D of one replicate by a whole wave, given D0, the largest term over the
// values up to 16 (the first jh, taken from the head sums), and z16 =
// zeta(a, 17).  counts: those of j = 1..hi (hi a multiple of 256, zero
// above); ov[-1 - p], p < oc: the draws above kHW.  Negative when a bucket in
// reach of the maximum holds more than kGather draws (the caller redoes the
// replicate another way).
template <bool kCut>
static __device__ __noinline__ double ks_rest(double a, double iz, int64_t xmin_,
                                              const uint32_t* counts, bool wide_, int hi_,
                                              const int64_t* ov_, uint32_t oc_, int64_t n_,
                                              double D0, double z16, LdsU32* tab, LdsU64* list,
                                              const double* ln_) {
  // every argument is the wave's
  const int lane = lane_id();
  const int64_t n = uniform64(n_);
  const int hi = __builtin_amdgcn_readfirstlane(hi_);
  const uint32_t oc = (uint32_t)__builtin_amdgcn_readfirstlane((int)oc_);
  const int64_t* __restrict__ ov = reinterpret_cast<const int64_t*>(uniform64((int64_t)ov_));
  const double* __restrict__ ln = reinterpret_cast<const double*>(uniform64((int64_t)ln_));
  const CountView cv{reinterpret_cast<const uint32_t*>(uniform64((int64_t)counts)),
                     __builtin_amdgcn_readfirstlane((int)wide_) != 0};
  KsLaw<kCut> w;
  w.E = em_coef(a);
  w.iz = iz;
  w.xmin = kCut ? uniform64(xmin_) : 1;
  const int jh = w.xmin < 17 ? 17 - (int)w.xmin : 0;
  const double idn = 1.0 / (double)n;
  const int64_t off = kCut ? w.xmin - 1 : 0;
  const uint32_t nu = (uint32_t)n;
  const uint64_t below = lanes_below(lane);
  double D = D0;
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
    const bool need = sum != 0u && 16 * (lane + 1) > jh &&
                      fmax(zl - s, sl - z) > Dlow - kPruneMargin;
    uint64_t mask = __ballot(need);
    // four chunks per round, one value per lane
    while (mask != 0ull) {
      int p = -1;
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const int q = mask != 0ull ? __ffsll((long long)mask) - 1 : -1;
        mask &= mask - 1ull;
        if ((lane >> 4) == g) p = q;
      }
      const int pc = p < 0 ? 0 : p;
      const int b = 16 * pc + (lane & 15);
      const uint32_t cnt = p < 0 ? 0u : cv.at(b);
      const uint32_t Ca = (uint32_t)__shfl((int)Cl, pc, 64) + row_incl_scan_u32(cnt);
      const int64_t v = off + b + 1;
      const double zv = w.survival(v, ln);
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
      if (cnt != 0u && b >= jh) {
        const double zv1 = cp != 0u ? zp : zv + w.point(v, ln);
        const double t2 = fabs(fma(zv1, w.iz, -(double)(nu - (Ca - cnt)) * idn));
        const double t1 = fabs(fma(zv, w.iz, -(double)(nu - Ca) * idn));
        D = fmax(D, fmax(t1, t2));
      }
    }
    D = dpp_max_f64(D);
  }
  if (oc == 0u) return D;
  // 2. the larger draws: none can matter when their whole mass is below D
  const double zE = readlane_f64(zr, 63);
  if (fmax(zE * w.iz, (double)oc * idn) <= D - kPruneMargin) return D;
  const bool has_top = __builtin_amdgcn_readlane((int)last, 63) != 0;  // j = kHW was drawn
  const uint32_t nbody = nu - oc;
  wave_sync();
  for (int k = lane; k < kHW; k += 64) tab[k] = 0u;
  wave_sync();
  for (uint32_t p = (uint32_t)lane; p < oc; p += 64u)
    lds_inc(&tab[bucket_of((uint64_t)ov[-1 - (int64_t)p])]);
  wave_sync();
  // an octave per lane, then the buckets of the octaves in reach, four
  // octaves per round; a bucket in reach keeps an entry, the others zero
  uint32_t total = 0;
  {
    const bool oct = lane < (kBuckets >> kBucketBits);
    uint32_t cs = 0;
    if (oct) {
#pragma unroll
      for (int k = 0; k < 16; ++k) cs += tab[16 * lane + k];
    }
    const uint32_t cr = dpp_incl_scan_u32(cs), cl = cr - cs;
    const int64_t tr = (int64_t)min((uint64_t)off + bucket_end(16 * (oct ? lane : 52) + 15),
                                    (uint64_t)INT64_MAX);
    const double zo = w.survival(tr, ln) * w.iz;
    const double s = (double)(oc - cr) * idn;
    double Dlow = fmax(D, dpp_max_f64(fabs(zo - s)));
    double zl = prev_lane_f64(zo);
    if (lane == 0) zl = zE * w.iz;
    const bool need = cs != 0u && fmax(zl - s, (double)(oc - cl) * idn - zo) > Dlow - kPruneMargin;
    uint64_t mask = __ballot(need);
    if (oct && cs != 0u && !need) {
#pragma unroll
      for (int k = 0; k < 16; ++k) tab[16 * lane + k] = 0u;
    }
    while (mask != 0ull) {
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
      const int64_t t = (int64_t)min((uint64_t)off + bucket_end(b), (uint64_t)INT64_MAX);
      const double z = w.survival(t, ln) * w.iz;
      const double sb = (double)(oc - ca) * idn;
      double zp = prev_lane_f64(z);
      const double zq = shfl_f64(zl, pc);
      if ((lane & 15) == 0) zp = zq;
      Dlow = fmax(Dlow, dpp_max_f64(p < 0 ? 0.0 : fabs(z - sb)));
      const bool in = cnt != 0u &&
                      fmax(zp - sb, (double)(oc - (ca - cnt)) * idn - z) > Dlow - kPruneMargin;
      if (p >= 0) tab[b] = in ? bucket_entry(cnt, ca - cnt) : 0u;
      total += in ? cnt : 0u;
    }
    total = dpp_sum_u32(total);
  }
  wave_sync();
  // 3. the draws of the buckets in reach, gathered into LDS: in one pass when
  // they fit, else a window of buckets at a time.  A draw equal to the value
  // just below a gathered bucket is gathered as well (it decides a term).
  int wlo = 0;
  while (total != 0u && wlo < kBuckets) {
    int whi = kBuckets;
    if (total > (uint32_t)kGather) {
      const uint32_t e = wlo + lane < kBuckets ? tab[wlo + lane] : 0u;
      const uint32_t c = (e >> 31) ? ((e >> 22) & 511u) : 0u;
      const uint32_t cum = dpp_incl_scan_u32(c);
      const uint64_t fit = __ballot(cum <= (uint32_t)kGather);
      const int take = fit == ~0ull ? 64 : __ffsll((long long)~fit) - 1;
      if (take == 0) return -1.0;  // one bucket above the room
      whi = wlo + take;
      if (__ballot(c != 0u && lane < take) == 0ull) {
        wlo = whi;
        continue;
      }
    }
    uint32_t m = 0;  // wave-uniform
    for (uint32_t p0 = 0; p0 < oc; p0 += 64u) {
      const uint32_t p = p0 + (uint32_t)lane;
      bool take = false;
      uint64_t j = 0;
      if (p < oc) {
        j = (uint64_t)ov[-1 - (int64_t)p];
        const int b = bucket_of(j), b1 = bucket_of(j + 1u);
        take = (b >= wlo && b < whi && (tab[b] >> 31) != 0u) ||
               (b1 != b && b1 >= wlo && b1 < whi && (tab[b1] >> 31) != 0u);
      }
      const uint64_t mt = __ballot(take);
      if (mt != 0ull) {
        const uint32_t pos = m + (uint32_t)__popcll(mt & below);
        if (take && pos < (uint32_t)kBatchRing) list[pos] = j;
        m += (uint32_t)__popcll(mt);
      }
    }
    if (m > (uint32_t)kBatchRing) return -1.0;
    wave_sync();
    for (uint32_t i0 = 0; i0 < m; i0 += 64u) {
      const uint32_t i = i0 + (uint32_t)lane;
      const bool valid = i < m;
      const uint64_t j = valid ? list[i] : (uint64_t)kHW + 1u;
      const int b = bucket_of(j);
      const uint32_t e = tab[b];
      const uint64_t jlo = b > 0 ? bucket_end(b - 1) + 1u : (uint64_t)kHW;
      uint32_t lt = 0, eq = 0, pres = j == (uint64_t)kHW + 1u && has_top ? 1u : 0u;
      for (uint32_t k = 0; k < m; ++k) {
        const uint64_t x = list[k];
        lt += (x >= jlo && x < j) ? 1u : 0u;
        eq += x == j ? 1u : 0u;
        pres |= x + 1u == j ? 1u : 0u;
      }
      if (valid && b >= wlo && b < whi && (e >> 31) != 0u) {
        const uint32_t Cb = nbody + (e & 0x3fffffu) + lt;
        const int64_t v = off + (int64_t)j;
        const double zv = w.survival(v, ln);
        const double zv1 = pres ? w.survival(v - 1, ln) : zv + w.point(v, ln);
        const double t2 = fabs(fma(zv1, w.iz, -(double)(nu - Cb) * idn));
        const double t1 = fabs(fma(zv, w.iz, -(double)(nu - Cb - eq) * idn));
        D = fmax(D, fmax(t1, t2));
      }
    }
    wave_sync();
    wlo = whi;
  }
  return dpp_max_f64(D);
}

// ln x 2^53 as an integer, from the context's table behind the logarithms.
__device__ __forceinline__ const uint64_t* ln_fixed_table(const double* ln) {
  return reinterpret_cast<const uint64_t*>(ln + kH + 2);
}
__device__ __forceinline__ uint64_t ln_fixed_at(int64_t v, const double* __restrict__ ln) {
  return v <= (int64_t)(kH + 1) ? ln_fixed_table(ln)[v] : (uint64_t)(log((double)v) * 0x1p53);
}

// One proposal of the tail sampler (tail_draw_from): taken (X), rejected,
// rejected above 2^63, or undecided in FP64 (tail_hard repeats it with the
// floor in double-double).  The last attempt that an entry can hold is taken
// as the sampler's last resort is (never reached: it would follow 2^21
// rejections).
constexpr uint32_t kTailAttempts = (1u << 21) - 1u;
constexpr uint32_t kTailTaken = 0, kTailRejected = 1, kTailCapped = 2, kTailHard = 3;
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

// The draws of replicate rep by one wave (the wave form's pipelined loop):
// counts of j <= kHW into L->hist (the rows of 1..3 added in at the end),
// larger ones to top[-1 - p], p < ovn, as far as `room` reaches (ovn counts
// them all).  On entry bins [0, hi) may be nonzero and are cleared; on return
// hi covers the bins that may be nonzero.
template <bool kCut>
__device__ __forceinline__ void draw_batch_replicate(const DevCell& c, uint32_t rep, BatchLds* L,
                                                     int64_t* __restrict__ top, uint32_t room,
                                                     int lane, const uint64_t* __restrict__ T,
                                                     const uint32_t* __restrict__ guide,
                                                     uint32_t& fl, uint32_t& ovn, int& hi) {
  const uint64_t below = lanes_below(lane);
  for (int k = lane; k < hi; k += 64) L->hist[k] = 0u;
#pragma unroll
  for (int k = 0; k < 3; ++k) L->hist[kWaveOwn + k * 64 + lane] = 0u;
  wave_sync();
  const uint32_t nblk = (uint32_t)((c.n + 1) >> 1);
  const uint32_t n32 = (uint32_t)c.n;
  const uint64_t timax = table_int(c.tmax);
  const int sh = (int)c.gsh;
  int xm = 0;
  fl = 0;
  ovn = 0;
  uint32_t qh = 0, qn = 0;  // deferred draws, wave-uniform
  // the value of one lane (j, or 0 for none) counted in converged code
  auto put_big = [&](int64_t j) {
    const uint64_t mb = __ballot(j > kHW);
    if (mb != 0ull) {
      const uint32_t pos = ovn + (uint32_t)__popcll(mb & below);
      if (j > kHW && pos < room) top[-1 - (int64_t)pos] = j;
      ovn += (uint32_t)__popcll(mb);
    }
  };
  uint32_t hh = 0, hn = 0;  // the second ring, wave-uniform
  auto wrap = [](uint32_t p, int size) { return p >= (uint32_t)size ? p - (uint32_t)size : p; };
  const double m0 = kCut ? (double)(c.xmin + kH) : kTailM;
  // resolves m entries (one per lane) of the ring, or of the second one
  auto drain = [&](uint32_t m, bool second) {
    wave_sync();
    int64_t j = 0;
    uint32_t code = kTailTaken;
    uint64_t e = 0;
    if ((uint32_t)lane < m) {
      e = second ? L->hard[wrap(hh + (uint32_t)lane, kHardRing)]
                 : L->ring[wrap(qh + (uint32_t)lane, kBatchRing)];
      if (e >> 63) {
        const TailTry t =
            second ? tail_hard(m0, c.beta, c.gm, c.k0, c.k1, (uint32_t)e, rep, c.stream,
                               (uint32_t)(e >> 32) & kTailAttempts)
                   : tail_try(m0, c.beta, c.gm, c.k0, c.k1, (uint32_t)e, rep, c.stream,
                              (uint32_t)(e >> 32) & kTailAttempts);
        code = t.code;
        j = kCut ? t.X - (c.xmin - 1) : t.X;
        if (code == kTailCapped) fl |= kFlagTailCapped;
      } else {
        j = (int64_t)slow_search(e & ((1ull << 53) - 1), T, guide, sh);
      }
    }
    if (second) {
      hh = wrap(hh + m, kHardRing);
      hn -= m;
    } else {
      qh = wrap(qh + m, kBatchRing);
      qn -= m;
    }
    const uint64_t mr = __ballot(code == kTailRejected || code == kTailCapped);
    if (mr != 0ull) {
      if ((mr >> lane) & 1ull)
        L->ring[wrap(wrap(qh + qn, kBatchRing) + (uint32_t)__popcll(mr & below), kBatchRing)] =
            e + (1ull << 32);
      qn += (uint32_t)__popcll(mr);
    }
    const uint64_t mh = __ballot(code == kTailHard);
    if (mh != 0ull) {
      if (code == kTailHard)
        L->hard[wrap(wrap(hh + hn, kHardRing) + (uint32_t)__popcll(mh & below), kHardRing)] = e;
      hn += (uint32_t)__popcll(mh);
    }
    if (code != kTailTaken) j = 0;
    if (j >= 1 && j <= kHW) {
      atomicAdd(&L->hist[j - 1], 1u);
      xm = max(xm, (int)j);
    }
    put_big(j);
  };
  auto gen = [&](uint32_t j0, uint64_t (&Uo)[2 * kWaveBlocks]) {
    uint32_t k0 = c.k0, k1 = c.k1;  // round keys per block (see lane_wave)
    asm volatile("" : "+s"(k0), "+s"(k1));
#pragma unroll
    for (int b = 0; b < kWaveBlocks; ++b) {
      const Words4 w = philox4x32_10(j0 + 64u * (uint32_t)b + (uint32_t)lane, rep, c.stream, 0u,
                                     k0, k1);
      Uo[2 * b] = m53(w.w0, w.w1);
      Uo[2 * b + 1] = m53(w.w2, w.w3);
    }
  };
  uint64_t U[2 * kWaveBlocks];
  int gi[2 * kWaveBlocks];
  gen(0u, U);
#pragma unroll
  for (int d = 0; d < 2 * kWaveBlocks; ++d) gi[d] = guide_index(U[d], sh);
  for (uint32_t j0 = 0; j0 < nblk; j0 += 64u * kWaveBlocks) {
    uint32_t gg[2 * kWaveBlocks];
#pragma unroll
    for (int d = 0; d < 2 * kWaveBlocks; ++d) gg[d] = guide[gi[d]];
    uint64_t Un[2 * kWaveBlocks] = {1ull, 1ull, 1ull, 1ull};
    if (j0 + 64u * kWaveBlocks < nblk) gen(j0 + 64u * kWaveBlocks, Un);  // none past the end
    asm volatile("" : "+v"(Un[0]), "+v"(Un[1]), "+v"(Un[2]), "+v"(Un[3]));  // made here
    uint64_t t[2 * kWaveBlocks];
#pragma unroll
    for (int d = 0; d < 2 * kWaveBlocks; ++d) t[d] = T[(int)(gg[d] & 0xffffu) - 1];
    __builtin_amdgcn_sched_barrier(0);  // the table reads issue before the index math
#pragma unroll
    for (int d = 0; d < 2 * kWaveBlocks; ++d) gi[d] = guide_index(Un[d], sh);
    asm volatile("" : "+v"(gi[0]), "+v"(gi[1]), "+v"(gi[2]), "+v"(gi[3]));  // made here
    asm volatile("" : "+v"(t[0]), "+v"(t[1]), "+v"(t[2]), "+v"(t[3]));  // reads stay unconditional
    int x[2 * kWaveBlocks];
    bool def[2 * kWaveBlocks];
    bool big = false;
#pragma unroll
    for (int d = 0; d < 2 * kWaveBlocks; ++d) {
      const int xd = fast_select(gg[d], t[d], U[d]);
      const uint32_t i =
          2u * (j0 + 64u * (uint32_t)(d >> 1) + (uint32_t)lane) + (uint32_t)(d & 1);
      const bool valid = i < n32;
      const bool drawn = xd < kDeferred;
      x[d] = valid && drawn ? xd : -1;
      def[d] = valid && !drawn;
      big = big || x[d] > kHW;
      const uint32_t xm1 = (uint32_t)(x[d] - 1);
      const int slot = xm1 < 3u ? kWaveOwn + (int)xm1 * 64 + lane
                                : (xm1 < (uint32_t)kHW ? (int)xm1 : kWavePad + lane);
      atomicAdd(&L->hist[slot], 1u);
      xm = max(xm, x[d]);  // values above kHW are clamped once, below
    }
    if (__ballot(big) != 0ull) {
#pragma unroll
      for (int d = 0; d < 2 * kWaveBlocks; ++d) put_big((int64_t)x[d]);
    }
    ring_append<2 * kWaveBlocks, kBatchRing>(L->ring, qh, qn, def, [&](int d) {
      return defer_entry(U[d], timax,
                         2u * (j0 + 64u * (uint32_t)(d >> 1) + (uint32_t)lane) + (uint32_t)(d & 1),
                         0);
    }, lane);
    while (qn >= 64u || hn >= 64u) {
      const bool second = hn >= 64u;
      drain(64u, second);
    }
#pragma unroll
    for (int d = 0; d < 2 * kWaveBlocks; ++d) U[d] = Un[d];
  }
  while (qn > 0u || hn > 0u) {
    const bool second = hn >= 64u || qn == 0u;
    drain(min(second ? hn : qn, 64u), second);
  }
  fl = dpp_or_u32(fl);
  hi = ((int)min(dpp_max_u32((uint32_t)xm), (uint32_t)kHW) + 255) & ~255;
  hi = hi < 256 ? 256 : hi;
  wave_sync();
  const uint32_t c1 = dpp_sum_u32(L->hist[kWaveOwn + lane]);
  const uint32_t c2 = dpp_sum_u32(L->hist[kWaveOwn + 64 + lane]);
  const uint32_t c3 = dpp_sum_u32(L->hist[kWaveOwn + 128 + lane]);
  if (lane == 0) {
    L->hist[0] += c1;  // drains count 1..3 into the bins themselves
    L->hist[1] += c2;
    L->hist[2] += c3;
  }
  wave_sync();
}

// MLE and the values up to 16 of the KS, one replicate per lane: alpha_hat,
// 1 / normaliser, zeta(a, 17) and the largest term over those values.
struct HeadOut {
  double a, iz, z16, D;
  uint32_t flags;
};
template <bool kCut>
static __device__ __noinline__ HeadOut head_lane(U128 S, int64_t n, int64_t xmin,
                                                 const uint32_t* counts, bool wide,
                                                 uint32_t flags, const double* __restrict__ ln) {
  HeadOut o;
  o.flags = flags;
  const CountView cv{counts, wide};
  double suf[17];
  if constexpr (kCut) {
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
    o.a = mle_alpha(Sd / (double)n, ln, &o.flags);
    survival_head(em_coef(o.a), ln, suf);
    o.iz = 1.0 / suf[0];
  }
  o.z16 = suf[16];
  const double idn = 1.0 / (double)n;
  const int off = kCut ? (int)(xmin < 17 ? xmin - 1 : 16) : 0;
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
  return o;
}

// Replicates r0 .. r0 + nrep - 1 of a cell by one wave, in batches that fill
// its scratch (`stride` int64): 64 records, then the counts of each replicate
// from below and the draws above kHW from the end.  The heavy layout's stride
// holds at least one replicate's n draws and counts; more replicates join
// while n draws still fit.  A replicate that the KS cannot finish within LDS
// goes to the escalation list.
template <bool kCut>
__device__ __forceinline__ void replicate_batch(const DevCell& c, int32_t cell_id, int64_t r0,
                                                int nrep, BatchLds* L, int64_t* scratch,
                                                int64_t stride, int lane,
                                                const uint64_t* __restrict__ T,
                                                const uint32_t* __restrict__ guide,
                                                const double* __restrict__ ln, const Outputs& out,
                                                uint64_t* esc_list, uint32_t* esc_count,
                                                uint32_t esc_cap, uint32_t* err) {
  const int64_t n = c.n;
  const bool wide = n >= 65536;
  const int64_t cw = wide ? kHW / 2 : kHW / 4;  // int64 per replicate's counts
  constexpr int64_t kRecords = 64 * (int64_t)kWaveSlotBytes / 8;
  WaveSlot* slots = reinterpret_cast<WaveSlot*>(scratch);
  int64_t* counts = scratch + kRecords;
  const int64_t off = kCut ? c.xmin - 1 : 0;
  const bool want_fp = out.fp != nullptr;
  int hi = kHW;  // the region's LDS held other data
  int done = 0;
  while (done < nrep) {
    int q = 0;
    int64_t top = stride;  // the larger draws of the next replicate lie below it
    while (done + q < nrep && q < 64 && (q == 0 || top - (kRecords + (q + 1) * cw) >= n)) {
      const uint32_t rep = (uint32_t)(r0 + done + q);
      uint32_t fl, ovn;
      const uint32_t room = (uint32_t)min(top - (kRecords + (q + 1) * cw), n);
      draw_batch_replicate<kCut>(c, rep, L, scratch + top, room, lane, T, guide, fl, ovn, hi);
      // counts to scratch; exact sums of the low and high words of ln x 2^53
      uint32_t* cp = reinterpret_cast<uint32_t*>(counts + q * cw);
      uint64_t slo = 0, shi = 0, fp = 0;
      for (int b0 = 0; b0 < hi; b0 += 256) {
        const uint4 h = *reinterpret_cast<const uint4*>(L->hist + b0 + 4 * lane);
        if (wide)
          *reinterpret_cast<uint4*>(cp + b0 + 4 * lane) = h;
        else
          *reinterpret_cast<uint2*>(cp + (b0 >> 1) + 2 * lane) =
              uint2{h.x | (h.y << 16), h.z | (h.w << 16)};
        const uint32_t cs[4] = {h.x, h.y, h.z, h.w};
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
      const uint32_t no = ovn < room ? ovn : room;
      if (no != 0u) wave_sync_global();  // read back by other lanes than the writers
      for (uint32_t p = (uint32_t)lane; p < no; p += 64u) {
        const int64_t v = off + scratch[top - 1 - (int64_t)p];
        const uint64_t lf = ln_fixed_at(v, ln);
        slo += (uint32_t)lf;
        shi += lf >> 32;
        if (want_fp) fp += mix64((uint64_t)v);
      }
      slo = dpp_sum_u64(slo);
      shi = dpp_sum_u64(shi);
      if (want_fp) fp = dpp_sum_u64(fp);
      if (lane == 0) {
        WaveSlot sl;
        sl.S = U128{slo + (shi << 32), (shi >> 32) + (slo + (shi << 32) < slo ? 1u : 0u)};
        sl.fp = fp;
        sl.xmax = top;
        sl.off = (uint32_t)hi;
        sl.len = no;
        sl.flags = fl;
        sl.esc = ovn > room ? 1u : 0u;
        slots[q] = sl;
      }
      top -= no;
      ++q;
    }
    wave_sync_global();  // the batch's records, counts and draws, before they are read back
    // MLE and the head of the KS, one replicate per lane
    HeadOut h = {2.0, 1.0, 0.0, 0.0, 0u};
    uint32_t esc = 0, oc = 0, hib = 256;
    uint64_t fp = 0;
    int64_t ovtop = 0;
    if (lane < q) {
      const WaveSlot sl = slots[lane];
      esc = sl.esc;
      oc = sl.len;
      hib = sl.off;
      fp = sl.fp;
      ovtop = sl.xmax;
      h = head_lane<kCut>(sl.S, n, c.xmin, reinterpret_cast<const uint32_t*>(counts + lane * cw),
                          wide, sl.flags, ln);
    }
    // the rest of the KS, one replicate per wave
    for (int i = 0; i < q; ++i) {
      if (__builtin_amdgcn_readlane((int)esc, i) != 0) continue;
      const int64_t tp =
          ((int64_t)__builtin_amdgcn_readlane((int)(ovtop >> 32), i) << 32) |
          (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)ovtop, i);
      const double Di = ks_rest<kCut>(
          readlane_f64(h.a, i), readlane_f64(h.iz, i), c.xmin,
          reinterpret_cast<const uint32_t*>(counts + i * cw), wide,
          __builtin_amdgcn_readlane((int)hib, i), scratch + tp,
          (uint32_t)__builtin_amdgcn_readlane((int)oc, i), n, readlane_f64(h.D, i),
          readlane_f64(h.z16, i), (LdsU32*)L->hist, (LdsU64*)L->ring, ln);
      if (lane == i) h.D = Di;
    }
    hi = kHW;  // the bucket tables went through the histogram
    if (lane < q) {
      const int64_t rep = r0 + done + lane;
      if (esc != 0u || h.D < 0.0) {
        const uint32_t slot = atomicAdd(esc_count, 1u);
        if (slot < esc_cap)
          esc_list[slot] = ((uint64_t)(uint32_t)cell_id << 32) | (uint32_t)rep;
        else
          atomicOr(err, kErrEscOverflow);
      } else {
        write_outputs(out, c.out_off + rep, h.D, h.a, h.flags, fp, 0);
      }
    }
    wave_sync_global();  // the next batch overwrites the records
    done += q;
  }
}

// Persistent kernel of the batched replicates: a workgroup takes a unit (up
// to 64 replicates of one cell for each of its waves) from the queue and gives each
// wave a contiguous share.
template <int kWavesPer>
struct BatchKernelLds {
  alignas(16) uint64_t T[kH];  // floor(F(k) 2^53)
  uint32_t guide[kGuide];
  BatchLds w[kWavesPer];
  int unit;
};
static_assert(sizeof(BatchKernelLds<kBatchWaves>) <= 160 * 1024, "one workgroup per compute unit");

template <bool kCut, int kWavesPer>
__global__ __launch_bounds__(64 * kWavesPer, kWavesPer / 4) void k_batch(
    const DevCell* __restrict__ cells, const double* __restrict__ tables,
    const uint16_t* __restrict__ guides, const double* __restrict__ ln,
    const Unit* __restrict__ units, int n_units, uint32_t* queue, Outputs out,
    uint64_t* esc_list, uint32_t* esc_count, uint32_t esc_cap, int64_t* scratch, int64_t stride,
    uint32_t* err) {
  __shared__ BatchKernelLds<kWavesPer> L;
  const int tid = (int)threadIdx.x;
  const int wave = tid >> 6;
  const int lane = tid & 63;
  int64_t* mine = scratch + ((int64_t)blockIdx.x * kWavesPer + wave) * stride;
  int loaded = -1;
  for (;;) {
    if (tid == 0) L.unit = (int)atomicAdd(queue, 1u);
    __syncthreads();
    const int u = L.unit;
    if (u >= n_units) break;
    const Unit un = units[u];
    const DevCell c = cells[un.cell];
    if (un.cell != loaded) {
      load_cell_tables(L.T, L.guide, tables + (size_t)un.cell * kH,
                       guides + (size_t)un.cell * (kGuide + 1), c, tid, 64 * kWavesPer);
      loaded = un.cell;
      __syncthreads();
    }
    const int share = (un.count + kWavesPer - 1) / kWavesPer;
    const int first = wave * share;
    if (first < un.count)
      replicate_batch<kCut>(c, un.cell, un.r0 + first,
                            un.count - first < share ? un.count - first : share, &L.w[wave], mine,
                            stride, lane, L.T, L.guide, ln, out, esc_list, esc_count, esc_cap, err);
    __syncthreads();
  }
}

}  // namespace zpl
