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

// Support values are handled as the table index j = v - (xmin - 1) (v itself
// for the pure law): 1..kHW in the LDS histogram, larger ones in the wave's
// global scratch.
struct alignas(16) BatchLds {
  // bins j = 1..kHW, a pad slot per lane, three rows of per-lane counts of
  // j = 1..3 (the wave form's layout); the bucket table of the larger draws
  // during the KS
  uint32_t hist[kHW + 64 + 3 * 64];
  uint64_t ring[kRing];  // deferred draws; the gathered draws during the KS
};

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
__device__ __forceinline__ uint32_t wave_incl_scan32(uint32_t v, int lane) {
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const uint32_t o = (uint32_t)__shfl_up((int)v, d, 64);
    if (lane >= d) v += o;
  }
  return v;
}
// Inclusive sum within each group of 16 lanes.
__device__ __forceinline__ uint32_t row_incl_scan32(uint32_t v, int lane) {
#pragma unroll
  for (int d = 1; d < 16; d <<= 1) {
    const uint32_t o = (uint32_t)__shfl_up((int)v, d, 16);
    if ((lane & 15) >= d) v += o;
  }
  return v;
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
// first jh values (those up to 16, taken from the head sums), and z16 =
// zeta(a, 17).  cv: the counts of j = 1..hi (hi a multiple of 256, zero
// above); ov[-1 - p], p < oc: the draws above kHW.  Negative when a bucket in
// reach of the maximum holds more than kGather draws (the caller redoes the
// replicate another way).
template <bool kCut>
__device__ __forceinline__ double ks_rest(const KsLaw<kCut>& w, const CountView& cv, int hi,
                                          const int64_t* __restrict__ ov, uint32_t oc, int64_t n,
                                          double D0, double z16, int jh, BatchLds* L,
                                          const double* __restrict__ ln, int lane) {
  const double idn = 1.0 / (double)n;
  const int64_t off = kCut ? w.xmin - 1 : 0;
  const uint32_t nu = (uint32_t)n;
  const uint64_t below = lanes_below(lane);
  double D = D0;
  // 1. the histogram in 64 chunks of 16 values, one per lane
  uint32_t last = 0, sum = 0;
  if (16 * lane < hi) sum = cv.sum16(lane, last);
  const uint32_t Cr = wave_incl_scan32(sum, lane), Cl = Cr - sum;
  const double zr = w.survival(off + 16 * (lane + 1), ln);  // right edge of the chunk
  {
    const double z = zr * w.iz, s = (double)(nu - Cr) * idn;
    const double Dlow = fmax(D, wave_max_f64(fabs(z - s)));
    double zl = shfl_f64(z, lane > 0 ? lane - 1 : 0), sl = (double)(nu - Cl) * idn;
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
      const uint32_t Ca = (uint32_t)__shfl((int)Cl, pc, 64) + row_incl_scan32(cnt, lane);
      const int64_t v = off + b + 1;
      const double zv = w.survival(v, ln);
      double zp = shfl_f64(zv, lane > 0 ? lane - 1 : 0);
      uint32_t cp = (uint32_t)__shfl_up((int)cnt, 1, 64);
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
    D = wave_max_f64(D);
  }
  if (oc == 0u) return D;
  // 2. the larger draws: none can matter when their whole mass is below D
  const double zE = readlane_f64(zr, 63);
  if (fmax(zE * w.iz, (double)oc * idn) <= D - kPruneMargin) return D;
  const bool has_top = __builtin_amdgcn_readlane((int)last, 63) != 0;  // j = kHW was drawn
  const uint32_t nbody = nu - oc;
  uint32_t* tab = L->hist;
  wave_sync();
  for (int k = lane; k < kHW; k += 64) tab[k] = 0u;
  wave_sync();
  for (uint32_t p = (uint32_t)lane; p < oc; p += 64u)
    atomicAdd(&tab[bucket_of((uint64_t)ov[-1 - (int64_t)p])], 1u);
  wave_sync();
  // an octave per lane, then the buckets of the octaves in reach, four
  // octaves per round; a bucket in reach keeps an entry, the others zero
  uint32_t total = 0;
  {
    const bool oct = lane < (kBuckets >> kBucketBits);
    uint32_t cs = 0;
    if (oct) {
      const uint4* q = reinterpret_cast<const uint4*>(tab + 16 * lane);
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const uint4 t = q[k];
        cs += t.x + t.y + t.z + t.w;
      }
    }
    const uint32_t cr = wave_incl_scan32(cs, lane), cl = cr - cs;
    const int64_t tr = (int64_t)min((uint64_t)off + bucket_end(16 * (oct ? lane : 52) + 15),
                                    (uint64_t)INT64_MAX);
    const double zo = w.survival(tr, ln) * w.iz;
    const double s = (double)(oc - cr) * idn;
    double Dlow = fmax(D, wave_max_f64(fabs(zo - s)));
    double zl = shfl_f64(zo, lane > 0 ? lane - 1 : 0);
    if (lane == 0) zl = zE * w.iz;
    const bool need = cs != 0u && fmax(zl - s, (double)(oc - cl) * idn - zo) > Dlow - kPruneMargin;
    uint64_t mask = __ballot(need);
    if (oct && cs != 0u && !need) {
      uint4* q = reinterpret_cast<uint4*>(tab + 16 * lane);
#pragma unroll
      for (int k = 0; k < 4; ++k) q[k] = uint4{0u, 0u, 0u, 0u};
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
      const uint32_t ca = (uint32_t)__shfl((int)cl, pc, 64) + row_incl_scan32(cnt, lane);
      const int64_t t = (int64_t)min((uint64_t)off + bucket_end(b), (uint64_t)INT64_MAX);
      const double z = w.survival(t, ln) * w.iz;
      const double sb = (double)(oc - ca) * idn;
      double zp = shfl_f64(z, lane > 0 ? lane - 1 : 0);
      const double zq = shfl_f64(zl, pc);
      if ((lane & 15) == 0) zp = zq;
      Dlow = fmax(Dlow, wave_max_f64(p < 0 ? 0.0 : fabs(z - sb)));
      const bool in = cnt != 0u &&
                      fmax(zp - sb, (double)(oc - (ca - cnt)) * idn - z) > Dlow - kPruneMargin;
      if (p >= 0) tab[b] = in ? bucket_entry(cnt, ca - cnt) : 0u;
      total += in ? cnt : 0u;
    }
    total = wave_sum_u32(total);
  }
  wave_sync();
  // 3. the draws of the buckets in reach, gathered into LDS: in one pass when
  // they fit, else a window of buckets at a time.  A draw equal to the value
  // just below a gathered bucket is gathered as well (it decides a term).
  uint64_t* list = L->ring;
  int wlo = 0;
  while (total != 0u && wlo < kBuckets) {
    int whi = kBuckets;
    if (total > (uint32_t)kGather) {
      const uint32_t e = wlo + lane < kBuckets ? tab[wlo + lane] : 0u;
      const uint32_t c = (e >> 31) ? ((e >> 22) & 511u) : 0u;
      const uint32_t cum = wave_incl_scan32(c, lane);
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
        if (take && pos < (uint32_t)kRing) list[pos] = j;
        m += (uint32_t)__popcll(mt);
      }
    }
    if (m > (uint32_t)kRing) return -1.0;
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
  return wave_max_f64(D);
}

// ln x 2^53 as an integer, from the context's table behind the logarithms.
__device__ __forceinline__ const uint64_t* ln_fixed_table(const double* ln) {
  return reinterpret_cast<const uint64_t*>(ln + kH + 2);
}
__device__ __forceinline__ uint64_t ln_fixed_at(int64_t v, const double* __restrict__ ln) {
  return v <= (int64_t)(kH + 1) ? ln_fixed_table(ln)[v] : (uint64_t)(log((double)v) * 0x1p53);
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
  auto drain = [&](int m) {
    wave_sync();
    int64_t j = 0;
    if (lane < m) {
      uint32_t p = qh + (uint32_t)lane;
      if (p >= (uint32_t)kRing) p -= (uint32_t)kRing;
      const uint64_t e = L->ring[p];
      if (e >> 63) {
        const double m0 = kCut ? (double)(c.xmin + kH) : kTailM;
        j = tail_draw_from(m0, c.beta, c.gm, c.k0, c.k1, (uint32_t)e, rep, c.stream, &fl);
        if constexpr (kCut) j -= c.xmin - 1;
      } else {
        j = (int64_t)slow_search(e & ((1ull << 53) - 1), T, guide, sh);
      }
      if (j <= kHW) atomicAdd(&L->hist[j - 1], 1u);
    }
    xm = max(xm, j <= kHW ? (int)j : 0);
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
    ring_append(L->ring, qh, qn, def, [&](int d) {
      return defer_entry(U[d], timax,
                         2u * (j0 + 64u * (uint32_t)(d >> 1) + (uint32_t)lane) + (uint32_t)(d & 1),
                         0);
    }, lane);
    while (qn >= 64u) {
      drain(64);
      qh = qh + 64u >= (uint32_t)kRing ? qh + 64u - (uint32_t)kRing : qh + 64u;
      qn -= 64u;
    }
#pragma unroll
    for (int d = 0; d < 2 * kWaveBlocks; ++d) U[d] = Un[d];
  }
  if (qn > 0u) drain((int)qn);
  fl = wave_or_u32(fl);
  hi = ((int)min(wave_max_i64((int64_t)xm), (int64_t)kHW) + 255) & ~255;
  hi = hi < 256 ? 256 : hi;
  wave_sync();
  const uint32_t c1 = wave_sum_u32(L->hist[kWaveOwn + lane]);
  const uint32_t c2 = wave_sum_u32(L->hist[kWaveOwn + 64 + lane]);
  const uint32_t c3 = wave_sum_u32(L->hist[kWaveOwn + 128 + lane]);
  if (lane == 0) {
    L->hist[0] += c1;  // drains count 1..3 into the bins themselves
    L->hist[1] += c2;
    L->hist[2] += c3;
  }
  wave_sync();
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
      slo = wave_sum_u64(slo);
      shi = wave_sum_u64(shi);
      if (want_fp) fp = wave_sum_u64(fp);
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
    double a = 2.0, D = 0.0, iz = 1.0, z16 = 0.0;
    uint32_t flags = 0, esc = 0, oc = 0, hib = 256;
    uint64_t fp = 0;
    int64_t ovtop = 0;
    const int jh = off < 16 ? 16 - (int)off : 0;
    if (lane < q) {
      const WaveSlot sl = slots[lane];
      flags = sl.flags;
      esc = sl.esc;
      oc = sl.len;
      hib = sl.off;
      fp = sl.fp;
      ovtop = sl.xmax;
      const CountView cv{reinterpret_cast<const uint32_t*>(counts + lane * cw), wide};
      double suf[17];
      if constexpr (kCut) {
        U128 S = sl.S, Sx = {0, 0};
        u128_add_mul(Sx, (uint64_t)n, ln_fixed(c.xmin, ln));
        if (S.lo == Sx.lo && S.hi == Sx.hi) {  // every value at the cutoff: one counts as xmin + 1
          S = U128{0, 0};
          u128_add_mul(S, (uint64_t)(n - 1), ln_fixed(c.xmin, ln));
          u128_add(S, ln_fixed(c.xmin + 1, ln), 0);
          flags |= kFlagAllOnes;
        }
        a = mle_alpha_hz(u128_to_S(S) / (double)n, c.xmin, ln, &flags);
        const EmCoef E = em_coef(a);
        survival_head_cut(E, ln, suf);
        double zx = 0.0;
#pragma unroll
        for (int t = 1; t <= 16; ++t)
          if (c.xmin - 1 == t) zx = suf[t];
        if (c.xmin > 17) zx = survival_rel(E, c.xmin - 1, c.xmin);
        iz = 1.0 / zx;
      } else {
        double Sd;
        if (sl.S.lo == 0 && sl.S.hi == 0) {  // every draw was 1: S := ln 2
          Sd = ln[2];
          flags |= kFlagAllOnes;
        } else {
          Sd = u128_to_S(sl.S);
        }
        a = mle_alpha(Sd / (double)n, ln, &flags);
        survival_head(em_coef(a), ln, suf);
        iz = 1.0 / suf[0];
      }
      z16 = suf[16];
      const double idn = 1.0 / (double)n;
      int64_t C = 0;
#pragma unroll
      for (int v = 1; v <= 16; ++v) {
        const int b = v - 1 - (int)(kCut ? (off < 16 ? off : 16) : 0);
        const uint32_t cn = b >= 0 && b < jh ? cv.at(b < 0 ? 0 : b) : 0u;
        if (cn) {
          const double t2 = fabs(fma(suf[v - 1], iz, -(double)(n - C) * idn));
          C += cn;
          const double t1 = fabs(fma(suf[v], iz, -(double)(n - C) * idn));
          D = fmax(D, fmax(t1, t2));
        }
      }
    }
    // the rest of the KS, one replicate per wave
    for (int i = 0; i < q; ++i) {
      if (__builtin_amdgcn_readlane((int)esc, i) != 0) continue;
      KsLaw<kCut> w;
      w.E = em_coef(readlane_f64(a, i));
      w.iz = readlane_f64(iz, i);
      w.xmin = kCut ? c.xmin : 1;
      const CountView cv{reinterpret_cast<const uint32_t*>(counts + i * cw), wide};
      const int64_t tp =
          ((int64_t)__builtin_amdgcn_readlane((int)(ovtop >> 32), i) << 32) |
          (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)ovtop, i);
      const double Di = ks_rest<kCut>(
          w, cv, __builtin_amdgcn_readlane((int)hib, i), scratch + tp,
          (uint32_t)__builtin_amdgcn_readlane((int)oc, i), n, readlane_f64(D, i),
          readlane_f64(z16, i), jh, L, ln, lane);
      if (lane == i) D = Di;
    }
    hi = kHW;  // the bucket tables went through the histogram
    if (lane < q) {
      const int64_t rep = r0 + done + lane;
      if (esc != 0u || D < 0.0) {
        const uint32_t slot = atomicAdd(esc_count, 1u);
        if (slot < esc_cap)
          esc_list[slot] = ((uint64_t)(uint32_t)cell_id << 32) | (uint32_t)rep;
        else
          atomicOr(err, kErrEscOverflow);
      } else {
        write_outputs(out, c.out_off + rep, D, a, flags, fp, 0);
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
