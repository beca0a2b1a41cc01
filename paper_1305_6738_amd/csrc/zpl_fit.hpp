// zpl_fit.hpp -- fits of datasets (eq. 2 and eq. 3), and the scan over lower
// cutoffs.
//
// A dataset becomes the counts of the values 1..kFitBins and the sorted larger
// values.  Both give every count S_n needs by position, so no list of distinct
// values is built: C(v) is a prefix sum of the counts or the place of v's last
// copy in the sorted array.  The distance's terms are those of the
// replicates (the same expressions, hence the same bits), spread over all waves; their
// maximum does not depend on the order.
//
// Small datasets take one workgroup from the data to the result (k_fit_block), or,
// with few enough candidate cutoffs, one per candidate (k_fit_cand<true>).
// Other scans are counted and sorted once, by one workgroup or, from kFitGridMin
// values on, as larger fits are, by many (k_fit_count, k_fit_merge, k_fit_runs), and
// then finished per candidate cutoff (k_fit_cand<false>).
//
// Included by zpl_kernels.hip after zpl_batch.hpp.
#pragma once

namespace zpl {

constexpr int kFitBins = kH;        // values counted by value
constexpr int kFitThreads = 512;    // k_fit_block, k_fit_merge
constexpr int kFitCandThreads = 256;
constexpr int kFitRun = 4096;       // values sorted in LDS at a time
// From this size on many workgroups count and sort; at most kFitGroups, of at
// least kFitChunkMin values each.  A fit by one workgroup and by the grid (us,
// from the device): alpha 2.2, 32,768 values 41 and 49, 65,536 49 and 50,
// 131,072 65 and 53; alpha 1.7, 55 and 56, 65 and 57, 95 and 64.  Heavier tails
// cross earlier (more than kFitRun larger values leave LDS in the one).
constexpr int64_t kFitGridMin = 32768;
constexpr int64_t kFitChunkMin = 8192;
constexpr int kFitGroups = 512;
static_assert(kFitGroups <= kFitThreads, "k_fit_merge: a thread per group");
// Datasets of up to kFitSmall values are counted and sorted by the workgroup of each
// of up to kFitAlone candidates, two to a compute unit: one launch instead of two
// (1,000 values, one candidate 46.5 and 41.2 us, 128 of them 79.7 and 75.1; 1,000
// candidates take as long either way).
constexpr int kFitSmall = 1024;
constexpr int kFitAlone = 512;
constexpr int kFitShares = 64;      // workgroups that share one distance, at most
constexpr int kFitAcc = 128;        // candidates that may be shared
constexpr int kFitFan = 16;         // runs merged per pass
static_assert(kFitBins % (4 * kFitThreads) == 0, "whole 16-byte groups of bins per thread");

struct FitView {
  int64_t* g0;      // larger values as counted (a segment per workgroup); sorted passes alternate
  int64_t* g1;      // between g1 and g0
  uint32_t* slots;  // [groups][kFitBins] counts of each workgroup
  uint32_t* hist;   // [kFitBins] counts
  int64_t* meta;    // [groups][4] larger values, invalid flag, their sum of logarithms
  uint32_t* ctl;    // 0: larger values, 1: invalid, 2: g0 holds them sorted (else g1);
                    // 4..7: their sum of logarithms
  int64_t* acc;     // [kFitAcc][2] distance so far and finished workgroups of a candidate
};
__device__ __forceinline__ FitView fit_view(int64_t* base, int64_t n, int groups) {
  FitView f;
  f.g0 = base;
  f.g1 = f.g0 + n;
  int64_t* p = f.g1 + n;
  f.slots = reinterpret_cast<uint32_t*>(p);
  p += (int64_t)groups * (kFitBins / 2);
  f.hist = reinterpret_cast<uint32_t*>(p);
  p += kFitBins / 2;
  f.meta = p;
  p += (int64_t)groups * 4;
  f.ctl = reinterpret_cast<uint32_t*>(p);
  p += 8;
  f.acc = p;
  return f;
}

// Sum over the workgroup; part holds one entry per wave.  Every thread gets it.
template <int kThreads>
__device__ __forceinline__ U128 block_sum_u128(U128 v, U128* part) {
  v = wave_sum_u128(v);
  __syncthreads();
  if (lane_id() == 0) part[threadIdx.x >> 6] = v;
  __syncthreads();
  U128 s = {0, 0};
  for (int w = 0; w < kThreads / 64; ++w) u128_add(s, part[w].lo, part[w].hi);
  return s;
}

// cum[v] = values <= v (v = 0..kFitBins) from hist, both in LDS.
template <int kThreads>
__device__ __forceinline__ void fit_prefix(const uint32_t* hist, uint32_t* cum, uint32_t* part) {
  constexpr int kPer = kFitBins / kThreads;
  const int tid = (int)threadIdx.x, lane = lane_id(), wave = tid >> 6;
  uint32_t c[kPer], s = 0;
#pragma unroll
  for (int k = 0; k < kPer; k += 4) {
    const uint4 h = *reinterpret_cast<const uint4*>(hist + tid * kPer + k);
    c[k] = h.x;
    c[k + 1] = h.y;
    c[k + 2] = h.z;
    c[k + 3] = h.w;
  }
#pragma unroll
  for (int k = 0; k < kPer; ++k) s += c[k];
  const uint32_t inc = dpp_incl_scan_u32(s);
  if (lane == 63) part[wave] = inc;
  __syncthreads();
  uint32_t run = inc - s;
  for (int w = 0; w < wave; ++w) run += part[w];
  if (tid == 0) cum[0] = 0u;
#pragma unroll
  for (int k = 0; k < kPer; ++k) {
    run += c[k];
    cum[tid * kPer + k + 1] = run;
  }
  __syncthreads();
}

// Sum of logarithms of the counted values from xmin on (this thread's share).
template <int kThreads>
__device__ __forceinline__ U128 fit_bin_sum(const uint32_t* hist, int64_t xmin,
                                            const double* __restrict__ ln) {
  U128 S = {0, 0};
  for (int v = (int)threadIdx.x + 1; v <= kFitBins; v += kThreads) {
    const uint32_t c = hist[v - 1];
    if (c && v >= xmin) u128_add_mul(S, c, ln_fixed_table(ln)[v]);
  }
  return S;
}

__device__ __forceinline__ int64_t lower_bound_i64(const int64_t* __restrict__ a, int64_t lo,
                                                   int64_t hi, int64_t v) {
  while (lo < hi) {
    const int64_t mid = (lo + hi) >> 1;
    if (a[mid] < v)
      lo = mid + 1;
    else
      hi = mid;
  }
  return lo;
}

// What wave 0 hands the workgroup: the estimate, the normaliser and the sums
// of the first values.
constexpr int kFitDirect = 192;  // above every K that trunc_em refuses
static_assert(kFitDirect > 17 + 102 + 48 + 1, "em_start(64) = 113");
struct FitSolved {
  double a, iz;
  uint32_t flags;
  uint32_t em;               // truncated law by Euler-Maclaurin
  double suf[17];            // sums above 0..16
  double P[kFitDirect];      // truncated law, few values: partial sums from 1 on
};

// The laws of a fit, as the survival sums of their distances differ.
enum FitLaw { kFitPure, kFitCut, kFitCutRel, kFitTrunc, kFitTruncDirect };

// One wave: eq. 2 and the sums the distance starts from.  n values from xmin
// on with the sum of logarithms S; atmin: all of them equal xmin.
__device__ __forceinline__ void fit_solve(FitSolved* o, U128 S, int64_t n, int64_t xmin,
                                          uint32_t K, bool atmin, const double* __restrict__ ln) {
  const int lane = lane_id();
  uint32_t fl = 0;
  double a, iz, suf[17];
  if (xmin > 1) {
    if (atmin) {  // one value counts as xmin + 1
      S = U128{0, 0};
      u128_add_mul(S, (uint64_t)(n - 1), ln_fixed(xmin, ln));
      u128_add(S, ln_fixed(xmin + 1, ln), 0);
      fl |= kFlagAllOnes;
    }
    a = mle_alpha_hz(u128_to_S(S) / (double)n, xmin, ln, &fl);
    const EmCoef E = em_coef(a);
    survival_head_cut(E, ln, suf);
    double zx = 0.0;  // zeta(a, xmin) = suf[xmin - 1] (static indices: no scratch)
#pragma unroll
    for (int t = 1; t <= 16; ++t)
      if (xmin - 1 == t) zx = suf[t];
    // above 17 every value is: survival values relative to xmin^-a
    if (xmin > 17) zx = survival_rel(E, xmin - 1, xmin);
    iz = 1.0 / zx;
  } else {
    double Sd;
    if (S.lo == 0 && S.hi == 0) {  // every value is 1: S := ln 2
      Sd = ln[2];
      fl |= kFlagAllOnes;
    } else {
      Sd = u128_to_S(S);
    }
    if (K) {
      a = mle_alpha_trunc(Sd / (double)n, K, ln, &fl);
      const bool em = trunc_em(a, K);
      if (lane == 0) o->em = em ? 1u : 0u;
      if (em) {
        const EmCoef E = em_coef(a);
        survival_head_trunc(E, trunc_end(E, K, ln), ln, suf);
        iz = 1.0 / suf[0];
      } else {
        iz = 1.0 / zeta3_trunc(a, K, ln).z0;
        double pw[kDirect + 1];
        direct_powers(a, K, ln, pw);
#pragma unroll
        for (int k = 1; k <= kDirect; ++k)
          if (lane == 0) o->P[k] = pw[k];
        for (int k = kDirect + 1 + lane; k <= (int)K && k < kFitDirect; k += 64)
          o->P[k] = pow_neg(a, ln[k]);
        wave_sync();
        if (lane == 0) {  // in ascending order, as ks_distance_trunc sums them
          double P = 0.0;
          o->P[0] = 0.0;
          for (int k = 1; k <= (int)K && k < kFitDirect; ++k) {
            P += o->P[k];
            o->P[k] = P;
          }
        }
#pragma unroll
        for (int t = 0; t <= 16; ++t) suf[t] = 0.0;
      }
    } else {
      a = mle_alpha_start(Sd / (double)n, ln, mle_guess_table(ln), &fl);
      survival_head(em_coef(a), ln, suf);
      iz = 1.0 / suf[0];
    }
  }
  if (lane == 0) {
    o->a = a;
    o->iz = iz;
    o->flags = fl;
#pragma unroll
    for (int t = 0; t <= 16; ++t) o->suf[t] = suf[t];
  }
}

// This wave's share (wave gw of nw) of the distance over the n values from
// xmin on: the counted values in groups of 63, each lane one value and lane 0
// the one before them (its survival sum is the next value's lower term when
// both occur), then the sorted larger ones from p0 on.
template <int kLaw>
__device__ __forceinline__ double fit_ks(const FitSolved& f, const uint32_t* hist,
                                         const uint32_t* cum, const int64_t* __restrict__ ov,
                                         int64_t oc, int64_t p0, int64_t n, int64_t xmin,
                                         uint32_t K, int gw, int nw,
                                         const double* __restrict__ ln) {
  const int lane = lane_id();
  const double idn = 1.0 / (double)n, iz = f.iz;
  const EmCoef E = em_coef(f.a);
  TruncEnd te = {};
  if (kLaw == kFitTrunc) te = trunc_end(E, K, ln);
  auto upper = [&](int64_t v) -> double {
    if (kLaw == kFitCut) return survival_next_cut(E, v, ln);
    if (kLaw == kFitCutRel) return survival_rel(E, v, xmin);
    if (kLaw == kFitTrunc) return trunc_tail(E, te, v, ln[v + 1]);  // v <= K <= kH
    return survival_next(E, v, ln);
  };
  auto power = [&](int64_t v) -> double {
    return kLaw == kFitCutRel ? pow_rel(E.s, v, xmin) : pow_neg(E.s, ln_value(v, ln));
  };
  double D = 0.0;
  const int64_t below = xmin <= kFitBins + 1 ? (int64_t)cum[xmin - 1] : 0;
  const int top = K ? (int)K : kFitBins;
  if (xmin <= top) {
    for (int w = (int)((xmin - 1) / 63) + gw; w * 63 < top; w += nw) {
      const int v = 63 * w + lane;
      const uint32_t c = v >= xmin && v <= top ? hist[v - 1] : 0u;
      if (!__ballot(c != 0u && lane > 0)) continue;
      if (kLaw == kFitTruncDirect) {  // F(t) = P(t) / Z
        if (c && lane > 0) {
          const int64_t C = (int64_t)cum[v - 1];
          const double t2 = fabs(fma(f.P[v - 1], iz, -(double)C * idn));
          const double t1 = fabs(fma(f.P[v], iz, -(double)(C + c) * idn));
          D = fmax(D, fmax(t1, t2));
        }
        continue;
      }
      double zv = 0.0;
      if (c) zv = v <= 16 ? f.suf[v] : upper(v);
      const double zp = __shfl_up(zv, 1, 64);
      const uint32_t cp = (uint32_t)__shfl_up((int)c, 1, 64);
      if (c && lane > 0) {
        const double zv1 = v <= 17 ? f.suf[v - 1] : (cp ? zp : zv + power(v));
        const int64_t C = (int64_t)cum[v - 1] - below;
        const double t2 = fabs(fma(zv1, iz, -(double)(n - C) * idn));
        const double t1 = fabs(fma(zv, iz, -(double)(n - (C + c)) * idn));
        D = fmax(D, fmax(t1, t2));
      }
    }
  }
  if (kLaw == kFitPure || kLaw == kFitCut || kLaw == kFitCutRel) {
    // values before ov[0] counted from xmin on, or the ones to leave out
    const int64_t off = xmin <= kFitBins + 1 ? (int64_t)cum[kFitBins] - below : -p0;
    for (int64_t p = p0 + (int64_t)gw * 64 + lane; p < oc; p += (int64_t)nw * 64) {
      const int64_t v = ov[p];
      if (p + 1 < oc && ov[p + 1] == v) continue;  // not its last copy
      const int64_t first = p > p0 && ov[p - 1] == v ? lower_bound_i64(ov, p0, p, v) : p;
      const int64_t vp = first > p0 ? ov[first - 1] : (hist[kFitBins - 1] ? kFitBins : 0);
      const double zv = upper(v);
      const double zv1 = v - 1 == vp && vp >= xmin ? upper(v - 1) : zv + power(v);
      const double t2 = fabs(fma(zv1, iz, -(double)(n - (off + first)) * idn));
      const double t1 = fabs(fma(zv, iz, -(double)(n - (off + p + 1)) * idn));
      D = fmax(D, fmax(t1, t2));
    }
  }
  return wave_max_f64(D);
}

__device__ __forceinline__ double fit_ks_any(const FitSolved& f, const uint32_t* hist,
                                             const uint32_t* cum, const int64_t* __restrict__ ov,
                                             int64_t oc, int64_t p0, int64_t n, int64_t xmin,
                                             uint32_t K, int gw, int nw,
                                             const double* __restrict__ ln) {
  if (K)
    return f.em ? fit_ks<kFitTrunc>(f, hist, cum, ov, oc, p0, n, xmin, K, gw, nw, ln)
                : fit_ks<kFitTruncDirect>(f, hist, cum, ov, oc, p0, n, xmin, K, gw, nw, ln);
  return fit_ks<kFitPure>(f, hist, cum, ov, oc, p0, n, xmin, K, gw, nw, ln);
}

// Counts x[i0..i1) into hist (LDS, zeroed) and appends what is above the bins
// to ov; the ones (the most frequent value of these laws) are counted in a
// register.  Four loads per thread are in flight.
struct FitCount {
  U128 S;        // this thread's sum of logarithms of the larger values
  uint32_t bad;  // this thread saw a value outside 1..xhi
};
template <int kThreads>
__device__ __forceinline__ FitCount fit_count(const int64_t* __restrict__ x, int64_t i0,
                                              int64_t i1, int64_t xhi, uint32_t* hist,
                                              uint32_t* ovc, int64_t* ov,
                                              const double* __restrict__ ln) {
  constexpr int kUnroll = 8;
  FitCount r = {{0, 0}, 0u};
  uint32_t ones = 0;
  auto one = [&](int64_t v) {
    if (v == 1) {
      ++ones;
    } else if (v < 1 || v > xhi) {
      r.bad = 1u;
    } else if (v <= kFitBins) {
      atomicAdd(&hist[v - 1], 1u);
    } else {
      ov[atomicAdd(ovc, 1u)] = v;
      u128_add(r.S, ln_fixed(v, ln), 0);
    }
  };
  int64_t i = i0 + (int64_t)threadIdx.x;
  for (; i + (int64_t)(kUnroll - 1) * kThreads < i1; i += (int64_t)kUnroll * kThreads) {
    int64_t v[kUnroll];
#pragma unroll
    for (int k = 0; k < kUnroll; ++k) v[k] = x[i + (int64_t)k * kThreads];
#pragma unroll
    for (int k = 0; k < kUnroll; ++k) one(v[k]);
  }
  for (; i < i1; i += kThreads) one(x[i]);
  if (ones) atomicAdd(&hist[0], ones);
  return r;
}

// Ascending sort of a[0..P) (P a power of two) by the workgroup, in LDS or
// global memory.
template <class Ptr>
__device__ __forceinline__ void block_sort_pow2(Ptr a, int64_t P, int tid, int nt) {
  for (int64_t k = 2; k <= P; k <<= 1)
    for (int64_t j = k >> 1; j > 0; j >>= 1) {
      __syncthreads();
      for (int64_t i = tid; i < P / 2; i += nt) {
        const int64_t l = ((i & ~(j - 1)) << 1) | (i & (j - 1));  // the pair's lower index
        const int64_t u = a[l], w = a[l | j];
        if ((u > w) == ((l & k) == 0)) {
          a[l] = w;
          a[l | j] = u;
        }
      }
    }
  __syncthreads();
}

// One dataset per workgroup.  xs: datasets xs[i] of ns[i] values (a workgroup
// takes every gridDim-th and has its own scratch), or the one dataset x of n.
// kPrep: only the counts and the sorted larger values, for k_fit_cand.
// Bound by latency (loads, one wave's Newton step, the evaluations of the
// distance): a dataset of 5,000 values takes 15 us; with a list built and walked
// by one wave it took 20.
template <bool kPrep>
__global__ __launch_bounds__(kFitThreads) void k_fit_block(
    const int64_t* const* __restrict__ xs, const int64_t* __restrict__ ns, int n_sets,
    const int64_t* x1, int64_t n1, const double* __restrict__ ln, int64_t* scratch, int64_t stride,
    double* ahat_out, double* D_out, uint32_t* flags_out, uint32_t* status_out, uint32_t K) {
  __shared__ __align__(16) uint32_t hist[kFitBins];
  __shared__ uint32_t cum[kFitBins + 1];
  __shared__ int64_t sbuf[kFitRun];
  __shared__ FitSolved f;
  __shared__ U128 part[kFitThreads / 64];
  __shared__ uint32_t ovc, sbad;
  __shared__ uint32_t upart[kFitThreads / 64];
  __shared__ double dpart[kFitThreads / 64];
  const int tid = (int)threadIdx.x, lane = lane_id(), wave = tid >> 6;
  constexpr int kWaves = kFitThreads / 64;
  int64_t* base = scratch + (int64_t)blockIdx.x * stride;
  const int64_t xhi = K ? (int64_t)K : INT64_MAX;
  for (int set = (int)blockIdx.x; set < n_sets; set += (int)gridDim.x) {
    const int64_t* x = as_global(xs ? xs[set] : x1);
    const int64_t n = xs ? ns[set] : n1;
    for (int k = tid; k < kFitBins; k += kFitThreads) hist[k] = 0u;
    if (tid == 0) ovc = sbad = 0u;
    __syncthreads();
    const FitCount r = fit_count<kFitThreads>(x, 0, n, xhi, hist, &ovc, base, ln);
    if (r.bad) atomicOr(&sbad, 1u);
    __syncthreads();
    const bool bad = sbad != 0u;
    const int oc = (int)ovc;
    U128 S = r.S;
    if (!kPrep) {
      const U128 sb = fit_bin_sum<kFitThreads>(hist, 1, ln);
      u128_add(S, sb.lo, sb.hi);
    }
    S = block_sum_u128<kFitThreads>(S, part);
    if (oc > 1 && !bad) {
      const int P = next_pow2(oc);
      if (P <= kFitRun) {
        for (int k = tid; k < P; k += kFitThreads) sbuf[k] = k < oc ? base[k] : INT64_MAX;
        block_sort_pow2(sbuf, P, tid, kFitThreads);
        for (int k = tid; k < oc; k += kFitThreads) base[k] = sbuf[k];
      } else {
        for (int k = oc + tid; k < P; k += kFitThreads) base[k] = INT64_MAX;
        block_sort_pow2(base, P, tid, kFitThreads);
      }
      __syncthreads();
    }
    if (kPrep) {
      const FitView v = fit_view(base, n, 0);
      for (int k = tid; k < kFitBins; k += kFitThreads) v.hist[k] = hist[k];
      for (int k = tid; k < 2 * kFitAcc; k += kFitThreads) v.acc[k] = 0;
      if (tid == 0) {
        v.ctl[0] = (uint32_t)oc;
        v.ctl[1] = bad ? 1u : 0u;
        v.ctl[2] = 1u;
        v.ctl[4] = (uint32_t)S.lo;
        v.ctl[5] = (uint32_t)(S.lo >> 32);
        v.ctl[6] = (uint32_t)S.hi;
        v.ctl[7] = (uint32_t)(S.hi >> 32);
      }
      return;
    }
    if (bad) {
      if (tid == 0) status_out[set] = kErrBadValue;
      __syncthreads();
      continue;
    }
    if (wave == 0) fit_solve(&f, S, n, 1, K, false, ln);
    fit_prefix<kFitThreads>(hist, cum, upart);
    const double d = fit_ks_any(f, hist, cum, base, oc, 0, n, 1, K, wave, kWaves, ln);
    if (lane == 0) dpart[wave] = d;
    __syncthreads();
    if (tid == 0) {
      double D = dpart[0];
      for (int w = 1; w < kWaves; ++w) D = fmax(D, dpart[w]);
      ahat_out[set] = f.a;
      D_out[set] = D;
      flags_out[set] = f.flags;
      status_out[set] = 0u;
    }
    __syncthreads();
  }
}

// Counts of a large dataset: workgroup g takes the g-th chunk, writes its
// counts to its own slot (no shared counters to clear or contend for) and its
// larger values to its chunk's place in g0.  Bound by the reads: 80 MB take 28 us,
// at the rate of a copy 17 us (one workgroup took 6.9 ms with all that follows).
constexpr int kFitCountThreads = 1024;
__global__ __launch_bounds__(kFitCountThreads) void k_fit_count(const int64_t* __restrict__ x,
                                                               int64_t n, int64_t chunk,
                                                               uint32_t K,
                                                               const double* __restrict__ ln,
                                                               int64_t* scratch) {
  __shared__ uint32_t hist[kFitBins];
  __shared__ U128 part[kFitCountThreads / 64];
  __shared__ uint32_t ovc, sbad;
  const int tid = (int)threadIdx.x, g = (int)blockIdx.x;
  const FitView f = fit_view(scratch, n, (int)gridDim.x);
  for (int k = tid; k < kFitBins; k += kFitCountThreads) hist[k] = 0u;
  if (tid == 0) ovc = sbad = 0u;
  if (g == 0)
    for (int k = tid; k < 2 * kFitAcc; k += kFitCountThreads) f.acc[k] = 0;
  __syncthreads();
  const int64_t i0 = (int64_t)g * chunk;
  const int64_t i1 = i0 + chunk < n ? i0 + chunk : n;
  const FitCount r = fit_count<kFitCountThreads>(x, i0, i1, K ? (int64_t)K : INT64_MAX, hist, &ovc,
                                                 f.g0 + i0, ln);
  if (r.bad) atomicOr(&sbad, 1u);
  const U128 S = block_sum_u128<kFitCountThreads>(r.S, part);  // (also orders the counts)
  uint32_t* slot = f.slots + (int64_t)g * kFitBins;
  for (int k = tid; k < kFitBins; k += kFitCountThreads) slot[k] = hist[k];
  if (tid == 0) {
    int64_t* m = f.meta + 4 * (int64_t)g;
    m[0] = (int64_t)ovc;
    m[1] = (int64_t)sbad;
    m[2] = (int64_t)S.lo;
    m[3] = (int64_t)S.hi;
  }
}

// The slots' sum, 64 bins per workgroup, and the larger values sorted in runs
// of kFitRun into g1.  groups <= kFitThreads.
__global__ __launch_bounds__(kFitThreads) void k_fit_merge(int64_t n, int64_t chunk, int groups,
                                                          int64_t* scratch) {
  __shared__ int64_t sbuf[kFitRun];
  __shared__ int64_t pre[kFitThreads + 1];
  __shared__ U128 part[kFitThreads / 64];
  __shared__ uint32_t red[kFitThreads];
  const int tid = (int)threadIdx.x, lane = lane_id();
  constexpr int kWaves = kFitThreads / 64;
  const FitView f = fit_view(scratch, n, groups);
  for (int j = (int)blockIdx.x; j < kFitBins / 64; j += (int)gridDim.x) {
    uint32_t s = 0;
#pragma unroll 8
    for (int g = tid >> 6; g < groups; g += kWaves)
      s += f.slots[(int64_t)g * kFitBins + 64 * j + lane];
    __syncthreads();
    red[tid] = s;
    __syncthreads();
    if (tid < 64) {
      for (int w = 1; w < kWaves; ++w) s += red[64 * w + tid];
      f.hist[64 * j + tid] = s;
    }
  }
  // where each workgroup's larger values start among all
  const int64_t mine = tid < groups ? f.meta[4 * (int64_t)tid] : 0;
  const uint32_t inc = dpp_incl_scan_u32((uint32_t)mine);  // at most n <= 2^31 in all
  __syncthreads();
  if (lane == 63) red[tid >> 6] = inc;
  __syncthreads();
  uint32_t off = 0;
  for (int w = 0; w < tid >> 6; ++w) off += red[w];
  pre[tid + 1] = (int64_t)off + inc;
  if (tid == 0) pre[0] = 0;
  __syncthreads();
  const int64_t oc = pre[kFitThreads];
  if (blockIdx.x == 0) {
    U128 S = {0, 0};
    uint32_t bad = 0;
    if (tid < groups) {
      S = U128{(uint64_t)f.meta[4 * (int64_t)tid + 2], (uint64_t)f.meta[4 * (int64_t)tid + 3]};
      bad = (uint32_t)f.meta[4 * (int64_t)tid + 1];
    }
    S = block_sum_u128<kFitThreads>(S, part);
    const int anybad = __syncthreads_or((int)bad);
    if (tid == 0) {
      int64_t run = kFitRun;
      uint32_t in0 = 0u;  // k_fit_runs alternates
      for (; run < oc; run *= kFitFan) in0 ^= 1u;
      f.ctl[0] = (uint32_t)oc;
      f.ctl[1] = anybad ? 1u : 0u;
      f.ctl[2] = in0;
      f.ctl[4] = (uint32_t)S.lo;
      f.ctl[5] = (uint32_t)(S.lo >> 32);
      f.ctl[6] = (uint32_t)S.hi;
      f.ctl[7] = (uint32_t)(S.hi >> 32);
    }
  }
  for (int64_t r0 = (int64_t)blockIdx.x * kFitRun; r0 < oc; r0 += (int64_t)gridDim.x * kFitRun) {
    const int len = (int)(oc - r0 < kFitRun ? oc - r0 : kFitRun);
    const int P = next_pow2(len);
    __syncthreads();
    for (int k = tid; k < P; k += kFitThreads) {
      int64_t v = INT64_MAX;
      if (k < len) {
        const int64_t p = r0 + k;
        int lo = 0, hi = groups;  // the group g with pre[g] <= p < pre[g + 1]
        while (hi - lo > 1) {
          const int mid = (lo + hi) >> 1;
          if (pre[mid] <= p)
            lo = mid;
          else
            hi = mid;
        }
        v = f.g0[(int64_t)lo * chunk + (p - pre[lo])];
      }
      sbuf[k] = v;
    }
    block_sort_pow2(sbuf, P, tid, kFitThreads);
    for (int k = tid; k < len; k += kFitThreads) f.g1[r0 + k] = sbuf[k];
  }
}

// Merges groups of kFitFan sorted runs of `run` values: a value's place is its
// place in its own run plus the number of smaller ones in each other run of
// the group (equal ones count in earlier runs), found by bisection.  Nothing
// to do when one run holds all.
__global__ __launch_bounds__(256) void k_fit_runs(int64_t n, int groups, int64_t run, int pass,
                                                 int64_t* scratch) {
  const FitView f = fit_view(scratch, n, groups);
  const int64_t oc = (int64_t)f.ctl[0];
  if (oc <= run) return;
  const int64_t* __restrict__ src = (pass & 1) ? f.g0 : f.g1;
  int64_t* __restrict__ dst = (pass & 1) ? f.g1 : f.g0;
  for (int64_t p = (int64_t)blockIdx.x * 256 + threadIdx.x; p < oc;
       p += (int64_t)gridDim.x * 256) {
    const int64_t v = src[p];
    const int64_t own = p / run, first = own / kFitFan * kFitFan;
    int64_t to = first * run + (p - own * run);
    for (int64_t r = first; r < first + kFitFan && r * run < oc; ++r) {
      if (r == own) continue;
      const int64_t a = r * run, b = a + run < oc ? a + run : oc;
      // values below v, or up to it in an earlier run (v < INT64_MAX there,
      // as no earlier run's value can exceed it)
      int64_t lo = a, hi = b;
      while (lo < hi) {
        const int64_t mid = (lo + hi) >> 1;
        if (src[mid] < v || (r < own && src[mid] == v))
          lo = mid + 1;
        else
          hi = mid;
      }
      to += lo - a;
    }
    dst[to] = v;
  }
}

// The fit with each candidate cutoff (xmins; without them the one fit from 1
// on, with or without the upper limit K) from the counts and the sorted larger
// values, `wgs` workgroups per candidate.  kCount: of a dataset of up to kFitSmall
// values, which each candidate's one workgroup counts and sorts itself.  A candidate
// above every value gets D = +inf and status kErrNoTail; any value below 1 sets
// kErrBadValue.
// One wave solves eq. 2 (latency: a chain of Newton steps), all share the
// distance.  Registers for four workgroups per compute unit: 1,000 candidates
// over 100,000 values take 77 us so, 86 us with two.
template <bool kCount>
__global__ __launch_bounds__(kCount ? kFitThreads : kFitCandThreads, 4) void k_fit_cand(
    const int64_t* x, int64_t n, int groups, int64_t* scratch, const int64_t* __restrict__ xmins,
    int wgs, uint32_t K, const double* __restrict__ ln, double* ahat_out, double* D_out, int64_t* ntail_out,
    uint32_t* flags_out, uint32_t* status_out) {
  constexpr int kThreads = kCount ? kFitThreads : kFitCandThreads;
  __shared__ __align__(16) uint32_t hist[kFitBins];
  __shared__ uint32_t cum[kFitBins + 1];
  __shared__ FitSolved f;
  __shared__ U128 part[kThreads / 64];
  __shared__ uint32_t upart[kThreads / 64];
  __shared__ double dpart[kThreads / 64];
  const int tid = (int)threadIdx.x, lane = lane_id(), wave = tid >> 6;
  constexpr int kWaves = kThreads / 64;
  __shared__ int64_t larger[kCount ? kFitSmall : 1];
  __shared__ uint32_t ovc, sbad;
  const int cand = (int)blockIdx.x / wgs, share = (int)blockIdx.x % wgs;
  const FitView v = fit_view(scratch, n, groups);
  const int64_t xmin = xmins ? xmins[cand] : 1;
  U128 So = {0, 0};  // this thread's part of the larger values' sum of logarithms
  int64_t oc;
  bool bad;
  const int64_t* ov;
  if constexpr (kCount) {
    for (int k = tid; k < kFitBins; k += kThreads) hist[k] = 0u;
    if (tid == 0) ovc = sbad = 0u;
    __syncthreads();
    const FitCount r = fit_count<kThreads>(as_global(x), 0, n, K ? (int64_t)K : INT64_MAX,
                                                  hist, &ovc, larger, ln);
    if (r.bad) atomicOr(&sbad, 1u);
    So = r.S;
    __syncthreads();
    oc = (int64_t)ovc;
    bad = sbad != 0u;
    ov = larger;
    if (oc > 1) {
      const int P = next_pow2((int)oc);
      for (int k = (int)oc + tid; k < P; k += kThreads) larger[k] = INT64_MAX;
      block_sort_pow2(larger, P, tid, kThreads);
    }
  } else {
    oc = (int64_t)v.ctl[0];
    bad = v.ctl[1] != 0u;
    ov = v.ctl[2] ? v.g0 : v.g1;
    if (tid == 0)
      So = U128{(uint64_t)v.ctl[4] | (uint64_t)v.ctl[5] << 32,
                (uint64_t)v.ctl[6] | (uint64_t)v.ctl[7] << 32};
    for (int k = 4 * tid; k < kFitBins; k += 4 * kThreads)
      *reinterpret_cast<uint4*>(hist + k) = *reinterpret_cast<const uint4*>(v.hist + k);
  }
  __syncthreads();
  fit_prefix<kThreads>(hist, cum, upart);
  const int64_t p0 = xmin > kFitBins + 1 && !bad ? lower_bound_i64(ov, 0, oc, xmin) : 0;
  const int64_t nt = xmin > kFitBins + 1 ? oc - p0
                                         : (int64_t)cum[kFitBins] - (int64_t)cum[xmin - 1] + oc;
  if (bad || nt == 0) {
    if (tid == 0 && share == 0) {
      if (ntail_out) {  // (a single fit leaves its outputs)
        ahat_out[cand] = 0.0;
        D_out[cand] = __builtin_inf();
        ntail_out[cand] = nt;
        flags_out[cand] = 0u;
      }
      status_out[cand] = bad ? kErrBadValue : kErrNoTail;
    }
    return;
  }
  U128 S = {0, 0};
  if (xmin <= kFitBins) S = fit_bin_sum<kThreads>(hist, xmin, ln);
  if (xmin > kFitBins + 1) {
    for (int64_t p = p0 + tid; p < oc; p += kThreads) u128_add(S, ln_fixed(ov[p], ln), 0);
  } else {
    u128_add(S, So.lo, So.hi);
  }
  S = block_sum_u128<kThreads>(S, part);
  if (wave == 0) {
    bool atmin;
    if (xmin <= kFitBins)
      atmin = (int64_t)hist[xmin - 1] == nt;
    else
      atmin = ov[p0] == xmin && ov[oc - 1] == xmin;
    fit_solve(&f, S, nt, xmin, K, atmin, ln);
  }
  __syncthreads();
  const int gw = share * kWaves + wave, nw = wgs * kWaves;
  double d;
  if (xmin > 17)
    d = fit_ks<kFitCutRel>(f, hist, cum, ov, oc, p0, nt, xmin, 0u, gw, nw, ln);
  else if (xmin > 1)
    d = fit_ks<kFitCut>(f, hist, cum, ov, oc, p0, nt, xmin, 0u, gw, nw, ln);
  else
    d = fit_ks_any(f, hist, cum, ov, oc, p0, nt, xmin, K, gw, nw, ln);
  if (lane == 0) dpart[wave] = d;
  __syncthreads();
  if (tid != 0) return;
  double D = dpart[0];
  for (int w = 1; w < kWaves; ++w) D = fmax(D, dpart[w]);
  if (wgs > 1) {  // the last workgroup to finish writes the maximum
    unsigned long long* acc = reinterpret_cast<unsigned long long*>(v.acc + 2 * (int64_t)cand);
    atomicMax(acc, (unsigned long long)__double_as_longlong(D));  // D >= 0: ordered as its bits
    __threadfence();
    if (atomicAdd(acc + 1, 1ull) + 1ull != (unsigned long long)wgs) return;
    __threadfence();
    D = __longlong_as_double((long long)atomicMax(acc, 0ull));
  }
  ahat_out[cand] = f.a;
  D_out[cand] = D;
  if (ntail_out) ntail_out[cand] = nt;
  flags_out[cand] = f.flags;
  status_out[cand] = 0u;
}

}  // namespace zpl
