// zpl_kernels.hpp -- device-side data layout shared by the kernels and the
// host runtime of libzpl (not part of the public C ABI).
#pragma once

#include <stdint.h>

namespace zpl {

// Two-part guide table over U.  For U < 1/2: kGA bins uniform in U.  For
// U > 1/2: bins on e = 1 - U (exact in FP64), one per (octave of e, top
// kGBits + gsh mantissa bits), ordered so that the bin index increases with
// U.  Entry g[b] is the smallest k a uniform in bin b can map to, so U in bin
// b maps into [g[b], g[b+1]].  On the Zipf law the survival is close to a
// power of k, so log-scale bins keep most brackets one or two entries wide.
// gsh (0..kGuideShMax, per cell) refines the bins when the table's part of
// U > 1/2 spans few octaves of e (heavy tails: at alpha = 1.2 the table ends
// at e = 0.17, two octaves): the 3,328 entries then cover 52 >> gsh octaves,
// and indices of deeper octaves (tail draws) are clamped to the last entry.
// gsh = kGuideUniform selects a uniform layout instead, for a table whose
// support is bounded (the truncated law: no tail) and spread out: 2048 bins
// uniform in U (bin m >> 42, entries from 2048 on unused).
constexpr int kGuideShMax = 4;
constexpr int kGuideUniform = 8;
constexpr int kGA = 256;
constexpr int kGBits = 6;
constexpr int kOctaves = 52;  // e in [2^-53, 1/2)
constexpr int kGuide = kGA + (kOctaves << kGBits);

// Lane-form kernel geometry: twelve wave64 per workgroup share the CDF table and
// the guide in LDS.
constexpr int kWaves = 12;  // three per SIMD
constexpr int kBlock = 64 * kWaves;
// Lane form: one replicate per lane; per-lane histogram of values 1..kHLB
// (16-bit counters packed two per dword) plus a per-lane list of up to
// kLaneCap larger values in the wave's global scratch (a replicate with more
// is escalated).
constexpr int kHLB = 48;
constexpr int kLaneCap = 224;
// int64 of scratch per wave of the lane form: kLaneCap slots per lane, and as
// many again for the finish.
constexpr int kLaneScratch = 64 * 2 * kLaneCap;
// Wave and heavy forms: one replicate per wave at a time, in batches that a
// wave finishes together (replicate_batch): histogram of values 1..kHW in LDS, larger
// ones in the wave's global scratch.  Waves per workgroup (one workgroup per
// compute unit) without and with a lower cutoff: three per SIMD are better than
// two (heavy tails of 10,000 draws: 5.81 against 6.16 ms; cutoffs, 1,000 draws:
// 5.69 against 6.45 ms).
constexpr int kHW = 1024;
constexpr int kBatchWaves = 12;
constexpr int kBatchWavesCut = 12;
// A replicate with more values above the histogram than kPartMin partitions them
// by bin in the scratch that is left behind its counts (ks_many): kPartLevel
// int64 for the bins of a level and a copy of the draws in reach, and the same for
// the ranges within a bin (an eighth of the draws or less, and for the longest
// replicates ranges within those).  Cutoff 1e6, so that all draws are such: 10,000
// replicates of 1,500 draws 1.25 ms by bins and 1.14 in windows over all of them, of
// 2,500 1.36 and 2.35; 1,000 replicates of 20,000 4.2 and 23.6; alpha 1.2, 10,000
// draws (about 1,700 such): 1.9 and 2.3.
constexpr int64_t kPartMin = 1536;
constexpr int64_t kPartLevel = 3 * kHW / 2;
constexpr int64_t part_words(int64_t room) {
  return room <= kPartMin ? 0
         : room < 65536   ? room + room / 8 + 2 * kPartLevel
                          : room + room / 4 + 3 * kPartLevel;
}
// Truncated law: up to this K the lanes of a batch of 16 replicates and more walk
// the support themselves for the KS distance (head_lane).
constexpr uint32_t kTruncLaneK = 100;
// Waves per workgroup that run escalated replicates (whole replicates of
// scratch each, so few).
constexpr int kEscWaves = 4;
// Part of a dataset's scratch that does not grow with it (heavy_stride).
constexpr int kHeavyHist = 1024;
// Allocation-free fit: the larger values and the counts of one dataset of up to
// kNoAllocMaxN values (fit_view) live in a fixed device array of
// kNoAllocStride int64 (heavy_stride of that n:
// 2 * max(2^20, 2 * (kHeavyHist + 2^20))).
constexpr int64_t kNoAllocMaxN = (int64_t)1 << 20;
constexpr int64_t kNoAllocStride = 2 * (2 * ((int64_t)kHeavyHist + kNoAllocMaxN));

// Quantiles per selection pass and the per-(cell, quantile) capacity of the
// bracket gather scratch.
constexpr int kSelQ = 4;
constexpr int64_t kSelGather = 32768;
// Size of the per-replicate record of a batch (global scratch, 64 per wave).
constexpr int kWaveSlotBytes = 48;

enum Mode : uint32_t { kModeLane = 0, kModeWave = 1, kModeHeavy = 2 };

struct DevCell {
  double alpha;   // exponent the draws use
  double beta;    // alpha - 1
  double gm;      // tail acceptance constant g(kH + 1)
  double tmax;    // T[kH], written by the guide kernel
  int64_t n;      // draws per replicate
  int64_t R;      // replicates
  int64_t out_off;  // offset of replicate 0 in the per-replicate outputs
  uint32_t k0, k1;  // Philox key = seed
  uint32_t stream;  // Philox counter word 2
  uint32_t mode;    // Mode
  uint32_t K;       // 0: the pure law; else the truncated law on 1..K
  uint32_t gsh;     // guide refinement: 2^(kGBits + gsh) bins per octave of 1 - U
  int64_t xmin;     // lower cutoff of the pure law (1: none); values >= xmin
  // wave and heavy forms: scratch kept free for a replicate's values above the
  // histogram before it is begun (n: all it can have)
  uint32_t room;
  uint32_t pad;
};

struct Unit {
  int32_t cell;
  int32_t count;  // replicates in this unit
  int64_t r0;     // first replicate
};

// Launch shape of the simulation kernel: workgroups 0 .. lane_wgs - 1 take
// lane-form units (of at most 64 lane_waves replicates), the last batch_wgs
// wave- and heavy-form ones.  Of those the first big_wgs take the first n_big
// units before the others, by big_waves waves with big_stride int64 of scratch
// each; in the other workgroups it is `waves` with `stride` each.  Workgroup g of
// the lane form has its slots at lane_area g of the scratch, workgroup b of the
// others its waves' scratch at big_area + big_waves big_stride b, or at rest +
// area (b - big_wgs).  (A workgroup that takes both kinds may have both at one place: it
// ends the one before it begins the other.)
struct SimGrid {
  int32_t grid, lane_wgs, lane_waves, batch_wgs;
  int32_t n_big, big_wgs, big_waves, waves;
  int64_t lane_area, big_area, big_stride, rest, area, stride;
};

struct Outputs {
  double* D;
  double* ahat;
  uint32_t* flags;
  uint64_t* fp;
};

// Error bits written by kernels into the context's error word.
constexpr uint32_t kErrEscOverflow = 1u;
constexpr uint32_t kErrBadValue = 2u;
constexpr uint32_t kErrNoTail = 4u;  // no value at or above the cutoff (xmin scan)

}  // namespace zpl
