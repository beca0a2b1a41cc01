// zpl_scratch.hpp -- how a simulation call's scratch is sized and shared by the
// waves of the batch kernels (host only).
#pragma once

#include <algorithm>

#include "zpl_kernels.hpp"

namespace zpl {

// int64 of scratch of one sorted replicate or dataset of up to max_n values.
inline int64_t heavy_stride(int64_t max_n) {
  int64_t p2 = 1;
  while (p2 < max_n) p2 <<= 1;
  int64_t half = std::max<int64_t>(p2, 2 * ((int64_t)kHeavyHist + max_n));
  half = (half + 1) & ~(int64_t)1;
  return 2 * half;
}

// What a wave works with besides a replicate's values above the histogram: the
// records and one replicate's counts (the wider ones, of n >= 65536).
constexpr int64_t kBatchFixed = 64 * (int64_t)kWaveSlotBytes / 8 + kHW / 2;

// An area of int64 shared by `grid` workgroups, `stride` for each of their waves.
struct Share {
  int grid;
  int64_t stride;
};
// The most workgroups, up to `units` and one per compute unit, whose waves each
// hold a replicate with `room` values above the histogram.  The strides are
// multiples of 32, and it is the rounded one that has to hold it: a replicate
// whose room is all of its n draws has nowhere else to go.  Grid 0: not even
// one workgroup's do.
inline Share share_scratch(int64_t area, int64_t units, int waves, int64_t room, int n_cu) {
  auto stride = [&](int64_t g) { return area / (g * waves) & ~(int64_t)31; };
  int64_t g = std::min<int64_t>(units, n_cu);
  while (g > 1 && stride(g) < kBatchFixed + room) g = (g + 1) / 2;
  if (g < 1 || stride(g) < kBatchFixed + room) return Share{0, 0};
  return Share{(int)g, stride(g)};
}

// int64 of scratch for a call's replicates: the lane form's slots, then what the
// waves of the other forms share.  It follows the forms: kFormScratch for each
// wave of a workgroup per kBlock lane- and wave-form replicates (2.8 MiB a
// workgroup; sim_units of them), and four areas of a sorted replicate's size for
// each 8 heavy-form ones (heavy8), up to two per compute unit and a quarter of
// the budget; less what the escalation list takes for them (esc).
constexpr int64_t kFormScratch = 30912;
static_assert(kLaneScratch <= kFormScratch, "a lane unit's slots are part of what it brings in");
inline int64_t scratch_words(int64_t heavy8, int64_t sim_units, int64_t max_n, int64_t esc,
                             uint64_t budget, int n_cu) {
  const int64_t hstride = heavy_stride(max_n);
  int64_t hg = std::min<int64_t>(heavy8 + 64, (int64_t)n_cu * 2);
  while (hg > 1 && (uint64_t)hg * 4 * hstride * 8 > budget / 4) hg /= 2;
  const int64_t sim_wgs = std::max<int64_t>(1, std::min<int64_t>(sim_units, n_cu));
  return hg * 4 * hstride + sim_wgs * kWaves * kFormScratch - esc;
}

}  // namespace zpl
