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

// An area of int64 shared by `grid` workgroups, of which `waves` waves each work
// on `stride` of it.
struct Share {
  int grid, waves;
  int64_t stride;
};
// For `units` of up to `waves` waves each, one workgroup per compute unit at most,
// whose waves each hold a replicate with `room` values above the histogram.
// Where the area does not hold that many, fewer waves per workgroup, and then
// fewer workgroups: waves on compute units of their own do not share issue
// slots.  The strides are multiples of 32, and it is the rounded one that has to
// hold a replicate: one whose room is all of its n draws has nowhere else to go.
// Grid 0: no units, or not even one replicate fits.
inline int64_t batch_need(int64_t room) {  // with what its KS partitions its draws in
  return (kBatchFixed + room + part_words(room) + 31) & ~(int64_t)31;
}
inline Share share_scratch(int64_t area, int64_t units, int waves, int64_t room, int n_cu) {
  int64_t most = area / batch_need(room);
  if (most < 1) most = area / ((kBatchFixed + room + 31) & ~(int64_t)31);
  const int64_t g = std::min<int64_t>(std::min<int64_t>(units, n_cu), most);
  if (g < 1) return Share{0, 0, 0};
  const int64_t w = std::min<int64_t>(waves, most / g);
  return Share{(int)g, (int)w, area / (g * w) & ~(int64_t)31};
}

// int64 with which all of the units' waves hold a replicate of `room` values and what
// its KS partitions them in: scratch_words follows the replicates, and with fewer
// waves than a unit has replicates, it takes a second pass (cutoffs 739, alpha 1.8 and
// 3.43, 1,531 replicates each of n = 1975: 457 us by 11 waves of 12, 322 by all).  0
// where the KS partitions nothing, and for the longest replicates, which pay with
// fewer waves too; up to a sixteenth of the budget.
inline int64_t parted_words(int64_t units, int waves, int64_t room, uint64_t budget, int n_cu) {
  if (room <= kPartMin || room >= 65536) return 0;
  const int64_t words = std::min<int64_t>(units, n_cu) * waves * batch_need(room);
  return (uint64_t)words <= budget / 128 ? words : 0;
}

// Cells of one call may differ by orders of magnitude in their rooms, and a share
// that holds the largest would leave the device to a few workgroups.  When it
// does (the result is true), cells of rooms up to `limit` share a quarter of the
// area among all workgroups, and the longer ones have the rest of it to
// themselves: six cells of 20,000 draws (1.15 ms alone) beside ten replicates of
// 10^7 at alpha = 2 (28 ms) took 45 ms in the workgroups that one share leaves.
inline bool split_batch(int64_t area, int64_t units, int waves, int64_t max_room, int n_cu,
                        int64_t& limit) {
  const Share all = share_scratch(area, units, waves, max_room, n_cu);
  if (all.grid == std::min<int64_t>(units, n_cu) && all.waves == waves) return false;
  limit = area / 4 / ((int64_t)n_cu * waves) & ~(int64_t)31;
  return true;
}

// The simulation kernel's scratch of `total` int64: g's lane_wgs, lane_waves and
// n_big given, `units` units of the wave and heavy forms of up to `waves` waves
// each, the first n_big of rooms up to max_room and the others of up to small_room.
// False when a replicate does not fit.
inline bool place_sim(SimGrid& g, int64_t total, int64_t units, int waves, int64_t max_room,
                      int64_t small_room, int n_cu) {
  const int64_t slots = (int64_t)g.lane_wgs * g.lane_waves * kLaneScratch, area = total - slots;
  // (multiples of 32, so that whole records and counts stay aligned)
  const int64_t big_words = g.n_big > 0 ? (area - area / 4) & ~(int64_t)31 : 0;
  const Share big = share_scratch(big_words, g.n_big, waves, max_room, n_cu);
  const int64_t others = units > g.n_big ? std::min<int64_t>(units, n_cu) - big.grid : 0;
  const Share rest = share_scratch(area - big_words, others, waves, small_room, n_cu);
  if ((g.n_big > 0 && big.grid == 0) || (others > 0 && rest.grid == 0)) return false;
  g.lane_area = (int64_t)g.lane_waves * kLaneScratch;
  g.big_wgs = big.grid;
  g.big_waves = big.waves;
  g.big_stride = big.stride;
  g.big_area = slots;
  g.waves = rest.waves;
  g.stride = rest.stride;
  g.rest = slots + big_words;
  g.area = rest.waves * rest.stride;
  g.batch_wgs = big.grid + rest.grid;
  g.grid = std::min(g.lane_wgs + g.batch_wgs, n_cu);
  // Where workgroups take units of both kinds, one after the other, each has an
  // equal part of all the scratch for both: beside them the slots leave a wave 8
  // replicates at a time (K = 50, n = 100, 12 exponents of which two are in the
  // wave form: 1.61 ms, 0.92 with whole batches).
  if (big.grid == 0 && rest.grid > 0 && g.lane_wgs + rest.grid > g.grid) {
    const int64_t part = total / g.grid & ~(int64_t)31;
    const Share one = share_scratch(part, 1, waves, small_room, n_cu);
    if (part >= g.lane_area && one.waves >= rest.waves && one.stride > rest.stride) {
      g.lane_area = g.area = part;
      g.rest = (int64_t)(g.grid - rest.grid) * part;
      g.waves = one.waves;
      g.stride = one.stride;
    }
  }
  return true;
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
