// Host build of the scratch sizes (zpl_scratch.hpp) for the CPU tests.
#include <vector>

#include "../../paper_1305_6738_amd/csrc/zpl_scratch.hpp"

using namespace zpl;

extern "C" {
int64_t sc_area(int64_t heavy8, int64_t sim_units, int64_t max_n, int64_t esc, uint64_t budget,
                int n_cu) {
  return scratch_words(heavy8, sim_units, max_n, esc, budget, n_cu);
}
void sc_share(int64_t area, int64_t units, int waves, int64_t room, int n_cu, int64_t* out) {
  const Share s = share_scratch(area, units, waves, room, n_cu);
  out[0] = s.grid;
  out[1] = s.stride;
  out[2] = s.waves;
}
int sc_split(int64_t area, int64_t units, int waves, int64_t max_room, int n_cu, int64_t* limit) {
  return split_batch(area, units, waves, max_room, n_cu, *limit) ? 1 : 0;
}
int64_t sc_parted(int64_t units, int waves, int64_t room, uint64_t budget, int n_cu) {
  return parted_words(units, waves, room, budget, n_cu);
}
int64_t sc_need(int64_t room) { return batch_need(room); }
// Values above the histogram that the first replicate of a wave's batch has
// place for, n draws of 32-bit (n >= 65536) or 16-bit counts: as the kernel
// computes it from its stride.
int64_t sc_first_room(int64_t stride, int64_t n) {
  const int64_t records = 64 * (int64_t)kWaveSlotBytes / 8;
  return stride - (records + (n >= 65536 ? kHW / 2 : kHW / 4));
}
// The simulation kernel's places, each [first, end) of the scratch: 0 on success,
// 1 when nothing fits, 2 when places of different workgroups (or of a workgroup's
// waves) overlap or lie outside, 3 when a wave's does not hold its replicate.
int sc_place(int64_t total, int lane_wgs, int lane_waves, int64_t units, int64_t n_big, int waves,
             int64_t max_room, int64_t small_room, int n_cu, int64_t* rest_stride) {
  SimGrid g = {};
  g.lane_wgs = lane_wgs;
  g.lane_waves = lane_waves;
  g.n_big = (int)n_big;
  if (!place_sim(g, total, units, waves, max_room, small_room, n_cu)) return 1;
  *rest_stride = g.stride;
  struct Place {
    int64_t first, end;
    int wg;
  };
  std::vector<Place> all;
  auto add = [&](int wg, int64_t first, int64_t words) { all.push_back({first, first + words, wg}); };
  for (int b = 0; b < lane_wgs; ++b) add(b, b * g.lane_area, lane_waves * (int64_t)kLaneScratch);
  const int64_t fixed = 64 * (int64_t)kWaveSlotBytes / 8 + kHW / 2;
  for (int b = 0; b < g.batch_wgs; ++b) {
    const int wg = b + g.grid - g.batch_wgs;
    const bool big = b < g.big_wgs;
    const int w = big ? g.big_waves : g.waves;
    const int64_t stride = big ? g.big_stride : g.stride;
    if (stride < fixed + (big ? max_room : small_room) || w < 1) return 3;
    add(wg, big ? g.big_area + (int64_t)b * w * stride : g.rest + (b - g.big_wgs) * g.area,
        w * stride);
    if (g.area < g.waves * g.stride) return 2;
  }
  std::sort(all.begin(), all.end(), [](const Place& x, const Place& y) { return x.first < y.first; });
  for (size_t i = 0; i < all.size(); ++i) {
    if (all[i].first < 0 || all[i].end > total || all[i].wg >= g.grid) return 2;
    for (size_t j = i + 1; j < all.size() && all[j].first < all[i].end; ++j)
      if (all[j].wg != all[i].wg) return 2;
  }
  return 0;
}
int sc_waves() { return kBatchWaves; }
int sc_waves_cut() { return kBatchWavesCut; }
int sc_esc_waves() { return kEscWaves; }
}
