// Host build of the scratch sizes (zpl_scratch.hpp) for the CPU tests.
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
int64_t sc_need(int64_t room) { return batch_need(room); }
// Values above the histogram that the first replicate of a wave's batch has
// place for, n draws of 32-bit (n >= 65536) or 16-bit counts: as the kernel
// computes it from its stride.
int64_t sc_first_room(int64_t stride, int64_t n) {
  const int64_t records = 64 * (int64_t)kWaveSlotBytes / 8;
  return stride - (records + (n >= 65536 ? kHW / 2 : kHW / 4));
}
int sc_waves() { return kBatchWaves; }
int sc_waves_cut() { return kBatchWavesCut; }
int sc_esc_waves() { return kEscWaves; }
}
