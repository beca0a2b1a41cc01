// Runs the batch kernels of libzpl on one cell with a given room and scratch per
// wave, so that replicates exceed them: what a simulation call's own sizes leave to
// events of twelve standard deviations.  Linked to the library under test.
#include <hip/hip_runtime_api.h>

#include <algorithm>
#include <vector>

#include "../../paper_1305_6738_amd/csrc/zpl_launch.hpp"
#include "../../paper_1305_6738_amd/csrc/zpl_scratch.hpp"

using namespace zpl;

namespace {
struct Buf {
  void* p = nullptr;
  explicit Buf(size_t bytes) {
    if (hipMalloc(&p, bytes) != hipSuccess) p = nullptr;
  }
  ~Buf() { (void)hipFree(p); }
};
}  // namespace

// `extra` int64 of scratch per wave beyond one replicate's records and counts.
// D, ahat, flags, fp: device arrays of R.  out: escalated replicates, error word.
// 0 on success, else the step that failed.
extern "C" int es_run(double alpha, int64_t n, int32_t R, uint64_t seed, uint32_t stream, uint32_t K,
                      int64_t xmin, uint32_t room, int64_t extra, int32_t unit, double* D,
                      double* ahat, uint32_t* flags, uint64_t* fp, uint32_t* out) {
  constexpr int kLnK = 4096;  // support values of the tables
  const int waves = xmin > 1 ? kBatchWavesCut : kBatchWaves;
  const int64_t stride =
      (64 * (int64_t)kWaveSlotBytes / 8 + (n >= 65536 ? kHW / 2 : kHW / 4) + extra + 31) & ~31ll;
  const int64_t estride = batch_need(n);
  DevCell c = {};
  c.alpha = alpha;
  c.n = n;
  c.R = R;
  c.k0 = (uint32_t)seed;
  c.k1 = (uint32_t)(seed >> 32);
  c.stream = stream;
  c.mode = kModeHeavy;
  c.K = K;
  c.xmin = xmin > 1 ? xmin : 1;
  c.room = room;
  std::vector<Unit> units;
  for (int32_t r = 0; r < R; r += unit) units.push_back(Unit{0, std::min(unit, R - r), r});
  Buf ln((kLnK + 2) * 16 + 16 * 1024), cells(sizeof c), tables(kLnK * 8), guides((kGuide + 1) * 2),
      du(sizeof(Unit) * units.size()), words(64 * 4), list(8 * (size_t)R),
      scratch(8 * (size_t)(waves * stride)), escratch(8 * (size_t)(2 * kEscWaves * estride));
  for (const Buf* b : {&ln, &cells, &tables, &guides, &du, &words, &list, &scratch, &escratch})
    if (!b->p) return 1;
  if (hipMemcpy(cells.p, &c, sizeof c, hipMemcpyHostToDevice) != hipSuccess ||
      hipMemcpy(du.p, units.data(), sizeof(Unit) * units.size(), hipMemcpyHostToDevice) != hipSuccess)
    return 2;
  uint32_t* w = (uint32_t*)words.p;  // queues 0..7, escalated 8, error 9
  const DevCell* dc = (const DevCell*)cells.p;
  const double* dl = (const double*)ln.p;
  const double* dt = (const double*)tables.p;
  const uint16_t* dg = (const uint16_t*)guides.p;
  const Outputs o{D, ahat, flags, fp};
  if (launch_ln_table((double*)ln.p, nullptr) != hipSuccess ||
      launch_tables((DevCell*)cells.p, 1, (double*)tables.p, (uint16_t*)guides.p, dl, nullptr,
                    K != 0, w, 64) != hipSuccess)
    return 3;
  hipError_t e;
  if (xmin > 1) {
    e = launch_cutoff(1, dc, dt, dg, dl, (const Unit*)du.p, (int)units.size(), w, o,
                      (uint64_t*)list.p, w + 8, (uint32_t)R, (int64_t*)scratch.p, waves, stride,
                      w + 9, nullptr);
  } else {
    SimGrid g = {};
    g.grid = g.batch_wgs = 1;
    g.waves = waves;
    g.stride = stride;
    g.area = waves * stride;
    e = launch_simulate(g, dc, dt, dg, dl, nullptr, 0, (const Unit*)du.p, (int)units.size(), w + 1,
                        w, w + 2, o, (uint64_t*)list.p, w + 8, (uint32_t)R, (int64_t*)scratch.p,
                        w + 9, nullptr);
  }
  if (e != hipSuccess) return 4;
  e = launch_escalated(2, dc, dt, dg, dl, w + 4, o, (uint64_t*)list.p, w + 8, (uint32_t)R,
                       (int64_t*)escratch.p, kEscWaves, estride, w + 9, nullptr);
  if (e != hipSuccess) return 5;
  if (hipDeviceSynchronize() != hipSuccess) return 6;
  return hipMemcpy(out, w + 8, 8, hipMemcpyDeviceToHost) == hipSuccess ? 0 : 7;
}
