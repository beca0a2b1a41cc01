// Host build of the draw loops' 32-bit steps (zpl_math.hpp) for the CPU tests.
#include <cstdint>

#include "../../paper_1305_6738_amd/csrc/zpl_math.hpp"

using namespace zpl;

extern "C" {
int fd_sh_max() { return kGuideShMax; }
int fd_uniform() { return kGuideUniform; }
// The number of the words w[i] (64 bits of a uniform) whose bin by the first
// 32 bits is not the bin of m = (w >> 11) | 1; *taken counts the ones it takes.
int64_t fd_bins(const uint64_t* w, int64_t n, int sh, int64_t* taken) {
  const GuideRule r = guide_rule(sh);
  int64_t bad = 0, t = 0;
  for (int64_t i = 0; i < n; ++i) {
    const uint32_t w0 = (uint32_t)(w[i] >> 32);
    if (w0 > r.last) continue;
    ++t;
    bad += guide_index32(w0, r) != guide_index((w[i] >> 11) | 1ull, sh);
  }
  *taken = t;
  return bad;
}
// The number of pairs for which the first words decide differently from t >= m.
int64_t fd_thresholds(const uint64_t* w, const uint64_t* t, int64_t n) {
  int64_t bad = 0;
  for (int64_t i = 0; i < n; ++i) {
    const uint32_t w0 = (uint32_t)(w[i] >> 32), hi = threshold_hi(t[i]), lo = threshold_lo(t[i]);
    bad += threshold(hi, lo) != t[i];
    if (w0 != hi) bad += (w0 < hi) != (t[i] >= ((w[i] >> 11) | 1ull));
  }
  return bad;
}
uint32_t fd_offsets(uint32_t gg) { return guide_offsets(gg); }
}
