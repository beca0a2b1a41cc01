// Host build of the truncated law's survival sums (zpl_math.hpp) for the CPU tests.
#include <cmath>
#include <cstdint>
#include <vector>

#include "../../paper_1305_6738_amd/csrc/zpl_math.hpp"

using namespace zpl;

static std::vector<double> g_ln = [] {
  std::vector<double> v(kH + 2);
  for (int k = 1; k <= kH + 1; ++k) v[k] = std::log((double)k);
  return v;
}();

extern "C" {
int tt_em(double s, uint32_t K) { return trunc_em(s, K) ? 1 : 0; }
// out[t], t = 0..K: the sum of k^-s over t < k <= K
void tt_sums(double s, uint32_t K, double* out) {
  const EmCoef E = em_coef(s);
  const TruncEnd e = trunc_end(E, K, g_ln.data());
  double suf[17];
  survival_head_trunc(E, e, g_ln.data(), suf);
  for (int t = 0; t <= 16; ++t) out[t] = suf[t];
  for (uint32_t t = 17; t <= K; ++t)
    out[t] = trunc_tail(E, e, (int64_t)t, t < K ? g_ln[t + 1] : 0.0);
}
}
