// Host build of the MLE's tabulated start (zpl_math.hpp) for the CPU tests.
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
static std::vector<double> g_guess = [] {
  std::vector<double> v(2 * kGuessN);
  for (int i = 0; i < kGuessN; ++i) mle_guess_entry(i, g_ln.data(), &v[2 * i]);
  return v;
}();

extern "C" {
double ms_general(double m, uint32_t* flags) { return mle_alpha(m, g_ln.data(), flags); }
double ms_start(double m, uint32_t* flags, int* iters) {
  return mle_alpha_start(m, g_ln.data(), g_guess.data(), flags, iters);
}
}
