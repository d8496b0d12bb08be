// C wrapper around the conjugate pairing of Ritz values, built by the CPU
// test-suite with g++ (no GPU, no HIP).
#include <complex>
#include <vector>

#include "../../paper_1903_06986_amd/csrc/smallla.h"

extern "C" void la_pair_conjugates(int n, double *w, int *partner) {
  using lqcd::la::cd;
  cd *wc = reinterpret_cast<cd *>(w);
  std::vector<cd> v(wc, wc + n);
  const std::vector<int> p = lqcd::la::pair_conjugates(v);
  for (int i = 0; i < n; ++i) {
    wc[i] = v[i];
    partner[i] = p[i];
  }
}
