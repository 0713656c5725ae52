// Host check of the sort's bins: every value gets one of them, in order, also where it lies any number of bins beyond the last.
#include <cmath>
#include <cstdio>
#include <initializer_list>
#include "bins.h"

int main() {
  int wrong = 0;
  for (int bins : {256, 512})
    for (float span : {1e-38f, 1e-3f, 1.0f, 77.0f, 3e38f}) {
      const float scale = float(bins - 1) / span;
      int before = 0;
      for (double share : {0.0, 1e-9, 0.25, 0.5, 1.0, 1.5, 4e6, 5e6, 1e9, 1e30, 1e60}) {
        const float above = float(std::fmin(share * double(span), 3e38));
        const int b = tslt::value_bin_of(above, scale, bins);
        wrong += b < before || b >= bins || (share >= 1.01 && std::isfinite(above * scale) && above > span && b != bins - 1);
        before = b;
      }
      wrong += tslt::value_bin_of(INFINITY, scale, bins) != bins - 1;
    }
  std::printf("wrong %d\n", wrong);
  return 0;
}
