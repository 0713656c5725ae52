// Host check of exp64.h's table-driven exponential against libm: the largest error, in ulps, over fp32 arguments of
// its whole range, and whether the table's ends are what they should be.
#include <cmath>
#include <cstdint>
#include <cstdio>
#include "exp64.h"

int main() {
  static uint64_t table[tslt::kPowEntries];
  for (int i = 0; i < tslt::kPowEntries; ++i) table[i] = tslt::pow_entry(i);
  double worst = 0.0;
  uint64_t s = 0x9E3779B97F4A7C15ull;
  for (int i = 0; i < 4000000; ++i) {
    s ^= s << 13; s ^= s >> 7; s ^= s << 17;
    const double u = double(s >> 11) * (1.0 / 9007199254740992.0);
    const float x = float(i % 4 == 0 ? 1200.0 * u - 600.0 : 60.0 * u - 50.0);
    const long double want = expl((long double)x);
    int e;
    std::frexp(double(want), &e);
    const double err = std::fabs(double((long double)tslt::pow_exp(x, table) - want)) / std::ldexp(1.0, e - 53);
    if (err > worst) worst = err;
  }
  const bool edge = tslt::pow_exp(0.0f, table) == 1.0 && tslt::pow_exp(-0.0f, table) == 1.0 && table[0] == 0x3FF0000000000000ull;
  std::printf("max_ulp %.4f edge %d\n", worst, edge ? 1 : 0);
  return 0;
}
