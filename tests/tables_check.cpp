// Host check of what the kernels' tables are made of: the copy of exp64.h's power table that workgroups read, entry for entry,
// and exp64_pair, which makes both signs of bfloat16's table, against libm over the table's range.
#include <algorithm>
#include <cmath>
#include <cstdint>
#include <cstdio>
#include "exp64.h"
#define __device__
#define __align__(n) alignas(n)
#include "pow_table.h"

int main() {
  int differ = 0;
  for (int i = 0; i < tslt::kPowEntries; ++i) differ += tslt::kPowTable[i] != tslt::pow_entry(i);
  double worst = 0.0;
  uint64_t s = 0x9E3779B97F4A7C15ull;
  for (int i = 0; i < 2000000; ++i) {
    s ^= s << 13; s ^= s >> 7; s ^= s << 17;
    const double u = double(s >> 11) * (1.0 / 9007199254740992.0);
    const float x = float(i % 3 == 0 ? 600.0 * u : (i % 3 == 1 ? 40.0 * u : std::ldexp(u, -14 * int(s & 1))));
    double got[2];
    tslt::exp64_pair(double(x), got[0], got[1]);
    for (int k = 0; k < 2; ++k) {
      const long double want = expl(k == 0 ? (long double)x : -(long double)x);
      int e;
      std::frexp(double(want), &e);
      worst = std::max(worst, std::fabs(double((long double)got[k] - want)) / std::ldexp(1.0, e - 53));
    }
  }
  std::printf("differ %d max_ulp %.4f\n", differ, worst);
  return 0;
}
