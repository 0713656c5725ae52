// The bin of a value among `bins` bins of equal width 1 / scale, of which the first and the last take whatever lies beyond: `above` is
// its distance from the first one's lower edge.  fp32 multiplication, minimum and truncation are monotone, which is all that a
// sort's bins have to be.  (The minimum comes before the conversion: a distance may be any number of bins, or infinite.)
#pragma once
#include "exp64.h"

namespace tslt {

TSLT_HD int value_bin_of(float above, float scale, int bins) {
  const int b = int(__builtin_fminf(above * scale, float(bins - 1)));
  return b < 0 ? 0 : b;
}

}  // namespace tslt
