// The bin of a value among `bins` bins of equal width 1 / scale, of which the first and the last take whatever lies beyond: `above` is
// its distance from the first one's lower edge.  fp32 multiplication, minimum and truncation are monotone, which is all that a
// sort's bins have to be.  (The bounds come before the conversion: a distance may be any number of bins, or infinite, or, where the width
// is, none at all.  One instruction for both of them.)
#pragma once
#include "exp64.h"

namespace tslt {

TSLT_HD int value_bin_of(float above, float scale, int bins) {
#if defined(__HIP_DEVICE_COMPILE__)
  return int(__builtin_amdgcn_fmed3f(above * scale, 0.0f, float(bins - 1)));
#else
  return int(__builtin_fminf(__builtin_fmaxf(above * scale, 0.0f), float(bins - 1)));
#endif
}

}  // namespace tslt
