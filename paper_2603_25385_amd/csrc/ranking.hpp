// The order of the singular values: descending, equal values by their row.
#pragma once

namespace glowq {

// Row b, value o, comes before row a, value s.  NaN counts as less than every number and as equal to NaN, so that the
// ranks (how many rows come before) are a permutation whatever the values are: they index rows and columns afterwards,
// and weights that are not finite make every value NaN.
__host__ __device__ inline bool ranks_before(double o, int b, double s, int a) {
  const bool o_nan = o != o, s_nan = s != s;
  if (o_nan || s_nan) return o_nan && s_nan ? b < a : s_nan;
  return o > s || (o == s && b < a);
}

}  // namespace glowq
