// The order of the singular values: descending, equal values by their row.
#pragma once

namespace glowq {

// Row b, value o, comes before row a, value s.  NaN counts as less than every number and as equal to NaN, so that the
// ranks (how many rows come before) are a permutation whatever the values are: they index rows and columns afterwards,
// and weights that are not finite make every value NaN.
__host__ __device__ inline bool ranks_before(double o, int b, double s, int a) {
  return s != s ? o == o || b < a : o > s || (o == s && b < a);
}

}  // namespace glowq
