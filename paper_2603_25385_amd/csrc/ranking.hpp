// The order of the singular values: descending, equal values by their row.
#pragma once

namespace glowq {

// How many of the n rows come before row a; value(b) is row b's value.  NaN counts as less than every number and as equal to
// NaN, so that the ranks are a permutation whatever the values are: they index rows and columns afterwards, and weights
// that are not finite make every value NaN.
template <class V> __host__ __device__ inline int rank_of(V value, int n, int a) {
  const double s = value(a);
  int rank = 0;
  if (s == s) {
    for (int b = 0; b < n; ++b) rank += value(b) > s || (value(b) == s && b < a) ? 1 : 0;
  } else {
    for (int b = 0; b < n; ++b) rank += value(b) == value(b) || b < a ? 1 : 0;
  }
  return rank;
}

}  // namespace glowq
