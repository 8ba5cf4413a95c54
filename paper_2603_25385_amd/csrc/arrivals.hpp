// Counts of workgroups in words that nobody clears: a word is {launch tag, count}, and one that carries another launch's
// tag, or any other data, counts as zero.
#pragma once

namespace glowq {

constexpr int ARRIVAL_BITS = 4;      // of the count
// (60 bits of the tag: the words lie where calls over other units put their partial results, and a 32-bit float agrees
// with 28 bits of a tag once in 2^28)
__host__ __device__ inline unsigned long long arrival_key(unsigned long long launch_tag) { return (launch_tag >> 1) << ARRIVAL_BITS; }
// the workgroups that the word says have arrived
__host__ __device__ inline unsigned arrivals(unsigned long long word, unsigned long long key) {
  constexpr unsigned long long COUNT = (1ull << ARRIVAL_BITS) - 1;
  return (word & ~COUNT) == key ? (unsigned)(word & COUNT) : 0u;
}

}  // namespace glowq
