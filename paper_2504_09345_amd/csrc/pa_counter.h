// Arrival counters of the parts of a cut item: the arithmetic, over any atomic
// 64-bit word (plain C++, so that it also runs on the host).
//
// A counter is 0 between calls, and a part counts with one fetch-and-add of
// the call's step, an odd number drawn anew for each call: a word v stands for
// v * step^-1 parts modulo 2^64.  What does not stand for fewer parts than the
// item has was not left by this call's parts: memory never used for counters
// before, a counter that the caller's other use of the workspace wrote over,
// wholly or in a few bytes, or what calls that overlapped on one workspace
// left.  (Of the 2^64 words, the item's few numbers of parts have one each, and
// which they are changes with every call.)  The parts that meet such a word put
// 0 in its place and count again, so nothing needs clearing beforehand and no
// call depends on what an earlier one left.
#pragma once

#include <stdint.h>

namespace pa {

struct CounterKey {
  uint64_t step;     // odd
  uint64_t inverse;  // step * inverse = 1 modulo 2^64
};

// Key of a call, from a number that no other call of the process has (mixed,
// so that the steps of successive calls have no small common multiples).
constexpr CounterKey counter_key(uint64_t call) {
  uint64_t x = call + 0x9e3779b97f4a7c15ull;
  x = (x ^ (x >> 30)) * 0xbf58476d1ce4e5b9ull;
  x = (x ^ (x >> 27)) * 0x94d049bb133111ebull;
  x = (x ^ (x >> 31)) | 1;
  uint64_t inv = x;  // Newton's iteration doubles the correct low bits, 3 to begin with
  for (int i = 0; i < 5; ++i) inv *= 2 - x * inv;
  return CounterKey{x, inv};
}

// Whether v stands for fewer than n parts.
constexpr bool counter_valid(uint64_t v, const CounterKey& key, int n) { return v * key.inverse < (uint64_t)n; }

// Count one of n parts and tell whether it is the last; the last leaves 0.
// Word: fetch_add(x) -> old value; swap(expected, x): compare-and-swap, which
// puts the present value into expected where it fails; store(x).
template <typename Word>
constexpr bool counter_arrive(Word& word, const CounterKey& key, int n) {
  uint64_t old = word.fetch_add(key.step);
  while (!counter_valid(old, key, n)) {
    // (a failed swap met another part's change; each part changes the word a
    // bounded number of times, and once valid it stays so)
    uint64_t now = old + key.step;
    while (!counter_valid(now, key, n) && !word.swap(now, 0)) {
    }
    old = word.fetch_add(key.step);
  }
  const bool last = old * key.inverse == (uint64_t)(n - 1);
  if (last) word.store(0);
  return last;
}

}  // namespace pa
