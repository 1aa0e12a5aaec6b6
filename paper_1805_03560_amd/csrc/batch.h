// Which scratch buffer a batch of right-hand sides works in.  Buffers hold 1, 2, 4, 8 or 16 right-hand sides
// (class k: 2^k), are made when a call first needs them and stay where they are until the context goes: a
// captured graph keeps their addresses, so none is outgrown, freed or moved.  All of them together take less
// than twice the largest.
#pragma once

namespace whmc {

constexpr int kBatchClasses = 5;

struct BatchClass {
  int cls, n;   // the buffer and how many of the right-hand sides it takes
};

inline int batch_class_of(int n) {
  int k = 0;
  while ((1 << k) < n) ++k;
  return k;
}

// For n <= 16 right-hand sides: the smallest buffer there is (bit k of have: class k) that holds them; else a
// new one of their class, or, if none can be made, the largest there is with as many as it holds (have != 0).
inline BatchClass batch_class(unsigned have, int n, bool can_make) {
  const int want = batch_class_of(n);
  for (int k = want; k < kBatchClasses; ++k)
    if ((have >> k) & 1u) return {k, n};
  if (can_make) return {want, n};
  int k = want;
  while (k > 0 && !((have >> k) & 1u)) --k;
  return {k, 1 << k};
}

}  // namespace whmc
