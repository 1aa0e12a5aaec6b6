// Division of an index by a number fixed per lattice: a 32 x 32 -> 64 bit product and a shift instead
// of the 25-instruction integer division.  For 1 <= d < 2^31, s = ceil(log2 d) and
// m = floor(2^(31 + s) / d) + 1 (below 2^32), m d = 2^(31 + s) + e with 0 < e <= d <= 2^s, hence
// n m / 2^(31 + s) = n / d + n e / (d 2^(31 + s)), and for n < 2^31 the second term is below 1 / d:
// the floor is that of n / d.
#pragma once
#include <stdint.h>

#if defined(__HIP__)
#define WHMC_FD __host__ __device__ __forceinline__
#else
#define WHMC_FD inline
#endif

namespace whmc {

struct FastDiv {
  uint32_t m;
  int sh;
  WHMC_FD int div(int n) const { return (int)(((uint64_t)(uint32_t)n * m) >> sh); }
};

inline FastDiv fast_div(int d) {
  int s = 0;
  while ((1LL << s) < d) ++s;
  return {(uint32_t)((1ULL << (31 + s)) / (uint64_t)d + 1), 31 + s};
}

}  // namespace whmc
