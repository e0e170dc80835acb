// How the launches are sized: which form of a kernel a call takes.  Plain C++, no HIP
// dependency, so that the rules can be evaluated on a host.
#pragma once
#include <cstdint>

namespace moe {

// One-block permute (up to 16384 assignments): groups of 64 that each of its 16 wavefronts
// takes, a constant of the kernel: the next built size up.  Sizes 6 and 12 because a third
// of the groups empty shows: 8200 assignments over 256 experts take 21.1 us in 16 groups,
// 17.4 in 12, and 5000 13.0 in 8, 11.9 in 6.
inline int permute_small_iters(int64_t R) {
  for (int n : {1, 2, 4, 6, 8, 12})
    if (R <= int64_t(n) * 1024) return n;
  return 16;
}

}  // namespace moe
