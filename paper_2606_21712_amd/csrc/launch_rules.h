// How the launches are sized: which form of a kernel a call takes.  Plain C++, no HIP
// dependency, so that the rules can be evaluated on a host.
#pragma once
#include <cstdint>

namespace moe {

// Grid of the kernels with one workgroup per tile: at least `tiles` workgroups, numbered
// y * kTileGridX + x, in eight parts (number n runs on XCD n % 8).  Two dimensions once one
// would pass the launch's limit of 2^32 threads along it (workgroups have at most 512): fp32
// gate/up tiles of a workspace of 137 GB are 2^24.
struct TileGrid {
  unsigned x, y;
};
constexpr unsigned kTileGridX = 1u << 22;
inline TileGrid tile_grid(int64_t tiles) {
  const int64_t n = (tiles + 7) / 8 * 8;
  if (n <= kTileGridX) return TileGrid{unsigned(n), 1};
  return TileGrid{kTileGridX, unsigned((n + kTileGridX - 1) / kTileGridX)};
}

// One-block permute (up to 16384 assignments): groups of 64 that each of its 16 wavefronts
// takes, a constant of the kernel: the next built size up.  Sizes 6 and 12 because a third
// of the groups empty shows: 8200 assignments over 256 experts take 21.1 us in 16 groups,
// 17.4 in 12, and 5000 13.0 in 8, 11.9 in 6.
inline int permute_small_iters(int64_t R) {
  for (int n : {1, 2, 4, 6, 8, 12})
    if (R <= int64_t(n) * 1024) return n;
  return 16;
}

// Sixteen-byte vectors of each row that a lane of combine loads at once: 32 loads in flight
// with k rows (k = 1, 2: 8 or 16).
constexpr int combine_unroll(int k) { return k == 1 || k == 2 || k == 4 ? 8 : 2; }

// Column split of combine: a token's row (nvec vectors) is cut into this many parts, one
// wavefront each, every one with a vector per lane at least.
//   Large batches run enough wavefronts with a few vectors per lane each (measured cold, %
//   of 8 TB/s: memory-constrained 71 -> 76 with 2 parts, Mixtral-shaped 32K tokens 75 -> 77
//   with 4, DeepSeek-shaped 65 -> 70 with 8).
//   Small ones are bound by the latency of a row.  Where a whole row is several passes of a
//   lane (loads, sums, store), up to 4096 wavefronts run them side by side (96 tokens, k 8,
//   H 7168: 16.9 -> 7.7 us cold; 2048: 53.4 -> 51.8).  Where it is one pass only the loads
//   per lane shrink, and that pays while the wavefronts stay under three per SIMD (509
//   tokens, H 4096, k 4: 9.8 us, 8.6 in 4 parts, 9.8 in 8); from 640 tokens whole rows are
//   the fastest or level (1024, H 4096, k 4: 12.0 us, 13.7 in 4; 2048, k 2: 9.4, in 2 11.7).
//   Batches between keep whole rows.
inline int combine_splits(int64_t T, int k, int nvec) {
  constexpr int kWave = 64;
  const bool one_pass = nvec <= kWave * combine_unroll(k);
  const int64_t small = !one_pass ? 4096 : T < 640 ? 2800 : 0;
  int splits = 1;
  if (T < 4096)
    while (splits < 16 && nvec / (2 * splits) >= kWave && T * (2 * splits) <= small) splits *= 2;
  else if (T >= 8192)
    while (splits < 8 && nvec / (2 * splits) >= kWave && T * splits < (int64_t(1) << 30) &&
           (nvec / splits > 4 * kWave || T * splits < 131072))
      splits *= 2;
  return splits;
}

}  // namespace moe
