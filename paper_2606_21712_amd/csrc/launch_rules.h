// How the launches are sized: which form of a kernel a call takes.  Plain C++, no HIP
// dependency, so that the rules can be evaluated on a host.
#pragma once
#include <cmath>
#include <cstdint>

#include "tiling.h"

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

// ---- the grouped GEMMs for small groups (ffn_stream.hip)

// Experts that R rows dealt evenly at random reach, and their average rows.
struct GroupLoad {
  double live;
  int64_t rows;
  GroupLoad(int64_t R, int E)
      : live(E > 1 ? E * -std::expm1(double(R) * std::log1p(-1.0 / E)) : 1.0), rows(int64_t(double(R) / live + 0.999)) {}
};

inline int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }

// Whether one GEMM of the grouped FFN (K wide, N outputs per row) is faster on the streaming
// kernels than on the large-batch ones, without a compute-unit budget.  Only the mean group is
// known here; loads differ, so each line lies where even loads and lognormal ones (sigma
// 0.5 and 1) are faster on average.  Time streaming / large-batch, each shape even, then the
// slower of the uneven (H / F / experts):
//   Few tiles leave the large-batch kernels' grid part empty, and there streaming wins far out.
//     MXFP8, tiles of 256 rows, fewer tiles than compute units: down 4096 / 4096 / 10 at 112
//       rows 0.85, 0.79, at 256 0.68, 0.71; 4096 / 14336 / 4 at 640 rows 0.72, 0.71.  A just full
//       grid: only up to 320 rows, where uneven loads spill into a second round (4096 / 14336 / 8
//       at 300 rows 1.14, 0.69; at 330 1.15, 1.13).
//     bf16, tiles of 320 rows, at most half as many tiles, as long as streaming's own tiles run
//       at once, one workgroup per compute unit: 4096 / 14336 / 8 down at 220 rows 0.77, 0.82,
//       256 0.73, 1.33, 300 1.20, 1.25; 4096 / 14336 / 4 down at 500 rows 0.70, 1.19.
//   Gate/up, bf16: 112 rows (7168 / 2048 / 64 0.87, 0.97; 4096 / 4096 / 64 0.87, 1.04); 144 while
//     the large-batch grid has less than four rounds, whose last is part empty (at 128 rows
//     4096 / 14336 / 8 0.78, 1.06; 5120 / 1536 / 32 0.83, 1.00; 2816 / 1408 / 60 0.88, 1.01);
//     beyond, it loses: 7168 / 2048 / 64 at 160 rows 1.15, 1.04.
//   Gate/up, MXFP8: 96 rows (7168 / 2048 / 64 0.85, 0.89; 4096 / 14336 / 8 0.91, 1.00; at 128 rows
//     1.09, 0.97 and 1.02, 1.09).
//   Down: as gate/up, except where the large-batch kernel is near its best rate:
//     more than four rounds of its tiles: 88 rows (7168 / 2048 / 64 at 80 rows 0.97, 1.06, MXFP8
//       0.96, 1.04, at 104 1.00, 1.07, MXFP8 at 96 0.98, 1.05), more than sixteen 32 (7168 / 2048 / 256 at 40 rows 1.00, 1.13);
//     short k loops, whose start and end a tile of few steps does not hide, once there are two
//       rounds: under 16 steps 40 rows, MXFP8 72 (2048 / 768 / 128 bf16 at 40 rows 0.96, 1.06, at
//       52 1.02, 1.10; MXFP8 2816 / 1408 / 60 at 64 rows 0.96, 0.97, at 96 1.01, 1.12), under 8
//       steps 24 (2048 / 768 / 128 MXFP8 at 24 rows 0.97, 1.04, at 52 1.11, 1.19).
inline bool stream_is_faster(int64_t R, int E, int K, int N, bool swiglu, bool fp8, int num_cu) {
  const GroupLoad l(R, E);
  const int64_t ntiles = ceil_div(N, swiglu ? kTileCols / 2 : kTileCols);
  const int64_t big = int64_t(l.live * double(ceil_div(l.rows, fp8 ? kTileRows : kTileRowsMax) * ntiles));
  const int steps = K * (fp8 ? 1 : 2) / 128;
  if (fp8) {
    if (big < num_cu || (big == num_cu && l.rows <= 320)) return true;
  } else if (2 * big <= num_cu) {
    // streaming tiles of 160 rows (from 321 rows 128); uneven groups have 0.4 more each than their mean says
    const int mr = l.rows <= 320 ? 160 : 128;
    const double mtiles = E == 1 ? double(ceil_div(l.rows, mr)) : double(l.rows) / mr + 0.4;
    if (l.live * mtiles * double(ntiles) <= num_cu) return true;
  }
  if (!swiglu) {
    if (big > 16 * num_cu) return l.rows <= 32;
    if (big > 4 * num_cu && l.rows > 88) return false;
    if (steps < 8 && big >= 2 * num_cu) return l.rows <= 24;
    if (steps < 16 && big >= 2 * num_cu) return l.rows <= (fp8 ? 72 : 40);
  }
  return l.rows <= (fp8 ? 96 : big < 4 * num_cu ? 144 : 112);
}

// The streaming kernels' tiles: 64 wn weight rows x mr activation rows, kg k groups, stages of the ring.
struct StreamTile {
  int wn, mr, kg, stages;
};

// Which tile.  More activation rows per tile read the weights fewer times and the
// activations less often, fewer give more workgroups; the lines lie where the mean group
// leaves its largest members inside one tile (a group cut in two reads its weights from L2
// twice).  Measured, us of one GEMM (M: H 4096, F 14336, 8 experts):
//   160 rows for means of 100 to 320: M down at 256 rows 289 (128 rows: 430); beyond that
//     128 rows (one expert, 2048 rows, H 7168, F 2048, gate/up: 114, 160 rows: 191);
//   fewer workgroups than two per compute unit: two k groups, which keep as many bytes in
//     flight on half the workgroups (M down at one row: 80 -> 52), and four on 64 weight
//     rows when even that leaves half the chip idle (one expert, F 2048, H 7168 at 8 rows,
//     gate/up: 31 -> 21).
inline StreamTile stream_tile(int64_t R, int E, int N, bool swiglu, bool fp8, int num_cu) {
  const GroupLoad l(R, E);
  auto workgroups = [&](int wn, int mr) {
    return int64_t(l.live * double(ceil_div(l.rows, mr)) * double(ceil_div(N, 64 * wn / (swiglu ? 2 : 1))));
  };
  if (!fp8 && l.rows > 100 && l.rows <= 320) {       // (three MXFP8 stages of 160 rows and their scales exceed the LDS)
    if (workgroups(4, 160) >= num_cu) return {4, 160, 1, 3};
    if (workgroups(2, 160) >= num_cu * 3 / 4) return {2, 160, 1, 4};
  }
  if (l.rows > 44) {
    if (workgroups(4, 128) >= num_cu) return {4, 128, 1, 3};
    if (workgroups(2, 128) >= num_cu * 3 / 4) return {2, 128, 1, 4};
  }
  const int mr = l.rows <= 16 ? 32 : 64;
  if (workgroups(2, mr) >= 2 * num_cu) return {2, mr, 1, 3};
  if (workgroups(2, mr) >= num_cu / 2) return {2, mr, 2, 3};
  return l.rows <= 16 ? StreamTile{1, 32, 4, 3} : StreamTile{1, 64, 2, 4};
}

// Whether a tile's weights bypass the caches (the nt policy): nothing reads them again soon when
// one m-tile holds the mean group.  Not for small weights, which the Infinity Cache may hold
// from one call to the next.  (Deciding per expert by its own m-tiles was slower: uneven
// loads gained 1 to 3% on average, but MXFP8 lost up to 10% in gate/up of H 7168, F 2048, 64
// experts at 80 to 120 rows, and 20% in down of H 4096, F 14336, 4 experts at 112 to 128.)
inline bool stream_nt(int64_t R, int E, int K, int N, bool swiglu, bool fp8, int mr) {
  const int64_t weight_bytes = int64_t(E) * N * K * (fp8 ? 1 : 2) * (swiglu ? 2 : 1);
  return weight_bytes >= (int64_t(128) << 20) && GroupLoad(R, E).rows <= mr;
}

}  // namespace moe
