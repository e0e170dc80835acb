// Finding a workgroup's m-tile from the device-side group offsets, without a kernel
// that writes a tile prefix first.
#pragma once
#include "common.h"
#include "launch_rules.h"

namespace moe {

struct MTile {
  int e;          // expert
  int nt;         // n-tile
  int row0;       // first grouped row of the tile
  int row_stop;   // end of the tile's rows
};

inline dim3 tile_dim(int64_t tiles) {
  const TileGrid g = tile_grid(tiles);
  return dim3(g.x, g.y);
}

// Number of this workgroup in a tile_grid() launch.  (gridDim.x in the constant's place would be
// read from memory, and cost the smallest fp32 layer 3%.)
__device__ __forceinline__ int tile_workgroup() { return int(blockIdx.y * kTileGridX + blockIdx.x); }

// The tile of workgroup b, false when it has none.  Expert e has ceil(rows / BM) m-tiles,
// its 32-row blocks shared out evenly among them (BM % 32 = 0, so none exceeds BM rows),
// times NT n-tiles; tiles are listed by expert, n-tile, m-tile, and workgroups, dealt
// round-robin to the 8 XCDs (b on XCD b % 8), take that list in eight contiguous parts:
// an XCD's workgroups share one expert's activation rows (and the m-tiles of one n-tile
// its weight panel) through its L2.
// Wave-uniform b and result; every lane of the wavefront must call it.  64 experts per
// pass: one load of their offsets, a scan over the lanes, and a ballot for the lane whose
// tiles hold the workgroup's.
template <int BM>
__device__ __forceinline__ bool locate_tile(const int32_t* __restrict__ offsets, int E, int NT, int b, MTile* t) {
  const int lane = threadIdx.x & (kWave - 1);
  int beg = 0, end = 0, mt = 0, x = 0;
  auto scan = [&](int c0) {          // the m-tiles of 64 experts, and their inclusive sum
    const int i = c0 + lane;
    beg = offsets[min(i, E)];
    end = offsets[min(i + 1, E)];    // equal past the last expert
    mt = (end - beg + BM - 1) / BM;
    x = mt;
#pragma unroll
    for (int d = 1; d < kWave; d <<= 1) {
      const int y = __shfl_up(x, d);
      if (lane >= d) x += y;
    }
  };
  int mtiles = 0;
  for (int c0 = 0; c0 < E; c0 += kWave) {
    scan(c0);
    mtiles += __builtin_amdgcn_readlane(x, kWave - 1);
  }
  const int total = mtiles * NT;
  const int per = (total + kNumXcd - 1) / kNumXcd;
  const int L = (b % kNumXcd) * per + b / kNumXcd;
  if (b / kNumXcd >= per || L >= total) return false;
  const int q = L / NT;
  int before = 0;
  for (int c0 = 0; c0 < E; c0 += kWave) {
    if (E > kWave) scan(c0);
    const int first = before + x - mt;
    const uint64_t hit = __ballot(q >= first && q < first + mt);
    if (hit != 0ull) {
      const int l = __builtin_ctzll(hit);
      t->e = c0 + l;
      const int mt_e = __builtin_amdgcn_readlane(mt, l);
      const int local = L - __builtin_amdgcn_readlane(first, l) * NT;
      t->nt = local / mt_e;
      const int mt_i = local % mt_e;
      const int row_beg = __builtin_amdgcn_readlane(beg, l), row_end = __builtin_amdgcn_readlane(end, l);
      const int64_t nb = (row_end - row_beg + kTileRowBlock - 1) / kTileRowBlock;
      t->row0 = row_beg + kTileRowBlock * int(mt_i * nb / mt_e);
      t->row_stop = min(row_end, row_beg + kTileRowBlock * int((mt_i + 1) * nb / mt_e));
      return true;
    }
    before = __builtin_amdgcn_readlane(before + x, kWave - 1);
  }
  return false;
}

}  // namespace moe
