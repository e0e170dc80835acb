// Finding a workgroup's m-tile from the device-side group offsets, without a kernel
// that writes a tile prefix first.
#pragma once
#include "common.h"

namespace moe {

struct MTile {
  int e;          // expert
  int nt;         // n-tile
  int row0;       // first grouped row of the tile
  int row_stop;   // end of the tile's rows
};

// Tile L of the experts' tiles in order: expert e has ceil(rows / BM) m-tiles, its 32-row
// blocks shared out evenly among them (BM % 32 = 0, so none exceeds BM rows), times NT
// n-tiles; false when there are not that many tiles.
// Inside an expert, the m-tiles of one n-tile, which share its weight panel, come 8 tiles
// apart, so that workgroups dealt round-robin to the 8 XCDs run them one after another on
// the same XCD and its L2 serves the panel; 8 n-tiles run side by side.
// Wave-uniform L and result; every lane of the wavefront must call it.  64 experts per
// pass: one load of their offsets, a scan over the lanes, and a ballot for the lane whose
// tiles hold L.
template <int BM>
__device__ __forceinline__ bool locate_tile(const int32_t* __restrict__ offsets, int E, int NT, int L, MTile* t) {
  const int q = L / NT;
  const int lane = threadIdx.x & (kWave - 1);
  int before = 0;
  for (int c0 = 0; c0 < E; c0 += kWave) {
    const int i = c0 + lane;
    const int beg = offsets[min(i, E)], end = offsets[min(i + 1, E)];   // equal past the last expert
    const int mt = (end - beg + BM - 1) / BM;
    int x = mt;
#pragma unroll
    for (int d = 1; d < kWave; d <<= 1) {
      const int y = __shfl_up(x, d);
      if (lane >= d) x += y;
    }
    const int first = before + x - mt;
    const uint64_t hit = __ballot(q >= first && q < first + mt);
    if (hit != 0ull) {
      const int l = __builtin_ctzll(hit);
      t->e = c0 + l;
      const int mt_e = __builtin_amdgcn_readlane(mt, l);
      const int local = L - __builtin_amdgcn_readlane(first, l) * NT;
      const int group = local / (kNumXcd * mt_e);                 // of 8 n-tiles, fewer at the end
      const int width = min(kNumXcd, NT - group * kNumXcd);
      const int rem = local - group * kNumXcd * mt_e;
      t->nt = group * kNumXcd + rem % width;
      const int mt_i = rem / width;
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
