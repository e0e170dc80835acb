// Finding a workgroup's m-tile from the device-side group offsets, without a kernel
// that writes a tile prefix first.
#pragma once
#include "common.h"

namespace moe {

struct MTile {
  int e;          // expert
  int row0;       // first grouped row of the tile
  int row_stop;   // end of the tile's rows
};

// m-tile q of the experts' tiles in order, ceil(rows / BM) tiles of BM rows each (the
// last one shorter); false when there are not that many.  Wave-uniform q and result;
// every lane of the wavefront must call it.  64 experts per pass: one load of their
// offsets, a scan over the lanes, and a ballot for the lane whose tiles hold q.
template <int BM>
__device__ __forceinline__ bool locate_mtile(const int32_t* __restrict__ offsets, int E, int q, MTile* t) {
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
      t->row0 = __builtin_amdgcn_readlane(beg, l) + (q - __builtin_amdgcn_readlane(first, l)) * BM;
      t->row_stop = min(__builtin_amdgcn_readlane(end, l), t->row0 + BM);
      return true;
    }
    before = __builtin_amdgcn_readlane(before + x, kWave - 1);
  }
  return false;
}

}  // namespace moe
