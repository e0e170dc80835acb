// The fp32 layer's grouped SwiGLU FFN on gfx950, on the fp32 matrix cores.
//
// Same mathematics and operand order as the bf16 GEMMs (ffn.hip): the weight tile is
// the MFMA A operand, the activation tile the B operand, GEMM-1 holds gate and up rows
// of the same features so that silu(g) * u is formed in registers.  Products and sums
// are fp32 (v_mfma_f32_32x32x2_f32); silu uses the full-precision expf and division.
//
// What bounds it: the fp32 matrix rate (256 flop per cycle and compute unit, an eighth
// of a bf16 step's rate for the same bytes), so a plain two-stage pipeline is enough, and
// what is left is evenness: tiles of 64 rows x 64 weight rows x 32 k per step, four
// wavefronts of 32 x 32, 16 KB per stage, four workgroups per compute unit, whose MFMAs
// run through each other's barriers.  One launch covers every expert's tiles: the grid
// holds the host's bound on them, and the workgroups past the device's count leave.
// Measured against 64 x 64 tiles of vector FMAs staged through registers: 2000 tokens,
// H 1024, 8 experts, top-2, F 2048: GEMM-1 477 -> 338 us (99 TFLOP/s), GEMM-2 305 -> 196 us;
// 256 tokens, H 256, F 512: 37 -> 11 us and 35 -> 14 us.  The library's dense fp32 matmul
// reaches 151 TFLOP/s at 8192^3.  With 64 x 128 tiles (three workgroups per compute unit)
// some compute units held three of the 512 down-projection tiles and some one: 232 us.
#include "group_locate.h"
#include "moe_internal.h"

namespace moe {
namespace {

constexpr int kFM = 64;                     // activation rows per tile
constexpr int kFN = 64;                     // weight rows per tile (GEMM-1: 32 gate + 32 up)
constexpr int kFRow = 128;                  // bytes of one tile row in LDS: 32 fp32 of k
constexpr int kFK = kFRow / 4;
constexpr int kFThreads = 256;              // 4 wavefronts: 2 (m) x 2 (n)
constexpr int kFWBytes = kFN * kFRow;
constexpr int kFStage = kFWBytes + kFM * kFRow;
constexpr int kFPad = 2048;                 // 34 KB of LDS: at most four workgroups per compute unit
constexpr int kFWaitVm0 = 0x0F70;

struct GemmArgsF {
  const float* act;
  const int32_t* gather;          // [R] token of each grouped row, or null
  const float* w0;
  const float* w1;
  float* out;
  const int32_t* offsets;
  int E, K, N, ntiles;
};

// 16-byte chunk c of row r sits at chunk c ^ ((r >> 1) & 7): no bank conflicts for
// the 16-byte-per-lane operand reads.
__device__ __forceinline__ int fswz(int row, int chunk) { return chunk ^ ((row >> 1) & 7); }

template <bool SWIGLU>
__global__ __launch_bounds__(kFThreads, 4) void grouped_gemm_f32_kernel(GemmArgsF p) {
  __shared__ __attribute__((aligned(1024))) uint8_t st0[kFStage];
  __shared__ __attribute__((aligned(1024))) uint8_t st1[kFStage + kFPad];
  const int tid = threadIdx.x;
  const int lane = tid & (kWave - 1);
  const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  const int wm = wave >> 1, wn = wave & 1;
  if (p.E < 0) {                  // never taken: keeps the DMA-filled stages' reads
    st0[tid] = 0;
    st1[tid] = 0;
  }
  MTile tile;
  if (!locate_tile<kFM>(p.offsets, p.E, p.ntiles, int(blockIdx.x), &tile)) return;     // uniform across the block
  const int e = tile.e, nt = tile.nt, row0 = tile.row0, row_stop = tile.row_stop;
  const int K = p.K, N = p.N;
  const int n0 = nt * (SWIGLU ? kFN / 2 : kFN);

  // DMA: wavefront w's pass i fills the 1 KB block 4 i + w of an operand (8 rows); lane q
  // lands at row 8 blk + q / 8, chunk position q % 8.  Rows past the tile read its
  // first row: their products land only in results that are never stored.  GEMM-1's
  // weight rows 32 j + r are 16 gate rows (r < 16) and the up rows of the same
  // features n0 + 16 j + r % 16, so one 32 x 32 result holds both.
  const int qrow = lane >> 3, qpos = lane & 7;
  const float* aptr[2];
  const float* wptr[2];
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int r = (4 * i + wave) * 8 + qrow;
    const int grow = row0 + r < row_stop ? row0 + r : row0;
    const int64_t arow = p.gather != nullptr ? int64_t(p.gather[grow]) : int64_t(grow);
    aptr[i] = p.act + arow * K + fswz(r, qpos) * 4;
    const float* w = SWIGLU && (r & 16) ? p.w1 : p.w0;
    const int n = n0 + (SWIGLU ? (r >> 5) * 16 + (r & 15) : r);
    wptr[i] = w + (int64_t(e) * N + n) * K + fswz(r, qpos) * 4;
  }
  auto issue = [&](uint8_t* stage, int kt) {
    const int k = kt * kFK;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      __builtin_amdgcn_global_load_lds(wptr[i] + k, stage + (4 * i + wave) * 1024, 16, 0, 0);
      __builtin_amdgcn_global_load_lds(aptr[i] + k, stage + kFWBytes + (4 * i + wave) * 1024, 16, 0, 0);
    }
  };

  const int rrow = lane & 31, khalf = lane >> 5;
  const int arow = wm * 32 + rrow;
  const int wrow = wn * 32 + rrow;
  f32x16 acc;
#pragma unroll
  for (int q = 0; q < 16; ++q) acc[q] = 0.f;
  // Sub-step s holds 8 of k: lane half h takes chunk 2 s + h, and its MFMA i multiplies
  // k = 8 s + i (half 0) and 8 s + 4 + i (half 1) of both operands.
  auto compute = [&](const uint8_t* stage) {
    f32x4 xf[4], wf[4];
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      const int c = 2 * s + khalf;
      wf[s] = *reinterpret_cast<const f32x4*>(stage + wrow * kFRow + fswz(wrow, c) * 16);
      xf[s] = *reinterpret_cast<const f32x4*>(stage + kFWBytes + arow * kFRow + fswz(arow, c) * 16);
    }
#pragma unroll
    for (int s = 0; s < 4; ++s)
#pragma unroll
      for (int i = 0; i < 4; ++i) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(wf[s][i], xf[s][i], acc, 0, 0, 0);
  };
  const bool active = row0 + wm * 32 < row_stop;                 // uniform across the wave
  const int KT = K / kFK;                                        // even: K % 64 = 0
  auto step = [&](uint8_t* cur, uint8_t* nxt, int kt) {
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_waitcnt(kFWaitVm0);
    __syncthreads();
    __builtin_amdgcn_sched_barrier(0);
    if (kt + 1 < KT) issue(nxt, kt + 1);
    if (active) compute(cur);
  };
  issue(st0, 0);
  for (int kt = 0; kt < KT; kt += 2) {
    step(st0, st1, kt);
    step(st1, st0, kt + 1);
  }

  // lane holds weight rows 8 blk + 4 khalf + {0..3} of the wavefront's 32, for row rrow
  const int row = row0 + arow;
  if (row >= row_stop) return;
  float* orow = p.out + int64_t(row) * N + n0;
  if (SWIGLU) {
#pragma unroll
    for (int blk = 0; blk < 2; ++blk) {
      f32x4 v;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const float g = acc[blk * 4 + q];
        v[q] = (g / (1.0f + expf(-g))) * acc[blk * 4 + 8 + q];
      }
      *reinterpret_cast<f32x4*>(orow + wn * 16 + blk * 8 + khalf * 4) = v;
    }
  } else {
#pragma unroll
    for (int blk = 0; blk < 4; ++blk) {
      f32x4 v;
#pragma unroll
      for (int q = 0; q < 4; ++q) v[q] = acc[blk * 4 + q];
      *reinterpret_cast<f32x4*>(orow + wn * 32 + blk * 8 + khalf * 4) = v;
    }
  }
}

}  // namespace

hipError_t launch_ffn_f32(const float* act, const int32_t* gather, const int32_t* offsets, int64_t R,
                          int E, int H, int F, const float* wg, const float* wu, const float* wd,
                          float* y_perm, float* h, hipStream_t s) {
  const int64_t mtiles_upper = (R + int64_t(E) * (kFM - 1)) / kFM;
  GemmArgsF a1{act, gather, wg, wu, h, offsets, E, H, F, F / (kFN / 2)};
  MOE_LAUNCH("ffn_gemm1_gate_up", grouped_gemm_f32_kernel<true>, dim3(tile_grid(mtiles_upper * a1.ntiles)),
             dim3(kFThreads), s, a1);
  GemmArgsF a2{h, nullptr, wd, nullptr, y_perm, offsets, E, F, H, H / kFN};
  MOE_LAUNCH("ffn_gemm2_down", grouped_gemm_f32_kernel<false>, dim3(tile_grid(mtiles_upper * a2.ntiles)),
             dim3(kFThreads), s, a2);
  return hipGetLastError();
}

}  // namespace moe
