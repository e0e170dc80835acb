// The fp32 layer's grouped SwiGLU FFN on gfx950, on the fp32 matrix cores.
//
// Same mathematics and operand order as the bf16 GEMMs (ffn.hip): the weight tile is
// the MFMA A operand, the activation tile the B operand, GEMM-1 holds gate and up rows
// of the same features so that silu(g) * u is formed in registers.  Products and sums
// are fp32 (v_mfma_f32_32x32x2_f32); silu uses the full-precision expf and division.
//
// What bounds it: the fp32 matrix rate (256 flop per cycle and compute unit, an eighth of
// a bf16 step's rate for the same bytes), and short of that evenness.  Tiles of 64 rows x
// 64 weight rows x 32 k per step, four wavefronts of 32 x 32, two stages of 16 KB, four
// workgroups per compute unit, whose MFMAs run through each other's waits and barriers while
// all four are there.  One launch covers every expert's tiles: the grid holds the host's
// bound on them, and the workgroups past the device's count leave.
// Measured against 64 x 64 tiles of vector FMAs staged through registers: 2000 tokens,
// H 1024, 8 experts, top-2, F 2048: GEMM-1 477 -> 338 us (99 TFLOP/s), GEMM-2 305 -> 196 us
// (86); 256 tokens, H 256, F 512: 37 -> 9.8 us and 35 -> 6.5 us (on the small kernel below).
// The library's dense fp32 matmul reaches 151 TFLOP/s at 8192^3.  At 2000 tokens the down
// projection has 1040 to 1088 tiles for 1024 places, gate/up 4160 to 4352: the 16 to 64 over
// a whole round run alone at the end, with every wait exposed.  With 64 x 128 tiles (three
// workgroups per compute unit) some compute units held three of its 512 and some one: 232 us.
#include "group_locate.h"
#include "lds_stage.h"
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
  if (!locate_tile<kFM>(p.offsets, p.E, p.ntiles, tile_workgroup(), &tile)) return;     // uniform across the block
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

// Small layers, whose tiles of 64 x 64 leave compute units idle.  The chain of k steps of one
// tile bounds them, so the tile is 32 rows x 32 weight rows (GEMM-1: 16 gate + 16 up) and
// its four wavefronts split k, 32 at a time in turn: a quarter of the steps.  Each takes
// its own part of both operands through two LDS stages of its own, without a barrier, and
// the four sums meet in LDS at the end, added in wavefront order.  A step asks to wait for its
// own stage only; the compiler does not tell the refill of a stage just read from the other's
// loads and waits for all of them at every second step.  Measured, 64 x 64 ->
// this: 512 rows over 8 experts, F 512, H 256, down 14.3 -> 9.0 us; 2 rows, H 4096,
// F 1024, gate/up 74 -> 28 us, down 22 -> 11 us.
template <bool SWIGLU>
__global__ __launch_bounds__(kFThreads, 2) void grouped_gemm_f32_small_kernel(GemmArgsF p) {
  constexpr int kWaveStage = 2 * 32 * kFRow;           // a wavefront's stage: 32 weight rows, 32 activation rows
  __shared__ __attribute__((aligned(1024))) uint8_t st0[4 * kWaveStage];
  __shared__ __attribute__((aligned(1024))) uint8_t st1[4 * kWaveStage];
  const int tid = threadIdx.x;
  const int lane = tid & (kWave - 1);
  const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  if (p.E < 0) {                  // never taken: keeps the DMA-filled stages' reads
    st0[tid] = 0;
    st1[tid] = 0;
  }
  MTile tile;
  if (!locate_tile<32>(p.offsets, p.E, p.ntiles, tile_workgroup(), &tile)) return;      // uniform across the block
  const int e = tile.e, row0 = tile.row0, row_stop = tile.row_stop;
  const int K = p.K, N = p.N;
  const int n0 = tile.nt * (SWIGLU ? 16 : 32);

  // DMA: pass i fills rows 8 i .. 8 i + 7 of an operand; rows past the tile read its first
  const int qrow = lane >> 3, qpos = lane & 7;
  const float* aptr[4];
  const float* wptr[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int r = i * 8 + qrow;
    const int grow = row0 + r < row_stop ? row0 + r : row0;
    const int64_t arow = p.gather != nullptr ? int64_t(p.gather[grow]) : int64_t(grow);
    aptr[i] = p.act + arow * K + fswz(r, qpos) * 4;
    const float* w = SWIGLU && (r & 16) ? p.w1 : p.w0;
    wptr[i] = w + (int64_t(e) * N + n0 + (SWIGLU ? (r & 15) : r)) * K + fswz(r, qpos) * 4;
  }
  const int KT = K / kFK;
  const int mine = (KT - wave + 3) / 4;                // k steps of this wavefront: wave, wave + 4, ...
  const int dst = opaque_s(wave * kWaveStage);
  auto issue = [&](uint8_t* stage, int i) {
    const int k = (min(i, mine - 1) * 4 + wave) * kFK;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      __builtin_amdgcn_global_load_lds(wptr[j] + k, stage + (dst + j * 1024), 16, 0, 0);
      __builtin_amdgcn_global_load_lds(aptr[j] + k, stage + (dst + 4096 + j * 1024), 16, 0, 0);
    }
  };
  const int rrow = lane & 31, khalf = lane >> 5;
  int at[4];
#pragma unroll
  for (int s = 0; s < 4; ++s) at[s] = opaque_v(wave * kWaveStage + rrow * kFRow + fswz(rrow, 2 * s + khalf) * 16);
  f32x16 acc;
#pragma unroll
  for (int q = 0; q < 16; ++q) acc[q] = 0.f;
  auto step = [&](uint8_t* cur, int i) {
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_waitcnt(wait_vm(8));            // this step's loads, sent before the next step's
    __builtin_amdgcn_sched_barrier(0);
    f32x4 xf[4], wf[4];
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      wf[s] = *reinterpret_cast<const f32x4*>(cur + at[s]);
      xf[s] = *reinterpret_cast<const f32x4*>(cur + (at[s] + 4096));
    }
#pragma unroll
    for (int s = 0; s < 4; ++s)
#pragma unroll
      for (int q = 0; q < 4; ++q) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(wf[s][q], xf[s][q], acc, 0, 0, 0);
    __builtin_amdgcn_sched_barrier(0);
    issue(cur, i + 2);                                 // (past the end the last step's again)
  };
  if (mine > 0) {
    issue(st0, 0);
    __builtin_amdgcn_sched_barrier(0);                 // the waits count on this order
    issue(st1, 1);
    int i = 0;
    for (; i + 2 <= mine; i += 2) {
      step(st0, i);
      step(st1, i + 1);
    }
    if (i < mine) step(st0, i);
  }
  __builtin_amdgcn_s_waitcnt(wait_vm(0));              // no load may still be on its way into this LDS
  f32x4* sums = reinterpret_cast<f32x4*>(st0);         // wavefront w's [4 blk][64 lanes] at w kWaveStage
#pragma unroll
  for (int blk = 0; blk < 4; ++blk)
    sums[wave * (kWaveStage / 16) + blk * kWave + lane] =
        f32x4{acc[4 * blk], acc[4 * blk + 1], acc[4 * blk + 2], acc[4 * blk + 3]};
  __syncthreads();
  auto total = [&](int blk) {
    f32x4 t = sums[blk * kWave + lane];
#pragma unroll
    for (int w = 1; w < 4; ++w) t += sums[w * (kWaveStage / 16) + blk * kWave + lane];
    return t;
  };
  // wavefront w stores block w: weight rows 8 w + 4 khalf + {0..3} of activation row rrow
  const int row = row0 + rrow;
  if (SWIGLU) {
    if (wave >= 2) return;
    const f32x4 g = total(wave), u = total(wave + 2);
    f32x4 v;
#pragma unroll
    for (int q = 0; q < 4; ++q) v[q] = (g[q] / (1.0f + expf(-g[q]))) * u[q];
    if (row < row_stop) *reinterpret_cast<f32x4*>(p.out + int64_t(row) * N + n0 + wave * 8 + khalf * 4) = v;
  } else {
    const f32x4 v = total(wave);
    if (row < row_stop) *reinterpret_cast<f32x4*>(p.out + int64_t(row) * N + n0 + wave * 8 + khalf * 4) = v;
  }
}

// The small kernel where its tiles are no more than run at once, two workgroups per compute
// unit (by LDS).  Past that a compute unit runs tiles in turn and the larger tile, which reads
// half as much per product, is as fast or faster.  8 experts, small against 64 x 64 (in us) by
// tiles of the small kernel: 320 (1024 rows, K 512) 12.1 and 14.5, 448 (200 rows, K 2048)
// 26.1 and 39.2, 576 (2048 rows, K 512) 16.6 and 15.2, 768 (512 rows, K 256) 13.2 and 11.4.
template <bool SWIGLU>
void launch_gemm_f32(const char* name, GemmArgsF a, int64_t R, int num_cu, hipStream_t s) {
  const int64_t live = R < a.E ? R : a.E;
  const int64_t small = (R + live * 31) / 32 * (a.N / (SWIGLU ? 16 : 32));
  if (small <= 2 * num_cu) {
    a.ntiles = a.N / (SWIGLU ? 16 : 32);
    MOE_LAUNCH(name, grouped_gemm_f32_small_kernel<SWIGLU>, tile_dim(small), dim3(kFThreads), s, a);
  } else {
    a.ntiles = a.N / (SWIGLU ? kFN / 2 : kFN);
    const int64_t mtiles = (R + live * (kFM - 1)) / kFM;
    MOE_LAUNCH(name, grouped_gemm_f32_kernel<SWIGLU>, tile_dim(mtiles * a.ntiles), dim3(kFThreads), s, a);
  }
}

}  // namespace

hipError_t launch_ffn_f32(const float* act, const int32_t* gather, const int32_t* offsets, int64_t R,
                          int E, int H, int F, const float* wg, const float* wu, const float* wd,
                          float* y_perm, float* h, int num_cu, hipStream_t s) {
  launch_gemm_f32<true>("ffn_gemm1_gate_up", GemmArgsF{act, gather, wg, wu, h, offsets, E, H, F, 0}, R, num_cu, s);
  launch_gemm_f32<false>("ffn_gemm2_down", GemmArgsF{h, nullptr, wd, nullptr, y_perm, offsets, E, F, H, 0}, R, num_cu,
                         s);
  return hipGetLastError();
}

}  // namespace moe
