// Grouped SwiGLU FFN for small expert groups (decode and short prefill batches), bf16
// and MXFP8, on gfx950.
//
// With up to some hundred rows per expert the FFN is a stream of the experts' weights:
// each weight is used by few rows, and the time is weight bytes over the HBM read rate.
// What counts is the bytes in flight per compute unit (about 64 KB at 6 TB/s and 2-3 us
// of loaded latency), all the time.  The large-batch kernels keep two stages and wait
// for one to arrive in full at every k step, so the requests in flight drop to nothing
// once per step, and again at every tile's start and end.  Here:
//   - a ring of S >= 3 LDS stages (128 bytes of k per row, direct global -> LDS loads);
//     a step waits for its own stage only, S - 2 more stay in flight behind it;
//   - small workgroups (four wavefronts, 128 weight rows), two per compute unit, so one
//     streams while the other starts or finishes a tile; groups of more rows take eight
//     wavefronts and 256 weight rows, so that the activation rows, which come from L2
//     for every tile, stay the smaller part of the traffic;
//   - tiles start their k loops at different steps, so that the tiles in flight do not
//     all ask the same HBM channels (row pitches are multiples of the channel stride).
//     Eight neighbouring n-tiles of an expert start together: an XCD's L2 then serves
//     them one activation panel (and the m-tiles of one n-tile its weight panel).  Mixtral
//     shape, down projection at 127 rows: 258 us with a start of each tile's own, 207 with
//     these; 256 tokens over 64 experts of H 4096, F 4096, both GEMMs: 1018 and 959;
//   - weights that one m-tile reads bypass the caches (nt): nothing reads them again soon,
//     and without the allocation HBM delivers 6.4 to 6.9 TB/s instead of 5.8 to 6.1.  DeepSeek shape at
//     12 rows, both GEMMs: 933 -> 842 us; Mixtral shape at 6 rows: 471 -> 428.  Not for
//     small weights (a GEMM's under 128 MB, which the Infinity Cache may hold from one
//     call to the next: a shared expert's 58 MB at 8 rows 22 us, 28 bypassed), and not for
//     groups of several m-tiles (600 rows: 77 us, 100);
//   - no tile prefix, counters or persistent loop: a workgroup finds its tile from the
//     device-side offsets, the grid holds the host's bound on the tiles.
// The operands, their LDS layout and the MFMA instructions are those of the large-batch
// kernels (ffn.hip, ffn_fp8.hip), with the weight tile as the MFMA A operand.
#include <algorithm>
#include <type_traits>

#include "group_locate.h"
#include "lds_stage.h"
#include "moe_internal.h"
#include "mxfp8.h"

namespace moe {
namespace {

constexpr int kRowBytes = 128;            // one tile row of a stage: 64 bf16 or 128 codes of k

struct StreamArgs {
  const uint8_t* act;             // activation rows of K elements: [R] grouped, or with a gather [T]
  const uint8_t* act_scales;      // MXFP8: [K / 128][act_rows][4]
  const int32_t* gather;          // [R] row of act of each grouped row, or null
  const uint8_t* w0;              // [E, N, K] (GEMM-1: W_gate; GEMM-2: W_down)
  const uint8_t* w0_scales;       // MXFP8: [K / 128][E * N][4]
  const uint8_t* w1;              // GEMM-1: W_up
  const uint8_t* w1_scales;
  uint16_t* out;                  // bf16 [R, N]: h or y
  uint8_t* h_codes;               // MXFP8 GEMM-1: h [R, N]
  uint8_t* h_scales;              // [N / 128][R][4]
  const int32_t* offsets;         // [E + 1]
  int64_t act_rows;               // rows of act
  int E, K, N, ntiles, R;
};

// 16-byte chunk c of row r sits at chunk c ^ ((r >> 1) & 7): conflict-free operand reads.
__device__ __forceinline__ int swz(int row, int chunk) { return chunk ^ ((row >> 1) & 7); }

// LDS of a workgroup (the kernel's stages), and the wavefronts per SIMD that it leaves room for:
// what the register allocation is bounded by.
constexpr int stream_stage(bool fp8, int wn, int mr) {
  return (64 * wn + mr) * kRowBytes + (fp8 ? (64 * wn + (mr + 63) / 64 * 64) * 4 : 0);
}
constexpr int stream_waves(bool fp8, int wn, int mr, int kg, int s) {
  const int fit = 160 * 1024 / (s * kg * stream_stage(fp8, wn, mr) + (s == 3 ? 16 : 0));
  const int waves = fit * 2 * wn * kg / 4;
  return waves < 2 ? waves : 2;
}

// 2 x WN wavefronts: each MR / 2 activation rows x 64 weight rows of the tile (GEMM-1: 32
// gate and 32 up rows of the same features).  MR: activation rows per tile; S: stages.
template <bool FP8, bool SWIGLU, int WN, int MR, int KG, int S, bool NTW>
__global__ __launch_bounds__(128 * WN * KG, stream_waves(FP8, WN, MR, KG, S)) void stream_gemm_kernel(StreamArgs p) {
  constexpr int kElt = FP8 ? 1 : 2;
  constexpr int kBN = 64 * WN;                       // weight rows of the tile
  constexpr int kCols = SWIGLU ? kBN / 2 : kBN;      // output columns of the tile
  constexpr int kWaves = 2 * WN;                     // wavefronts of a k group
  constexpr int kABlocks = MR / 8;
  constexpr int kAPass = (kABlocks + kWaves - 1) / kWaves;   // activation loads per wavefront and stage
  constexpr int kLoads = 4 + kAPass + (FP8 ? 1 : 0);
  constexpr int kAOff = kBN * kRowBytes;
  constexpr int kWSOff = kAOff + MR * kRowBytes;     // MXFP8 scale dwords: weight rows, then activation rows
  constexpr int kASOff = kWSOff + kBN * 4;
  constexpr int kARows64 = (MR + 63) / 64 * 64;
  constexpr int kStage = stream_stage(FP8, WN, MR);
  static_assert(kStage == (FP8 ? kASOff + kARows64 * 4 : kWSOff), "stage layout");
  constexpr int kBlocks = MR / 32;                   // 32-row blocks of the tile: block 2 mi + wm is
  constexpr int NB = (kBlocks + 1) / 2;              // the mi-th of wavefront row wm
  static_assert(S == 3 || S == 4, "stages");
  static_assert(!FP8 || (kBN + kARows64) / 64 <= kWaves, "a scale load for every 64 tile rows");
  static_assert(kAPass >= 1 && kAPass <= 5, "activation loads per wavefront");
  // distinct objects, so that the compiler tells the stages' loads and reads apart
  __shared__ __attribute__((aligned(1024))) uint8_t st0[KG * kStage];
  __shared__ __attribute__((aligned(1024))) uint8_t st1[KG * kStage];
  __shared__ __attribute__((aligned(1024))) uint8_t st2[KG * kStage];
  __shared__ __attribute__((aligned(1024))) uint8_t st3[S == 4 ? KG * kStage : 16];

  const int tid = threadIdx.x;
  const int lane = tid & (kWave - 1);
  const int kg = KG > 1 ? __builtin_amdgcn_readfirstlane(tid / (kWave * kWaves)) : 0;
  const int wave = __builtin_amdgcn_readfirstlane(tid / kWave) - kg * kWaves;      // in its k group
  const int gbase = kg * kStage;                     // the k group's part of every stage
  const int wm = wave / WN, wn = wave % WN;
  if (p.E < 0) {                  // never taken: keeps the DMA-filled stages' reads
    st0[tid] = 0;
    st1[tid] = 0;
    st2[tid] = 0;
    if (S == 4) st3[tid & 15] = 0;
  }
  MTile tile;
  if (!locate_tile<MR>(p.offsets, p.E, p.ntiles, tile_workgroup(), &tile)) return;     // uniform across the block
  const int e = tile.e, nt = tile.nt, row0 = tile.row0, row_stop = tile.row_stop;
  const int K = p.K, N = p.N;
  const int n0 = nt * kCols;
  const int64_t rowb = int64_t(K) * kElt;
  const int KT = int(rowb / kRowBytes);
  const int64_t EN = int64_t(p.E) * N;

  // ---- loads.  Pass i of wavefront w fills the 1 KB block kWaves i + w of an operand (8
  // rows); lane q lands at row 8 blk + q / 8, chunk position q % 8.
  const int wrows = min(kCols, N - n0);              // rows past N read as zeros
  const int64_t wfirst = (int64_t(e) * N + n0) * rowb;
  const __amdgpu_buffer_rsrc_t rw0 = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t*>(p.w0) + wfirst, 0,
                                                                      int(wrows * rowb), 0x00020000);
  const __amdgpu_buffer_rsrc_t rw1 = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<uint8_t*>(SWIGLU ? p.w1 : p.w0) + wfirst, 0, int(wrows * rowb), 0x00020000);
  const int qrow = lane >> 3, qpos = lane & 7;
  uint32_t woff[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int r = (kWaves * i + wave) * 8 + qrow;
    // GEMM-1: the first half of the tile rows are gate features n0.., the second the up rows
    woff[i] = uint32_t(SWIGLU ? r % kCols : r) * uint32_t(rowb) + uint32_t(swz(r, qpos) * 16);
  }
  // (a wavefront past the last block of a pass loads its first block again, so that all
  // wavefronts have the same loads in flight)
  const uint8_t* aptr[5];       // (sized by the template-dependent count, the host pass drops the launch stub)
  int adst[5];
#pragma unroll
  for (int i = 0; i < kAPass; ++i) {
    const int blk = kWaves * i + wave < kABlocks ? kWaves * i + wave : wave;
    const int r = blk * 8 + qrow;
    adst[i] = opaque_s(gbase + kAOff + blk * 1024);
    // a row past the tile reads its first one: its results are not stored
    const int grow = row0 + r < row_stop ? row0 + r : row0;
    const int64_t src = p.gather != nullptr ? int64_t(p.gather[grow]) : int64_t(grow);
    aptr[i] = p.act + src * rowb + swz(r, qpos) * 16;
  }
  // MXFP8: one scale load per wavefront and stage, a dword per lane for 64 tile rows: the
  // first kBN / 64 wavefronts the weight rows', the others the activation rows'
  const uint8_t* sptr = nullptr;
  int64_t sstep = 0;
  int soff = 0;
  if constexpr (FP8) {
    if (wave < kBN / 64) {
      const int r = wave * 64 + lane;
      const uint8_t* s = SWIGLU && r >= kCols ? p.w1_scales : p.w0_scales;
      // rows past N take another row's (finite) scale; their codes are zeros
      const int64_t row = min(int64_t(e) * N + n0 + (SWIGLU ? r % kCols : r), EN - 1);
      sptr = s + row * 4;
      sstep = EN * 4;
      soff = kWSOff + wave * 256;
    } else {
      const int c = min(wave - kBN / 64, kARows64 / 64 - 1);
      const int r = c * 64 + lane;
      const int grow = row0 + r < row_stop ? row0 + r : row0;
      const int64_t src = p.gather != nullptr ? int64_t(p.gather[grow]) : int64_t(grow);
      sptr = p.act_scales + src * 4;
      sstep = p.act_rows * 4;
      soff = kASOff + c * 256;
    }
  }
  const int krot = int((int64_t(e) * ((p.ntiles + 7) / 8) + nt / 8) * 7 % KT);
  const int wdst = opaque_s(gbase + wave * 1024);
  soff = opaque_s(gbase + soff);
  auto issue = [&](uint8_t* stage, int it) {         // k step it * KG + kg, or the last one past the end
    const int kt = min(it * KG + kg, KT - 1);
    const int kp = kt + krot >= KT ? kt + krot - KT : kt + krot;
    const int kb = kp * kRowBytes;
#pragma unroll
    for (int i = 0; i < 4; ++i)
      __builtin_amdgcn_raw_ptr_buffer_load_lds((SWIGLU && i >= 2) ? rw1 : rw0, stage + (wdst + kWaves * i * 1024),
                                               16, woff[i], kb, 0, NTW ? 2 : 0);
#pragma unroll
    for (int i = 0; i < kAPass; ++i)
      __builtin_amdgcn_global_load_lds(aptr[i] + kb, stage + adst[i], 16, 0, 0);
    if constexpr (FP8) __builtin_amdgcn_global_load_lds(sptr + kp * sstep, stage + soff, 4, 0, 0);
  };

  const int rrow = lane & 31, khalf = lane >> 5;
  const int wbase = SWIGLU ? wn * 32 : wn * 64;      // first weight rows of the wavefront's two blocks
  constexpr int kWStep = SWIGLU ? kCols : 32;
  f32x16 acc[NB][2];
#pragma unroll
  for (int mi = 0; mi < NB; ++mi)
#pragma unroll
    for (int ni = 0; ni < 2; ++ni)
#pragma unroll
      for (int q = 0; q < 16; ++q) acc[mi][ni][q] = 0.f;
  // a lane's operand chunk 2 j + khalf of its row in the first weight and activation block
  // (rows 32 n further have the same swizzle)
  int wlane[4], alane[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int wr = wbase + rrow, ar = wm * 32 + rrow;
    wlane[j] = opaque_v(gbase + wr * kRowBytes + swz(wr, 2 * j + khalf) * 16);
    alane[j] = opaque_v(gbase + kAOff + ar * kRowBytes + swz(ar, 2 * j + khalf) * 16);
  }
  const int wslane = opaque_v(gbase + kWSOff + (wbase + rrow) * 4);
  const int aslane = opaque_v(gbase + kASOff + (wm * 32 + rrow) * 4);
  auto wchunk = [&](const uint8_t* stage, int ni, int j) {
    return *reinterpret_cast<const u32x4*>(stage + (wlane[j] + ni * kWStep * kRowBytes));
  };
  auto achunk = [&](const uint8_t* stage, int mi, int j) {
    return *reinterpret_cast<const u32x4*>(stage + (alane[j] + mi * 64 * kRowBytes));
  };
  auto compute = [&](const uint8_t* stage, auto nb_c) {
    constexpr int NBW = decltype(nb_c)::value;       // blocks of this wavefront that hold rows
    if constexpr (FP8) {
      // scale dwords shifted so that byte 2 s is the block 2 s + khalf of the step
      uint32_t wsc[2], xsc[NBW];
#pragma unroll
      for (int ni = 0; ni < 2; ++ni)
        wsc[ni] = *reinterpret_cast<const uint32_t*>(stage + (wslane + ni * kWStep * 4)) >> (8 * khalf);
#pragma unroll
      for (int mi = 0; mi < NBW; ++mi)
        xsc[mi] = *reinterpret_cast<const uint32_t*>(stage + (aslane + mi * 64 * 4)) >> (8 * khalf);
      auto both = [&](u32x4 lo, u32x4 hi) {
        i32x8 v;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          v[q] = int(lo[q]);
          v[4 + q] = int(hi[q]);
        }
        return v;
      };
#pragma unroll
      for (int s = 0; s < 2; ++s) {
        i32x8 wf[2], xf[NBW];
#pragma unroll
        for (int ni = 0; ni < 2; ++ni) wf[ni] = both(wchunk(stage, ni, 2 * s), wchunk(stage, ni, 2 * s + 1));
#pragma unroll
        for (int mi = 0; mi < NBW; ++mi)
          xf[mi] = both(achunk(stage, mi, 2 * s), achunk(stage, mi, 2 * s + 1));
#pragma unroll
        for (int mi = 0; mi < NBW; ++mi)
#pragma unroll
          for (int ni = 0; ni < 2; ++ni)
            // op_sel must be a literal: byte 2 s of the shifted scale dwords
            acc[mi][ni] = s == 0 ? __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(
                                       wf[ni], xf[mi], acc[mi][ni], 0, 0, 0, int(wsc[ni]), 0, int(xsc[mi]))
                                 : __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(
                                       wf[ni], xf[mi], acc[mi][ni], 0, 0, 2, int(wsc[ni]), 2, int(xsc[mi]));
      }
    } else {
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        bf16x8 wf[2], xf[NBW];
#pragma unroll
        for (int ni = 0; ni < 2; ++ni)
          wf[ni] = __builtin_bit_cast(bf16x8, wchunk(stage, ni, s));
#pragma unroll
        for (int mi = 0; mi < NBW; ++mi)
          xf[mi] = __builtin_bit_cast(bf16x8, achunk(stage, mi, s));
#pragma unroll
        for (int mi = 0; mi < NBW; ++mi)
#pragma unroll
          for (int ni = 0; ni < 2; ++ni)
            acc[mi][ni] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf[ni], xf[mi], acc[mi][ni], 0, 0, 0);
      }
    }
  };

  // ---- k loop.  Step it waits for its stage (its own lanes' loads, then every wavefront's
  // through the barrier, which also frees the stage read in the step before), sends the
  // loads of step it + S - 1 into that stage, and multiplies.  The last S - 1 steps send
  // the last step's loads again (L2 hits), so that every wait is for the same count.
  // One loop per count of row blocks that the wavefront computes (0: it still loads and
  // synchronizes), so that a step is a fixed sequence.
  const int steps = (KT + KG - 1) / KG;              // the same for every k group
  const int nbw = max(0, (row_stop - row0 - wm * 32 + 63) / 64);   // uniform across the wave, at most NB
  auto kloop = [&](auto nb_c) {
    constexpr int NBW = decltype(nb_c)::value;
    auto step = [&](const uint8_t* cur, uint8_t* nxt, int it) {
      __builtin_amdgcn_sched_barrier(0);
      __builtin_amdgcn_s_waitcnt(wait_vm((S - 2) * kLoads));
      bare_barrier();
      __builtin_amdgcn_sched_barrier(0);
      issue(nxt, it + S - 1);
      __builtin_amdgcn_sched_barrier(0);
      if constexpr (NBW > 0) {
        if (KG == 1 || it * KG + kg < KT) compute(cur, nb_c);
      }
    };
    int it = 0;
    for (; it + S <= steps; it += S) {
      step(st0, S == 4 ? st3 : st2, it);
      step(st1, st0, it + 1);
      step(st2, st1, it + 2);
      if constexpr (S == 4) step(st3, st2, it + 3);
    }
    if (it < steps) step(st0, S == 4 ? st3 : st2, it);
    if (it + 1 < steps) step(st1, st0, it + 1);
    if (S == 4 && it + 2 < steps) step(st2, st1, it + 2);
  };
  issue(st0, 0);
  __builtin_amdgcn_sched_barrier(0);                 // the waits count on this order
  issue(st1, 1);
  __builtin_amdgcn_sched_barrier(0);
  if constexpr (S == 4) issue(st2, 2);
  if (nbw == 0) kloop(std::integral_constant<int, 0>{});
  else if (NB >= 3 && nbw == 3) kloop(std::integral_constant<int, (NB >= 3 ? 3 : 1)>{});
  else if (NB >= 2 && nbw == 2) kloop(std::integral_constant<int, (NB >= 2 ? 2 : 1)>{});
  else kloop(std::integral_constant<int, 1>{});
  // no load may still be on its way into this workgroup's LDS when it is used again or ends
  __builtin_amdgcn_s_waitcnt(wait_vm(0));
  if constexpr (KG > 1) {
    // the k groups' sums meet in LDS and are added in group order
    static_assert(NB == 1 && (KG - 1) * kWaves * 8192 <= KG * kStage, "sums fit a stage");
    __syncthreads();
    f32x4* mine = reinterpret_cast<f32x4*>(st0) + (kg * kWaves + wave) * 512 + lane;
    if (kg > 0) {
#pragma unroll
      for (int ni = 0; ni < 2; ++ni)
#pragma unroll
        for (int b = 0; b < 4; ++b)
          mine[(ni * 4 + b) * 64 - kWaves * 512] = f32x4{acc[0][ni][4 * b], acc[0][ni][4 * b + 1],
                                                        acc[0][ni][4 * b + 2], acc[0][ni][4 * b + 3]};
    }
    __syncthreads();
    if (kg > 0) return;
#pragma unroll
    for (int g = 0; g < KG - 1; ++g)
#pragma unroll
      for (int ni = 0; ni < 2; ++ni)
#pragma unroll
        for (int b = 0; b < 4; ++b) {
          const f32x4 v = mine[(ni * 4 + b) * 64 + g * kWaves * 512];
#pragma unroll
          for (int q = 0; q < 4; ++q) acc[0][ni][4 * b + q] += v[q];
        }
  }
  if (nbw == 0) return;

  // ---- epilogue: lane holds weight rows 8 blk + 4 khalf + {0..3} of each 32-row block for
  // activation row rrow.  The results are few next to the weights: stored from registers.
#pragma unroll
  for (int mi = 0; mi < NB; ++mi) {
    const int row = row0 + (2 * mi + wm) * 32 + rrow;
    if constexpr (SWIGLU) {
      float hv[16];
#pragma unroll
      for (int q = 0; q < 16; ++q) hv[q] = silu(acc[mi][0][q]) * acc[mi][1][q];
      const int f0 = n0 + wn * 32;                   // N % 64 = 0: 32 whole features
      if (f0 >= N) continue;                         // uniform across the wave
      if constexpr (FP8) {
        // the 32 features of a row are one MX block, held by lanes l and l ^ 32
        float amax = 0.f;
#pragma unroll
        for (int q = 0; q < 16; ++q) amax = fmaxf(amax, fabsf(hv[q]));
        amax = fmaxf(amax, __shfl_xor(amax, 32));
        const int se = mx_shared_exp(amax);
        const float inv = mx_inv_scale(se);
        if (row < row_stop) {
#pragma unroll
          for (int blk = 0; blk < 4; ++blk) {
            const float* hb = hv + blk * 4;
            *reinterpret_cast<uint32_t*>(p.h_codes + int64_t(row) * N + f0 + blk * 8 + khalf * 4) =
                e4m3_pack4(hb[0] * inv, hb[1] * inv, hb[2] * inv, hb[3] * inv);
          }
          const int b = f0 / 32;
          if (khalf == 0) p.h_scales[(int64_t(b / 4) * p.R + row) * 4 + (b & 3)] = uint8_t(se + 127);
        }
      } else if (row < row_stop) {
#pragma unroll
        for (int blk = 0; blk < 4; ++blk) {
          u32x2 pk;
          pk[0] = pack_bf16x2(hv[blk * 4], hv[blk * 4 + 1]);
          pk[1] = pack_bf16x2(hv[blk * 4 + 2], hv[blk * 4 + 3]);
          *reinterpret_cast<u32x2*>(p.out + int64_t(row) * N + f0 + blk * 8 + khalf * 4) = pk;
        }
      }
    } else if (row < row_stop) {
#pragma unroll
      for (int ni = 0; ni < 2; ++ni) {
        const int n = n0 + wn * 64 + ni * 32;
        if (n >= N) continue;
#pragma unroll
        for (int blk = 0; blk < 4; ++blk) {
          u32x2 pk;
          pk[0] = pack_bf16x2(acc[mi][ni][blk * 4], acc[mi][ni][blk * 4 + 1]);
          pk[1] = pack_bf16x2(acc[mi][ni][blk * 4 + 2], acc[mi][ni][blk * 4 + 3]);
          *reinterpret_cast<u32x2*>(p.out + int64_t(row) * N + n + blk * 8 + khalf * 4) = pk;
        }
      }
    }
  }
}

template <bool FP8, bool SWIGLU, int WN, int MR, int KG, int S>
void launch_tiles(const char* name, StreamArgs a, hipStream_t s) {
  const int cols = 64 * WN / (SWIGLU ? 2 : 1);
  a.ntiles = (a.N + cols - 1) / cols;
  const int64_t mtiles = (int64_t(a.R) + int64_t(std::min(a.E, a.R)) * (MR - 1)) / MR;
  const dim3 grid = tile_dim(mtiles * a.ntiles), block(128 * WN * KG);
  if (stream_nt(a.R, a.E, a.K, a.N, SWIGLU, FP8, MR))
    MOE_LAUNCH(name, (stream_gemm_kernel<FP8, SWIGLU, WN, MR, KG, S, true>), grid, block, s, a);
  else
    MOE_LAUNCH(name, (stream_gemm_kernel<FP8, SWIGLU, WN, MR, KG, S, false>), grid, block, s, a);
}

template <bool FP8, bool SWIGLU>
void launch_gemm(const char* name, const StreamArgs& a, int num_cu, hipStream_t s) {
  const StreamTile t = stream_tile(a.R, a.E, a.N, SWIGLU, FP8, num_cu);
  if constexpr (!FP8) {
    if (t.mr == 160 && t.wn == 4) return launch_tiles<FP8, SWIGLU, 4, 160, 1, 3>(name, a, s);
    if (t.mr == 160) return launch_tiles<FP8, SWIGLU, 2, 160, 1, 4>(name, a, s);
  }
  if (t.mr == 128 && t.wn == 4) return launch_tiles<FP8, SWIGLU, 4, 128, 1, 3>(name, a, s);
  if (t.mr == 128) return launch_tiles<FP8, SWIGLU, 2, 128, 1, 4>(name, a, s);
  if (t.mr == 64 && t.wn == 1) return launch_tiles<FP8, SWIGLU, 1, 64, 2, 4>(name, a, s);
  if (t.mr == 64 && t.kg == 2) return launch_tiles<FP8, SWIGLU, 2, 64, 2, 3>(name, a, s);
  if (t.mr == 64) return launch_tiles<FP8, SWIGLU, 2, 64, 1, 3>(name, a, s);
  if (t.wn == 1) return launch_tiles<FP8, SWIGLU, 1, 32, 4, 3>(name, a, s);
  if (t.kg == 2) return launch_tiles<FP8, SWIGLU, 2, 32, 2, 3>(name, a, s);
  launch_tiles<FP8, SWIGLU, 2, 32, 1, 3>(name, a, s);
}

}  // namespace

bool use_stream_gemm(int64_t R, int E, int K, int N, bool swiglu, bool fp8, int num_cu) {
  if (cu_budget_set()) return false;      // the caller leaves compute units to other streams
  return stream_is_faster(R, E, K, N, swiglu, fp8, num_cu);
}

hipError_t launch_stream_gemm_bf16(const uint16_t* act, const int32_t* gather, int64_t act_rows, const int32_t* offsets,
                                   int64_t R, int E, int K, int N, const uint16_t* w0, const uint16_t* w1,
                                   uint16_t* out, int num_cu, hipStream_t s) {
  auto u8 = [](const uint16_t* q) { return reinterpret_cast<const uint8_t*>(q); };
  const StreamArgs a{u8(act), nullptr, gather, u8(w0), nullptr, u8(w1), nullptr, out, nullptr, nullptr, offsets,
                     act_rows, E, K, N, 0, int(R)};
  if (w1 != nullptr) launch_gemm<false, true>("ffn_gemm1_gate_up", a, num_cu, s);
  else launch_gemm<false, false>("ffn_gemm2_down", a, num_cu, s);
  return hipGetLastError();
}

hipError_t launch_stream_gemm1_mxfp8(const uint8_t* x, const uint8_t* xs, const int32_t* gather, int64_t act_rows,
                                     const int32_t* offsets, int64_t R, int E, int K, int N, const uint8_t* wg,
                                     const uint8_t* wgs, const uint8_t* wu, const uint8_t* wus, uint8_t* h,
                                     uint8_t* hs, int num_cu, hipStream_t s) {
  launch_gemm<true, true>("ffn_gemm1_gate_up",
                          StreamArgs{x, xs, gather, wg, wgs, wu, wus, nullptr, h, hs, offsets, act_rows, E, K, N, 0,
                                     int(R)}, num_cu, s);
  return hipGetLastError();
}

hipError_t launch_stream_gemm2_mxfp8(const uint8_t* h, const uint8_t* hs, const int32_t* offsets, int64_t R, int E,
                                     int K, int N, const uint8_t* wd, const uint8_t* wds, uint16_t* y, int num_cu,
                                     hipStream_t s) {
  launch_gemm<true, false>("ffn_gemm2_down",
                           StreamArgs{h, hs, nullptr, wd, wds, nullptr, nullptr, y, nullptr, nullptr, offsets, R, E, K,
                                      N, 0, int(R)}, num_cu, s);
  return hipGetLastError();
}

}  // namespace moe
