// moe_router_topk: the MoE gate's router GEMM fused with top-k selection on gfx950.
//
// logits[t, e] = x[t] . w_router[e] (bf16 operands, fp32 accumulation on the
// matrix cores), then the gate of moe_route on those fp32 logits: the k largest,
// ties to the lower expert id, softmax over the selected (or all) logits.  The
// logits never leave the chip unless the caller asks for them.
//
// Two kernels, one k order (so a token's result does not depend on its batch): small
// batches with H % 128 = 0 split each 16-token block's k over four wavefronts
// (router_splitk_kernel); otherwise blocks of two or four wavefronts, 16 tokens each,
// share the router matrix (router_lds_kernel).  Both stream both operands through LDS and use
// v_mfma_f32_16x16x32_bf16 on up to four 16-expert blocks (E <= 64).  The fp32
// logits go through LDS to the selection, where 4 lanes hold one token's logits
// and each round takes a quad maximum of orderable keys, then a quad minimum of
// the expert ids holding it (DPP lane permutes).
#include "common.h"
#include "lds_stage.h"
#include "moe_internal.h"

namespace moe {
namespace {

constexpr int kTok = 16;                  // tokens per MFMA block

template <int CTRL>
__device__ __forceinline__ uint32_t dpp(uint32_t v) {
  return uint32_t(__builtin_amdgcn_update_dpp(0, int(v), CTRL, 0xF, 0xF, false));
}

__device__ __forceinline__ uint32_t quad_max(uint32_t v) {
  v = max(v, dpp<0xB1>(v));              // quad_perm [1, 0, 3, 2]
  return max(v, dpp<0x4E>(v));           // quad_perm [2, 3, 0, 1]
}
__device__ __forceinline__ uint32_t quad_min(uint32_t v) {
  v = min(v, dpp<0xB1>(v));
  return min(v, dpp<0x4E>(v));
}
__device__ __forceinline__ float quad_sum(float v) {
  v += __uint_as_float(dpp<0xB1>(__float_as_uint(v)));
  return v + __uint_as_float(dpp<0x4E>(__float_as_uint(v)));
}

// The gate of moe_route on one token's E logits, held by four lanes (g = lane % 4) as experts
// g V .. g V + V - 1 (key: orderable, 0 past E): the k largest, ties to the lower expert id,
// softmax over the selected (renormalize) or all logits.  Lane g = 0 of a valid token writes.
template <int V, int KMAX>
__device__ __forceinline__ void select_topk(const float (&vals)[V], uint32_t (&key)[V], int e0, int g, int E, int k,
                                            int renormalize, bool valid, int64_t t, int32_t* __restrict__ topk_ids,
                                            float* __restrict__ topk_w) {
  uint32_t selk[KMAX];
  uint32_t sele[KMAX];
#pragma unroll
  for (int j = 0; j < KMAX; ++j) {
    if (j < k) {
      uint32_t m = key[0];
#pragma unroll
      for (int v = 1; v < V; ++v) m = max(m, key[v]);
      m = quad_max(m);
      uint32_t id = 0xFFFFFFFFu;
#pragma unroll
      for (int v = V - 1; v >= 0; --v) id = key[v] == m ? uint32_t(e0 + v) : id;
      id = quad_min(id);
#pragma unroll
      for (int v = 0; v < V; ++v) key[v] = uint32_t(e0 + v) == id ? 0u : key[v];
      selk[j] = m;
      sele[j] = id;
    } else {
      selk[j] = 0u;
      sele[j] = 0u;
    }
  }
  const float lmax = from_orderable(selk[0]);
  float p[KMAX];
  float denom = 0.f;
#pragma unroll
  for (int j = 0; j < KMAX; ++j) {
    if (j < k) {
      p[j] = expf(from_orderable(selk[j]) - lmax);
      denom += p[j];
    }
  }
  if (!renormalize) {
    float sum = 0.f;
#pragma unroll
    for (int v = 0; v < V; ++v)
      if (e0 + v < E) sum += expf(vals[v] - lmax);
    denom = quad_sum(sum);
  }
  if (valid && g == 0) {
#pragma unroll
    for (int j = 0; j < KMAX; ++j) {
      if (j < k) {
        topk_ids[t * k + j] = int32_t(sele[j]);
        topk_w[t * k + j] = p[j] / denom;
      }
    }
  }
}

// Larger batches: WV (two or four) wavefronts per block, 16 tokens each.  Memory bounds it: x is
// read once, the router matrix once per block, from L2.  Token rows and router rows go
// through a ring of four LDS stages of 64 k each, by direct global -> LDS loads of whole
// 128-byte row pieces sent three steps ahead; a step waits for its own stage only.  (Loaded
// straight into the MFMA layout, adjacent lanes in different rows, the same bytes cost the
// address unit four times the cycles.)  16 KB per stage at 64 experts and four wavefronts, so
// two blocks share a compute unit; stages of 128 k, one block each, are no faster at one
// block per compute unit and slower past it.  Against token rows loaded into registers one
// slice ahead (in us): 16384 tokens x H 7168, 64 experts 63 -> 46 (5.1 TB/s); 65536 x 7168, 64:
// 216 -> 169 (5.6 TB/s); 131072 x 4096, 8: 203 -> 183 (5.9 TB/s); H % 128 != 0, against one
// wavefront per 16 to 64 tokens reading both operands from memory: 16384 x 7104, 64:
// 132 -> 45; 131072 x 1088, 8: 74 -> 43.
constexpr int kRingStages = 4;
constexpr int kRingK = 64;

template <int NB, int KMAX, int WV>
__global__ __launch_bounds__(WV * 64) void router_lds_kernel(const uint16_t* __restrict__ x,
                                                                   const uint16_t* __restrict__ w, int64_t T,
                                                                   int E, int k, int H, int renormalize,
                                                                   float* __restrict__ logits_out,
                                                                   int32_t* __restrict__ topk_ids,
                                                                   float* __restrict__ topk_w) {
  constexpr int EP = 16 * NB;
  constexpr int V = EP / 4;
  constexpr int kRow = kRingK * 2;                    // bytes of one row in a stage
  constexpr int kRowChunks = kRow / 16;
  constexpr int kDmaRows = 1024 / kRow;               // rows per 1 KB load
  constexpr int kXDma = kTok / kDmaRows;              // per wavefront: its own 16 rows
  constexpr int kWDma = EP / kDmaRows;
  constexpr int kWDmaPerWave = (kWDma + WV - 1) / WV;
  constexpr int kLoads = kXDma + kWDmaPerWave;
  constexpr int kXBytes = WV * kTok * kRow;
  constexpr int kStage = kXBytes + EP * kRow;
  static_assert(kWDmaPerWave <= 4 && kXDma == 2 && kRowChunks == 8, "fixed-size arrays, swz");
  static_assert(WV * kTok * EP * 4 <= kStage, "the logits fit a stage");
  __shared__ __attribute__((aligned(1024))) uint8_t st0[kStage];
  __shared__ __attribute__((aligned(1024))) uint8_t st1[kStage];
  __shared__ __attribute__((aligned(1024))) uint8_t st2[kStage];
  __shared__ __attribute__((aligned(1024))) uint8_t st3[kStage];

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  if (T < 0) {                                        // never taken: keeps the DMA-filled stages' reads
    st0[tid] = 0;
    st1[tid] = 0;
    st2[tid] = 0;
    st3[tid] = 0;
  }
  const int64_t t0 = (int64_t(blockIdx.x) * WV + wave) * kTok;
  const int r16 = lane & 15;
  const int kq = lane >> 4;

  // 16-byte chunk c of row r sits at swz(r, c): the 16 rows of an operand read touch
  // distinct banks.  Rows past T read the last one (never stored); experts past E are out of
  // range of the buffer and read as zero.
  auto swz = [](int r, int c) { return c ^ ((r >> 1) & 7); };
  const __amdgpu_buffer_rsrc_t rw =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(w), 0, int(int64_t(E) * H * 2), 0x00020000);
  const int drow = lane / kRowChunks, dpos = lane % kRowChunks;
  // (fixed sizes: with a template-dependent one the host pass drops the launch stub)
  const uint16_t* xrow[2];
  uint32_t woff[4];
  int wdst[4];
#pragma unroll
  for (int j = 0; j < kXDma; ++j) {
    const int row = kDmaRows * j + drow;
    xrow[j] = x + (t0 + row < T ? t0 + row : T - 1) * H + swz(row, dpos) * 8;
  }
#pragma unroll
  for (int j = 0; j < kWDmaPerWave; ++j) {
    const int i = (j * WV + wave) % kWDma;     // (few experts: some load the same rows again)
    const int row = kDmaRows * i + drow;
    woff[j] = row < E ? uint32_t(row) * uint32_t(H) * 2u + uint32_t(swz(row, dpos)) * 16u : 0x80000000u;
    wdst[j] = opaque_s(kXBytes + i * 1024);
  }
  const int xdst = opaque_s(wave * kTok * kRow);
  const int steps = H / kRingK;
  // past the end every lane reads x's first 16 bytes, and the router matrix out of range: the
  // waits count on the loads, and nothing more is read
  auto issue = [&](uint8_t* stage, int s) {
    const uint32_t past = s < steps ? 0u : 0x80000000u;
    const int kb = s < steps ? s * kRow : 0;
#pragma unroll
    for (int j = 0; j < kXDma; ++j)
      __builtin_amdgcn_global_load_lds(s < steps ? xrow[j] + s * kRingK : x, stage + (xdst + j * 1024), 16, 0, 2);
#pragma unroll
    for (int j = 0; j < kWDmaPerWave; ++j)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rw, stage + wdst[j], 16, woff[j] | past, kb, 0, 0);
  };

  int at[2], xat[2];                                  // the router row's and the token row's chunk of 32 k
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    at[u] = opaque_v(kXBytes + r16 * kRow + swz(r16, 4 * u + kq) * 16);
    xat[u] = opaque_v(wave * kTok * kRow + r16 * kRow + swz(r16, 4 * u + kq) * 16);
  }
  f32x4 acc[NB], tot[NB];
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) acc[nb] = f32x4{0.f, 0.f, 0.f, 0.f};
  // k order of the sum (the same in both kernels, so a token's logits do not depend on the
  // batch it arrives in): with H % 128 = 0, four quarter sums over consecutive 32-k chunks,
  // added as ((q0 + q1) + q2) + q3; otherwise one chain.
  const bool quarters = H % 128 == 0;
  const int qc = quarters ? H / 128 : H;              // 32-k chunks per quarter (one chain: never reached)
  int next = qc;
  auto step = [&](const uint8_t* cur, uint8_t* nxt, int s) {
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_waitcnt(wait_vm((kRingStages - 2) * kLoads));
    bare_barrier();                                   // ... for every wavefront; stage nxt is free
    __builtin_amdgcn_sched_barrier(0);
    issue(nxt, s + kRingStages - 1);
    __builtin_amdgcn_sched_barrier(0);
    bf16x8 a[2], b[2][NB];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      a[u] = *reinterpret_cast<const bf16x8*>(cur + xat[u]);
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) b[u][nb] = *reinterpret_cast<const bf16x8*>(cur + (at[u] + nb * 16 * kRow));
    }
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      if (2 * s + u == next) {
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) {
          tot[nb] = next == qc ? acc[nb] : tot[nb] + acc[nb];
          acc[nb] = f32x4{0.f, 0.f, 0.f, 0.f};
        }
        next += qc;
      }
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) acc[nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[u], b[u][nb], acc[nb], 0, 0, 0);
    }
  };
  issue(st0, 0);
  __builtin_amdgcn_sched_barrier(0);                  // the waits count on this order
  issue(st1, 1);
  __builtin_amdgcn_sched_barrier(0);
  issue(st2, 2);
  int s = 0;
  for (; s + kRingStages <= steps; s += kRingStages) {
    step(st0, st3, s);
    step(st1, st0, s + 1);
    step(st2, st1, s + 2);
    step(st3, st2, s + 3);
  }
  if (s < steps) step(st0, st3, s);
  if (s + 1 < steps) step(st1, st0, s + 1);
  if (s + 2 < steps) step(st2, st1, s + 2);
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) acc[nb] = quarters ? tot[nb] + acc[nb] : acc[nb];   // the last quarter
  __builtin_amdgcn_s_waitcnt(wait_vm(0));             // no load may still be on its way into this LDS
  __syncthreads();                                    // every wavefront is done with the stages

  // 16 x 16 outputs: lane holds tokens 4 (lane / 16) + q of expert column lane % 16
  float* const logits = reinterpret_cast<float*>(st0) + wave * kTok * EP;
  auto at_log = [](int row, int col) { return row * EP + (col ^ ((row & 3) << 2)); };
#pragma unroll
  for (int nb = 0; nb < NB; ++nb)
#pragma unroll
    for (int q = 0; q < 4; ++q) logits[at_log(4 * kq + q, nb * 16 + r16)] = acc[nb][q];
  __syncthreads();

  // selection: 16 tokens per wavefront, token tt = lane / 4, lane g = lane % 4 holds
  // experts g V .. g V + V - 1
  const int tt = lane >> 2;
  const int g = lane & 3;
  const int64_t t = t0 + tt;
  const bool valid = t < T;
  const int e0 = g * V;
  float vals[V];
  uint32_t key[V];
#pragma unroll
  for (int v = 0; v < V; ++v) {
    const bool live = e0 + v < E;
    vals[v] = live ? logits[at_log(tt, e0 + v)] : 0.f;
    key[v] = live ? orderable(vals[v]) : 0u;
  }
  if (logits_out != nullptr && valid) {
#pragma unroll
    for (int v = 0; v < V; ++v)
      if (e0 + v < E) logits_out[t * E + e0 + v] = vals[v];
  }
  select_topk<V, KMAX>(vals, key, e0, g, E, k, renormalize, valid, t, topk_ids, topk_w);
}

// Small batches: four wavefronts per 16 tokens, each a quarter of the k range, their fp32
// partial logits added in wavefront order through LDS; wavefront 0 then selects.  Each
// wavefront streams its part of both operands through a ring of three LDS stages of its own,
// 64 k each, without a barrier.  Against both operands loaded into the MFMA layout from
// memory (in us): 16 tokens x H 7168, 64 experts 35.8 -> 15.2; 4096 x 7168, 64: 43.3 -> 19.5;
// 6000 x 4096, 32: 28.8 -> 13.4; 12288 x 4096, 8: 25.4 -> 19.0.
// From cold caches, token rows with the nt policy: 8192 x 4096, 8: 21.0 -> 15.8 (30.2 without
// the policy); 4096 x 7168, 64: 45 -> 28 (36 without).
constexpr int kSplitWaves = 4;

template <int NB, int KMAX>
__global__ __launch_bounds__(kSplitWaves * 64) void router_splitk_kernel(const uint16_t* __restrict__ x,
                                                                        const uint16_t* __restrict__ w, int64_t T,
                                                                        int E, int k, int H, int renormalize,
                                                                        float* __restrict__ logits_out,
                                                                        int32_t* __restrict__ topk_ids,
                                                                        float* __restrict__ topk_w) {
  constexpr int EP = 16 * NB;
  constexpr int V = EP / 4;
  constexpr int kRow = kRingK * 2;
  constexpr int kRows = kTok + EP;                    // a wavefront's stage: 16 token rows, EP router rows
  constexpr int kLoads = kRows / 8;                   // of 1 KB, 8 rows each
  constexpr int kWaveStage = kRows * kRow;
  static_assert(kLoads - 2 <= 8 && kRow == 128, "fixed-size arrays, swizzle");
  __shared__ __attribute__((aligned(1024))) uint8_t st0[kSplitWaves * kWaveStage];
  __shared__ __attribute__((aligned(1024))) uint8_t st1[kSplitWaves * kWaveStage];
  __shared__ __attribute__((aligned(1024))) uint8_t st2[kSplitWaves * kWaveStage];

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(int(threadIdx.x) >> 6);
  if (T < 0) {                                        // never taken: keeps the DMA-filled stages' reads
    st0[threadIdx.x] = 0;
    st1[threadIdx.x] = 0;
    st2[threadIdx.x] = 0;
  }
  const int64_t t0 = int64_t(blockIdx.x) * kTok;
  const int r16 = lane & 15;
  const int kq = lane >> 4;
  const int Hq = H / kSplitWaves;                     // a multiple of 32
  const int chunks = Hq / 32;
  const int steps = (chunks + 1) / 2;
  // Swizzle, rows past T and experts past E as router_lds_kernel.  A quarter of an odd number
  // of chunks takes half of its last step: the token loads of the other half read x's first
  // 16 bytes, the router matrix's the 32 k behind (the next quarter's, the next row's or out
  // of range), and nothing multiplies them.
  const __amdgpu_buffer_rsrc_t rw =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(w), 0, int(int64_t(E) * H * 2), 0x00020000);
  const int drow = lane >> 3, dpos = lane & 7;
  auto swz = [](int r, int c) { return c ^ ((r >> 1) & 7); };
  const uint16_t* xrow[2];
  uint32_t woff[8];
  int xk[2];                                          // k of this lane's chunk within a step
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const int row = 8 * j + drow;
    xk[j] = swz(row, dpos) * 8;
    xrow[j] = x + (t0 + row < T ? t0 + row : T - 1) * H + wave * Hq + xk[j];
  }
#pragma unroll
  for (int j = 0; j < kLoads - 2; ++j) {
    const int row = 8 * j + drow;
    woff[j] = row < E ? (uint32_t(row) * uint32_t(H) + uint32_t(wave * Hq)) * 2u + uint32_t(swz(row, dpos)) * 16u
                      : 0x80000000u;
  }
  const int dst = opaque_s(wave * kWaveStage);
  auto issue = [&](uint8_t* stage, int s) {           // past the end as router_lds_kernel
    const uint32_t past = s < steps ? 0u : 0x80000000u;
    const int kb = s < steps ? s * kRow : 0;
#pragma unroll
    for (int j = 0; j < 2; ++j)
      __builtin_amdgcn_global_load_lds(s * kRingK + xk[j] < Hq ? xrow[j] + s * kRingK : x, stage + (dst + j * 1024),
                                       16, 0, 2);
#pragma unroll
    for (int j = 0; j < kLoads - 2; ++j)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rw, stage + (dst + (j + 2) * 1024), 16, woff[j] | past, kb, 0, 0);
  };
  int at[2];
#pragma unroll
  for (int u = 0; u < 2; ++u) at[u] = opaque_v(wave * kWaveStage + r16 * kRow + swz(r16, 4 * u + kq) * 16);
  f32x4 acc[NB];
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) acc[nb] = f32x4{0.f, 0.f, 0.f, 0.f};
  auto step = [&](const uint8_t* cur, uint8_t* nxt, int s) {
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_waitcnt(wait_vm(kLoads));
    __builtin_amdgcn_sched_barrier(0);
    issue(nxt, s + 2);
    __builtin_amdgcn_sched_barrier(0);
    bf16x8 a[2], b[2][NB];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      a[u] = *reinterpret_cast<const bf16x8*>(cur + at[u]);
#pragma unroll
      for (int nb = 0; nb < NB; ++nb)
        b[u][nb] = *reinterpret_cast<const bf16x8*>(cur + (at[u] + (kTok + nb * 16) * kRow));
    }
#pragma unroll
    for (int u = 0; u < 2; ++u)
      if (u == 0 || 2 * s + u < chunks) {
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) acc[nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[u], b[u][nb], acc[nb], 0, 0, 0);
      }
  };
  issue(st0, 0);
  __builtin_amdgcn_sched_barrier(0);                  // the waits count on this order
  issue(st1, 1);
  int s = 0;
  for (; s + 3 <= steps; s += 3) {
    step(st0, st2, s);
    step(st1, st0, s + 1);
    step(st2, st1, s + 2);
  }
  if (s < steps) step(st0, st2, s);
  if (s + 1 < steps) step(st1, st0, s + 1);
  __builtin_amdgcn_s_waitcnt(wait_vm(0));             // no load may still be on its way into this LDS
  __syncthreads();                                    // every wavefront is done with the stages
  static_assert(kSplitWaves * kTok * (EP + 1) * 4 <= kSplitWaves * kWaveStage, "the logits fit a stage");
  float (*s_part)[kTok][EP + 1] = reinterpret_cast<float (*)[kTok][EP + 1]>(st0);
#pragma unroll
  for (int nb = 0; nb < NB; ++nb)
#pragma unroll
    for (int q = 0; q < 4; ++q) s_part[wave][4 * kq + q][nb * 16 + r16] = acc[nb][q];
  __syncthreads();
  if (wave != 0) return;

  // selection: token tt = lane / 4, lane g = lane % 4 holds experts g V .. g V + V - 1
  const int tt = lane >> 2;
  const int g = lane & 3;
  const int64_t t = t0 + tt;
  const bool valid = t < T;
  const int e0 = g * V;
  float vals[V];
  uint32_t key[V];
#pragma unroll
  for (int v = 0; v < V; ++v) {
    const bool live = e0 + v < E;
    float l = 0.f;
    if (live) {
      l = s_part[0][tt][e0 + v];
#pragma unroll
      for (int q = 1; q < kSplitWaves; ++q) l += s_part[q][tt][e0 + v];   // quarters in k order
    }
    vals[v] = l;
    key[v] = live ? orderable(l) : 0u;
  }
  if (logits_out != nullptr && valid) {
#pragma unroll
    for (int v = 0; v < V; ++v)
      if (e0 + v < E) logits_out[t * E + e0 + v] = vals[v];
  }
  select_topk<V, KMAX>(vals, key, e0, g, E, k, renormalize, valid, t, topk_ids, topk_w);
}

template <int NB>
hipError_t launch_splitk(const uint16_t* x, const uint16_t* w, int64_t T, int E, int k, int H, int renorm,
                         float* logits, int32_t* ids, float* wts, hipStream_t s) {
  const dim3 grid(unsigned((T + kTok - 1) / kTok));
  const dim3 block(kSplitWaves * 64);
  if (k <= 4)
    MOE_LAUNCH("router_topk", (router_splitk_kernel<NB, 4>), grid, block, s, x, w, T, E, k, H, renorm, logits,
               ids, wts);
  else if (k <= 8)
    MOE_LAUNCH("router_topk", (router_splitk_kernel<NB, 8>), grid, block, s, x, w, T, E, k, H, renorm, logits,
               ids, wts);
  else
    MOE_LAUNCH("router_topk", (router_splitk_kernel<NB, kMaxTopK>), grid, block, s, x, w, T, E, k, H, renorm,
               logits, ids, wts);
  return hipGetLastError();
}

template <int NB, int WV>
hipError_t launch_lds(const uint16_t* x, const uint16_t* w, int64_t T, int E, int k, int H, int renorm,
                      float* logits, int32_t* ids, float* wts, hipStream_t s) {
  const dim3 grid(unsigned((T + WV * kTok - 1) / (WV * kTok)));
  const dim3 block(WV * 64);
  if (k <= 4)
    MOE_LAUNCH("router_topk", (router_lds_kernel<NB, 4, WV>), grid, block, s, x, w, T, E, k, H, renorm, logits, ids,
               wts);
  else if (k <= 8)
    MOE_LAUNCH("router_topk", (router_lds_kernel<NB, 8, WV>), grid, block, s, x, w, T, E, k, H, renorm, logits, ids,
               wts);
  else
    MOE_LAUNCH("router_topk", (router_lds_kernel<NB, kMaxTopK, WV>), grid, block, s, x, w, T, E, k, H, renorm, logits,
               ids, wts);
  return hipGetLastError();
}

// Split k where its blocks, one per 16 tokens, run all at once: by LDS a compute unit holds
// one (E > 32), two (E > 16) or three.  8192 tokens x H 7168, 64 experts (two rounds): 50 us,
// two wavefronts per block 36; 8192 x 2048, 32 (one round): 11.4 and 12.0.  Then two wavefronts
// per block while that leaves a compute unit at most one block (8192 x 7168, 64: 36 us, four
// wavefronts 41), then four (12288: 43 us, two 57).
template <int NB>
hipError_t launch_nb(const uint16_t* x, const uint16_t* w, int64_t T, int E, int k, int H, int renorm,
                     float* logits, int32_t* ids, float* wts, int num_cu, hipStream_t s) {
  const int64_t split_blocks = int64_t(num_cu) * (NB >= 3 ? 1 : NB == 2 ? 2 : 3);
  if (H % (kSplitWaves * 32) == 0 && T <= split_blocks * kTok)
    return launch_splitk<NB>(x, w, T, E, k, H, renorm, logits, ids, wts, s);
  if (T <= int64_t(num_cu) * 2 * kTok) return launch_lds<NB, 2>(x, w, T, E, k, H, renorm, logits, ids, wts, s);
  return launch_lds<NB, 4>(x, w, T, E, k, H, renorm, logits, ids, wts, s);
}

}  // namespace

hipError_t launch_router_topk(const uint16_t* x, const uint16_t* w, int64_t T, int E, int k, int H, int renorm,
                              float* logits, int32_t* ids, float* wts, int num_cu, hipStream_t s) {
  switch ((E + 15) / 16) {
    case 1: return launch_nb<1>(x, w, T, E, k, H, renorm, logits, ids, wts, num_cu, s);
    case 2: return launch_nb<2>(x, w, T, E, k, H, renorm, logits, ids, wts, num_cu, s);
    case 3: return launch_nb<3>(x, w, T, E, k, H, renorm, logits, ids, wts, num_cu, s);
    default: return launch_nb<4>(x, w, T, E, k, H, renorm, logits, ids, wts, num_cu, s);
  }
}

}  // namespace moe
