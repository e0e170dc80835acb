// Helpers of the kernels that stream through rings of LDS stages, filled by direct
// global -> LDS loads.
#pragma once
#include <hip/hip_runtime.h>

namespace moe {

// gfx9 s_waitcnt immediate with only vmcnt(n).
constexpr int wait_vm(int n) { return 0x0F70 | (n & 15) | ((n >> 4) << 14); }

// An offset into a stage's LDS object that the compiler keeps as one value.  It tells a
// stage's reads from the loads in flight to the others by the object that an address comes
// from, and loses that through more than a few additions: it would then wait for every load.
__device__ __forceinline__ int opaque_v(int x) {
  asm("" : "+v"(x));
  return x;
}
__device__ __forceinline__ int opaque_s(int x) {
  asm("" : "+s"(x));
  return x;
}

// A workgroup barrier alone.  __syncthreads would also wait for every load in flight; the
// caller waits for what it needs and keeps the scheduler from moving accesses across.
__device__ __forceinline__ void bare_barrier() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

}  // namespace moe
