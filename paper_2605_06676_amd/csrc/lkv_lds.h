// Direct copies from memory to LDS, without a register in between.
#pragma once
#include <hip/hip_runtime.h>

namespace lkv {

// 16 (4) bytes per lane from memory to LDS: lane l's go to dst + 16 l (4 l); dst is the same in the whole wave
__device__ __forceinline__ void lds_fill16(const unsigned char* src, unsigned char* dst) {
  __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)src,
                                   (__attribute__((address_space(3))) void*)dst, 16, 0, 0);
}
__device__ __forceinline__ void lds_fill4(const float* src, unsigned char* dst) {
  __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)src,
                                   (__attribute__((address_space(3))) void*)dst, 4, 0, 0);
}

// A barrier that publishes rows copied this way.  The barrier itself orders LDS reads and writes and waits for no copy
// (whether the compiler happens to wait in front of it depends on what else the wave has loaded), so every wave first
// waits for its own: vmcnt(0), the other counters untouched.
__device__ __forceinline__ void lds_fill_barrier() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt(0x0f70);
  asm volatile("" ::: "memory");
  __syncthreads();
}

}  // namespace lkv
