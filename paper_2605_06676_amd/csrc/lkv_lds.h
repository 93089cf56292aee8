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

}  // namespace lkv
