// Device-side helpers shared by the kernels.
#pragma once
#include <hip/hip_runtime.h>

namespace fps {

// A pointer read from a table, marked as one to global memory.  The compiler
// cannot know that and accesses through it as "flat", which counts as an LDS
// access too: every wait for LDS then waits for the loads in flight as well
// (product tables: 6.01 -> 5.83 ms for a batch of 256, 17.2 -> 16.3 ms for 16 x 2048
// forward and backward).
template <typename T>
__device__ __forceinline__ T *as_global(T *p) {
  return (T *)(__attribute__((address_space(1))) T *)(uintptr_t)p;
}

typedef double double2v __attribute__((ext_vector_type(2)));

// Doubles through a buffer descriptor: a uniform base, a uniform and the lanes' byte
// offset (below 2^32) are all added by the access.  (From a pointer the compiler adds
// 64-bit addresses per lane, and vector instructions take the matrix unit's time in
// FP64.)  load2 / store2 need 8-byte alignment only.
struct Buffer {
  __amdgpu_buffer_rsrc_t r;
  __device__ __forceinline__ explicit Buffer(const double *p)
      : r(__builtin_amdgcn_make_buffer_rsrc((void *)p, 0, 0xffffffffu, 0x00027000)) {}
  __device__ __forceinline__ double load(uint32_t lane, uint32_t uniform) const {
    return __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(r, lane, uniform, 0));
  }
  __device__ __forceinline__ void store(double v, uint32_t lane, uint32_t uniform) const {
    typedef uint32_t u2 __attribute__((ext_vector_type(2)));
    __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u2, v), r, lane, uniform, 0);
  }
  __device__ __forceinline__ void store2(double2v v, uint32_t lane, uint32_t uniform) const {
    typedef uint32_t u4 __attribute__((ext_vector_type(4)));
    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u4, v), r, lane, uniform, 0);
  }
  __device__ __forceinline__ double2v load2(uint32_t lane, uint32_t uniform) const {
    return __builtin_bit_cast(double2v, __builtin_amdgcn_raw_buffer_load_b128(r, lane, uniform, 0));
  }
};

}  // namespace fps
