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

}  // namespace fps
