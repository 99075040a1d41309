// Workgroup barrier of the kernels that keep global loads in flight across it.
#pragma once

#include <hip/hip_runtime.h>

namespace lbk {

// Workgroup barrier that orders LDS accesses only.  __syncthreads() would also
// wait for every outstanding global load, including what is requested ahead.
__device__ __forceinline__ void lds_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

}  // namespace lbk
