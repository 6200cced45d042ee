// Wave-level helpers shared by the kernels.
#pragma once
#include <hip/hip_runtime.h>

namespace niv {

// LDS accesses of one wave complete in order; the fences keep the compiler
// from moving LDS reads and writes of the wave across this point.
__device__ inline void wave_lds_fence()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

}  // namespace niv
