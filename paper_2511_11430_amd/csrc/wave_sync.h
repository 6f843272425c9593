// Exchange of data between the lanes of one wavefront through LDS.
#pragma once

#include <hip/hip_runtime.h>

namespace vpm {

// What any lane of this wavefront wrote to LDS before it is seen by every lane's reads after it, and
// reads before it are done before writes after it.  The hardware keeps a wavefront's LDS accesses
// in order, so no instruction is needed; the fences (of LDS only) keep the compiler from reordering them,
// which the barrier between them, declared as touching no memory, does not.
__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront", "local");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront", "local");
}

}  // namespace vpm
