// Exchange between the lanes of one wavefront through LDS.
#pragma once

#include <hip/hip_runtime.h>

namespace sclbm {

// What the lanes of a wavefront wrote to LDS before is read by its other lanes after.  The LDS unit
// runs a wavefront's accesses in order, so no instruction is needed, but the compiler must
// keep the order too: the barrier builtin alone orders execution, not memory, and a load of
// another type than the store's may be moved across it.  The fences order memory.
__device__ __forceinline__ void wave_lds_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

}  // namespace sclbm
