// Order of LDS accesses within a wave (device code of the image-domain kernels).
#pragma once
#include <hip/hip_runtime.h>

namespace lsrtm {

// What a lane of the wave wrote to LDS before is there for the others after,
// and what they read before is read.
__device__ __forceinline__ void wave_order() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

}  // namespace lsrtm
