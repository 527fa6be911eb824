// Exchanges through LDS between the lanes of one wave.
#pragma once

#include <hip/hip_runtime.h>

namespace fgl {

// Orders a wave's LDS accesses before this point against those after it, for
// lanes that read what other lanes of their wave wrote (or the reverse).  The
// lanes run in step and LDS serves a wave in order, so no instruction is needed;
// the fence keeps the compiler from moving the accesses, which the barrier alone
// (it has no memory effect) allows.
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

}  // namespace fgl
