// A workgroup barrier for data exchanged through LDS.
#pragma once

#include <hip/hip_runtime.h>

namespace qme {

// __syncthreads with its wait for the wave's own LDS accesses spelt out.  In a
// loop that writes at its end and has the barrier at its head (ds_write, branch,
// s_barrier) the compiler has left that wait out, so that another wave could read
// a value before it was written: a few elements of a batch of 256 systems
// differed in the last place between runs of the series passes.  Used wherever a
// loop has that form, whether or not the compiler keeps the wait there today.
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
  __builtin_amdgcn_s_waitcnt(0xC07F);   // lgkmcnt(0); vmcnt and expcnt not waited for
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
}

}  // namespace qme
