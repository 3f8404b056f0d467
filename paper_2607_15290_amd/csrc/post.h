// Device side of a Post (krylov.h): results of a reduction in the host's mapped
// memory, announced by a flag that the host polls.
#pragma once
#include "pipeline.h"

namespace llg {

// End of a one-block reduction whose threads have stored their values in the
// mirror (called by every thread of the block).
__device__ __forceinline__ void post_block(const Post& ps) {
  if (!ps.flag) return;
  if (threadIdx.x < ps.n_also) ps.also_mirror[threadIdx.x] = ps.also[threadIdx.x];
  __threadfence_system();
  __syncthreads();
  if (threadIdx.x == 0) __hip_atomic_store(ps.flag, ps.seq, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}

// Posts value v as number blockIdx.x of gridDim.x (called by every thread of
// the block; thread 0 holds v).
__device__ __forceinline__ void post_value(const Post& ps, double v) {
  if (!ps.flag) return;
  if (blockIdx.x == 0 && threadIdx.x < ps.n_also) {
    ps.also_mirror[threadIdx.x] = ps.also[threadIdx.x];
    __threadfence_system();
  }
  if (threadIdx.x == 0) {
    ps.mirror[blockIdx.x] = v;
    __threadfence_system();
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    bool last = true;
    if (gridDim.x > 1) {
      last = atomicAdd(ps.count, 1u) == gridDim.x - 1;
      if (last) atomicExch(ps.count, 0u);
      __threadfence_system();
    }
    if (last) __hip_atomic_store(ps.flag, ps.seq, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
  }
}

}  // namespace llg
