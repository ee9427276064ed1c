// The last block of a launch goes on with what the whole launch has left in memory: reductions that would otherwise be a
// second launch of one block.
#pragma once
#include "common.hpp"

namespace adapt {

// True in every thread of the block that finishes last.  The word is zero before the launch and zero again after it; the
// partial results are stored and read at device scope (store_partial, load_partial), and stored by threads of the block's
// first wavefront only: the release below is that wavefront's, and the barrier before it does not wait for global stores of
// the others to arrive.
__device__ __forceinline__ bool finished_last(uint32_t *ticket)
{
    __shared__ bool last;
    __syncthreads();
    if (threadIdx.x == 0) {
        // release this wavefront's partial results, acquire everyone else's
        last = __hip_atomic_fetch_add(ticket, 1u, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT) == gridDim.x - 1;
        if (last) __hip_atomic_store(ticket, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);      // for the next launch
    }
    __syncthreads();
    return last;
}

template <typename T>
__device__ __forceinline__ void store_partial(T *p, T v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
template <typename T>
__device__ __forceinline__ T load_partial(const T *p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }

}  // namespace adapt
