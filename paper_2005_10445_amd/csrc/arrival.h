// Results handed from the workgroups of one launch to the last of them to arrive.
#pragma once

#include <hip/hip_runtime.h>

namespace acq {

// Values that another workgroup of the same launch reads: stored through to, and
// loaded from, the memory that the XCDs share (no L2 write-back or invalidation,
// which would take the launch's other data with it).
template <class T>
__device__ __forceinline__ void agent_store(T* p, T v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

template <class T>
__device__ __forceinline__ T agent_load(const T* p) {
    return __hip_atomic_load(const_cast<T*>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Counts this workgroup's arrival at *ticket; true (in the whole workgroup) for
// the last of `total`, which then sees what the others stored with agent_store.
// Every thread of the workgroup comes here.
__device__ __forceinline__ bool last_arrival(unsigned* ticket, unsigned total) {
    __shared__ unsigned s_ticket;
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");     // the wave's stores have arrived
    __syncthreads();
    if (threadIdx.x == 0)
        s_ticket = __hip_atomic_fetch_add(ticket, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __syncthreads();
    return s_ticket == total - 1;
}

}  // namespace acq
