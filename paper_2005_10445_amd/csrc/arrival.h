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
// Every thread of the workgroup comes here.  The count wraps to zero with the last
// arrival, for the next launch, and does so as well when launches that their caller
// failed to order share a ticket: a reset by the last workgroup's store would lose
// the arrivals of the other launch and leave every later search a wrong count.
__device__ __forceinline__ bool last_arrival(unsigned* ticket, unsigned total) {
    __shared__ unsigned s_ticket;
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");     // the wave's stores have arrived
    __syncthreads();
    if (threadIdx.x == 0)
        s_ticket = atomicInc(ticket, total - 1u);          // relaxed, device scope
    __syncthreads();
    return s_ticket == total - 1;
}

// The last workgroup's compaction of a small search: the records of the found
// ones of at most MAX items, in item order, to out and h_out (either may be null),
// at most `capacity` of them; returns how many were found.  slot(e) is item e's
// record in dets, or -1.  NT threads; the slots are listed in LDS and the records
// copied word by word.
template <int NT, int MAX, class Rec, class Slot>
__device__ __forceinline__ int compact_records(int items, const Rec* dets, Slot slot, int capacity, Rec* out,
                                               Rec* h_out) {
    constexpr int WORDS = int(sizeof(Rec) / 8);
    static_assert(sizeof(Rec) % 8 == 0 && NT % 64 == 0, "records of whole words, whole waves");
    __shared__ int s_slot[MAX], s_wave[NT / 64];
    const int t = int(threadIdx.x), lane = t & 63, wave = t >> 6;
    int base = 0;
    for (int e0 = 0; e0 < items; e0 += NT) {
        const int e = e0 + t;
        const int s = e < items ? slot(e) : -1;
        const unsigned long long mask = __builtin_amdgcn_ballot_w64(s >= 0);
        if (lane == 0) s_wave[wave] = __popcll(mask);
        __syncthreads();
        int o = base + __popcll(mask & ((1ull << lane) - 1ull));
        for (int w = 0; w < NT / 64; ++w) {
            if (w < wave) o += s_wave[w];
            base += s_wave[w];
        }
        if (s >= 0) s_slot[o] = s;
        __syncthreads();
    }
    const int n = (base < capacity ? base : capacity) * WORDS;
    constexpr int U = 8;                     // words of a thread in flight together
    for (int i0 = t; i0 < n; i0 += U * NT) {
        unsigned long long v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int i = min(i0 + u * NT, n - 1), r = i / WORDS;
            v[u] = agent_load(reinterpret_cast<const unsigned long long*>(&dets[s_slot[r]]) + (i - r * WORDS));
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int i = i0 + u * NT;
            if (i >= n) break;
            if (out) reinterpret_cast<unsigned long long*>(out)[i] = v[u];
            if (h_out) reinterpret_cast<unsigned long long*>(h_out)[i] = v[u];
        }
    }
    return base;
}

// A record that another workgroup's compact_records reads.
template <class Rec>
__device__ __forceinline__ void agent_store_record(Rec* p, const Rec& r) {
    union {
        Rec rec;
        unsigned long long u[sizeof(Rec) / 8];
    } o;
    o.rec = r;
#pragma unroll
    for (int i = 0; i < int(sizeof(Rec) / 8); ++i) agent_store(reinterpret_cast<unsigned long long*>(p) + i, o.u[i]);
}

}  // namespace acq
