// Device helpers shared by the kernel files: wave reductions and the
// Stockham engine wrapper with the same interface as the 2^14-point engine.
#pragma once

#include <hip/hip_runtime.h>

#include "device_fft.h"
#include "fft14.h"
#include "storage.h"

namespace acq {
namespace kdev {

using dev::bflyc;
using dev::cadd;
using dev::cmul;
using dev::cmulc;
using dev::Fft;
using dev::dft16;

// One step of a wave sum: each lane adds the value DPP control CTRL routes to
// it (lanes with no source, or in rows outside ROW_MASK, add +0).
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ double dpp_add_step(double v) {
    const unsigned long long b = static_cast<unsigned long long>(__double_as_longlong(v));
    const int lo = __builtin_amdgcn_update_dpp(0, int(unsigned(b)), CTRL, ROW_MASK, 0xf, true);
    const int hi = __builtin_amdgcn_update_dpp(0, int(unsigned(b >> 32)), CTRL, ROW_MASK, 0xf, true);
    return v + __longlong_as_double(static_cast<long long>((static_cast<unsigned long long>(unsigned(hi)) << 32) |
                                                          unsigned(lo)));
}

// Sum over the wave in a fixed order (uniform result, no LDS): row_shr 1, 2,
// 4, 8 leave each 16-lane row's sum in its lane 15; row_bcast 15 (into rows 1
// and 3) and row_bcast 31 (into rows 2 and 3) carry the total to lane 63, each
// lane's value counted once.
__device__ __forceinline__ double wave_sum(double v) {
    v = dpp_add_step<0x111, 0xf>(v);
    v = dpp_add_step<0x112, 0xf>(v);
    v = dpp_add_step<0x114, 0xf>(v);
    v = dpp_add_step<0x118, 0xf>(v);
    v = dpp_add_step<0x142, 0xa>(v);
    v = dpp_add_step<0x143, 0xc>(v);
    const unsigned long long b = static_cast<unsigned long long>(__double_as_longlong(v));
    const unsigned lo = unsigned(__builtin_amdgcn_readlane(int(unsigned(b)), 63));
    const unsigned hi = unsigned(__builtin_amdgcn_readlane(int(unsigned(b >> 32)), 63));
    return __longlong_as_double(static_cast<long long>((static_cast<unsigned long long>(hi) << 32) | lo));
}

// Largest value over the wave (uniform, no LDS): the steps of wave_sum.
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ float dpp_fmax_step(float v) {
    const int b = int(__float_as_uint(v));
    return fmaxf(v, __uint_as_float(unsigned(__builtin_amdgcn_update_dpp(b, b, CTRL, ROW_MASK, 0xf, false))));
}

__device__ __forceinline__ float wave_fmax(float v) {
    v = dpp_fmax_step<0x111, 0xf>(v);
    v = dpp_fmax_step<0x112, 0xf>(v);
    v = dpp_fmax_step<0x114, 0xf>(v);
    v = dpp_fmax_step<0x118, 0xf>(v);
    v = dpp_fmax_step<0x142, 0xa>(v);
    v = dpp_fmax_step<0x143, 0xc>(v);
    return __uint_as_float(unsigned(__builtin_amdgcn_readlane(int(__float_as_uint(v)), 63)));
}

// A pointer that is the same in every lane, in scalar registers: a buffer resource made
// of it takes no loop over the lanes' values.
template <class T>
__device__ __forceinline__ const T* wave_uniform(const T* p) {
    const unsigned long long v = reinterpret_cast<unsigned long long>(p);
    const unsigned lo = unsigned(__builtin_amdgcn_readfirstlane(int(unsigned(v))));
    const unsigned hi = unsigned(__builtin_amdgcn_readfirstlane(int(unsigned(v >> 32))));
    return reinterpret_cast<const T*>((static_cast<unsigned long long>(hi) << 32) | lo);
}

// Smallest value over the wave (uniform, no LDS): the same steps.
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ unsigned dpp_umin_step(unsigned v) {
    const unsigned o = unsigned(__builtin_amdgcn_update_dpp(int(v), int(v), CTRL, ROW_MASK, 0xf, false));
    return o < v ? o : v;
}

__device__ __forceinline__ unsigned wave_umin(unsigned v) {
    v = dpp_umin_step<0x111, 0xf>(v);
    v = dpp_umin_step<0x112, 0xf>(v);
    v = dpp_umin_step<0x114, 0xf>(v);
    v = dpp_umin_step<0x118, 0xf>(v);
    v = dpp_umin_step<0x142, 0xa>(v);
    v = dpp_umin_step<0x143, 0xc>(v);
    return unsigned(__builtin_amdgcn_readlane(int(v), 63));
}

// Peak key of the lanes whose largest value bp is the wave's, wm >= 0: the
// smallest index idx among them.  (A loop over those lanes, nearly always one,
// takes 64 turns where all are equal, as in a block of zeros, whose every transform
// reaches its tag's best: 2^20 zeros against 64 tags in 11 bins
// 3.34 ms a call so, 2.17 ms now, noise 2.09.)
__device__ __forceinline__ unsigned long long wave_key(float bp, float wm, unsigned idx) {
    const unsigned best = wave_umin(bp == wm ? idx : ~0u);
    return (static_cast<unsigned long long>(__float_as_uint(wm)) << 32) | static_cast<unsigned long long>(~best);
}

// The value held by a peak key.  Keys only grow during a launch, so one read
// early (past the L1 and this XCD's view) is a lower bound.
__device__ __forceinline__ float key_value(const unsigned long long* key) {
    const unsigned long long k = __hip_atomic_load(key, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return __uint_as_float(unsigned(k >> 32));
}

// ------------------------------------------------------------------ transform engines
// Both engines take v[m] = a[in_index(m)] and leave output index
// out_base() + out_off(r) in v[r].  transform_rest takes the first butterflies
// as done: v[n] and v[n + 8], n < 8, hold the sum and the difference of inputs
// n and n + 8.

// Stockham passes (2^10 .. 2^13 points), see device_fft.h.  IN: twiddles taken
// into the butterflies (the FSK front end keeps products before the DFTs: its
// outputs are reported, and their roundings stay as they were).
template <int LOGN_, bool IN = true>
struct StockhamEngine {
    using F = Fft<LOGN_>;
    static constexpr int LOGN = LOGN_;
    static constexpr int N = F::N;
    static constexpr int NT = F::NT;
    static constexpr int LDS = F::LDS;
    static constexpr int EXTRA = 1;
    static constexpr int B1_TABLE = 1;
    int t;
    __amdgpu_buffer_rsrc_t tw;
    // r: the N unit roots (unused here) and the pass twiddles after them
    __device__ __forceinline__ void init(const float2* __restrict__ r, float2*) {
        t = int(threadIdx.x);
        tw = dev::make_rsrc(r + N, F::TW * 8);
    }
    __device__ __forceinline__ int in_index(int m) const { return t + m * NT; }
    __device__ __forceinline__ int out_base() const { return t; }
    // smallest / largest out_base() over the wave (wave-uniform)
    __device__ __forceinline__ int out_min() const { return __builtin_amdgcn_readfirstlane(t & ~63); }
    __device__ __forceinline__ int out_max() const { return out_min() + 63; }
    static constexpr int out_off(int r) { return r * NT; }
    static constexpr bool HAS_UPPER = false;    // no output is ever left out
    static constexpr int HI_OFF = 1 << 30;
    static constexpr int LOW_MAX = 15 * NT;     // largest out_off below HI_OFF
    // register holding the rr-th smallest output offset
    static constexpr int visit(int rr) { return rr; }
    template <int S>
    __device__ __forceinline__ void transform(float2 (&v)[16], float2* lds, __amdgpu_buffer_rsrc_t,
                                              const float2*, bool = true) const {
        int tq = t;
        asm volatile("" : "+v"(tq));            // recompute addressing per call, no hoisting
        if constexpr (IN)
            F::template transform_in<S, false>(v, lds, tw, tq);
        else
            F::template transform<S>(v, lds, tw, tq);
    }
    template <int S, class Mid>
    __device__ __forceinline__ void transform_rest(float2 (&v)[16], float2* lds, __amdgpu_buffer_rsrc_t, const float2*,
                                                   bool, Mid mid) const {
        static_assert(IN, "the products before the DFTs have no separate first butterflies");
        int tq = t;
        asm volatile("" : "+v"(tq));
        mid();
        F::template transform_in<S, true>(v, lds, tw, tq);
    }
};

using dev::bload;
using dev::dft16_first;
using dev::Fft14;
using dev::make_rsrc;

// LDS position of transform output i for the natural-order staging: bits 0-3
// XOR-ed with a function of bits 4-7 and 10-11, so that both the engine-order
// writes and the lane-consecutive reads hit 16 distinct 8-byte banks per
// 16 lanes (a permutation of [0, N)).
__device__ __forceinline__ int out_swizzle(int i) { return i ^ (((i >> 4) + 4 * (i >> 10)) & 15); }

// Store a transform's outputs in natural order to F[0 .. N): they leave in the
// engine's order, so they are put in order in LDS and whole lines stored.  Ends
// with a barrier (LDS is free again).
template <class E>
__device__ __forceinline__ void store_natural(const E& eng, const float2 (&v)[16], float2* lds, float2* F) {
    const int ob = eng.out_base();
    __syncthreads();                 // every wave is done with the transform's LDS
#pragma unroll
    for (int m = 0; m < 16; ++m) lds[out_swizzle(ob + E::out_off(m))] = v[m];
    __syncthreads();
#pragma unroll
    for (int m = 0; m < 16; ++m) {
        const int i = eng.in_index(m);
        F[i] = lds[out_swizzle(i)];
    }
    __syncthreads();
}

}  // namespace kdev
}  // namespace acq
