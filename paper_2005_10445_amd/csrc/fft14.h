// 16384-point FFT on one workgroup of 16 waves, with a single workgroup-wide
// exchange per transform.
//
// Thread t = 64 w + l (wave w, lane l) holds v[m] = x[t + 1024 m] on entry.
// With N = 16384 = 16 * 1024 and 1024 = 16 * 64 = 16 * (16 * 4):
//
//   A : 16-point DFT over m in registers -> A[t][k1]
//   X1: workgroup exchange through LDS: wave w' receives A[l + 64 m'][k1 = w'];
//       the outer twiddle exp(s j 2 pi t k1 / N) is split into a wave-uniform
//       part exp(s j 2 pi w' m' / 256) (scalar registers) and a per-lane part
//       exp(s j 2 pi w' l / N) that is common to all m' and is folded into the
//       next twiddle layer;
//   B1: 16-point DFT over m' -> k2a, whose outputs carry the twiddle
//       exp(s j 2 pi l (w' + 16 k2a) / N);
//   X2: wave-private exchange: lane (k2a, q) receives the 16 values l = q + 4 m'';
//   B2: 16-point DFT over m'' -> kb1, whose outputs carry exp(s j 2 pi q kb1 / 64);
//   X3: wave-private 4 x 4 exchange inside each lane quad;
//   B3: 4-point DFTs over q.
//
// Every twiddle layer is applied after its exchange, on the inputs of the next
// DFT, where a butterfly a +/- w b takes the product in (six instructions where
// product and additions take eight, see device_fft.h).  The layer before B2
// comes from a table laid out [w'][m''][lane]; the layer before B3 from LDS, a
// quarter of it being 1.  Against products on the outputs this took the
// VALU instructions of a transform from 776 to 652 per wave with half the
// outputs (searching 2^20 samples for 64 tags in 11 bins: 2.35 -> 2.18 ms a call;
// power errors against FP64 are the same to 1%, 3.17e-7 rms of max(P, L Pxhat)).
//
// On exit lane l of wave w holds, in v[4 j + kb2], the output with index
//   u = w + 16 (l >> 2) + 1024 (l & 3) + 256 j + 4096 kb2.
//
// Every wave works on its own slice of LDS after X1, so only X1 needs
// workgroup barriers; X2 and X3 are ordered within the wave.  Each slice is 16
// rows of 64 complex plus 4 pad, which makes every exchange free of bank
// conflicts (for both 32 and 64 four-byte banks).  A transform begins with a
// barrier before its X1 writes (the previous transform's X2/X3 use every
// slice), so work before that point -- loading and scaling the next input and
// stage A -- overlaps the slower waves' end of the previous transform.
// With hi = false only outputs kb2 = 0, 1 (u < 8192) are formed.
#pragma once

#include <hip/hip_runtime.h>

#include "device_fft.h"

namespace acq {
namespace dev {

// Order LDS accesses of one wave (LDS executes a wave's instructions in order;
// this only keeps the compiler from moving them across).
__device__ __forceinline__ void wave_lds_order() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

template <int S>
__device__ __forceinline__ float2 tw_sign(float2 w) {
    return S > 0 ? w : make_float2(w.x, -w.y);
}

struct Fft14 {
    static constexpr int LOGN = 14;
    static constexpr int N = 1 << 14;
    static constexpr int NT = 1024;
    static constexpr int ROW = 68;                  // 64 + 4 pad
    static constexpr int SLICE = 16 * ROW;
    static constexpr int LDS = 16 * SLICE;          // complex elements
    // B3 twiddles [p][j][q - 1] = exp(+j 2 pi q (4 p + j) / 64), q = 1 .. 3, in
    // rows of 13 entries: a lane reads its row from one base register with
    // immediate offsets, and the four rows of a lane quad start on distinct
    // LDS banks
    static constexpr int TROW = 13;
    static constexpr int EXTRA = 4 * TROW;
    // B2 twiddle table entries: [w][m][4 k2a + q] = exp(+j 2 pi l (w + 16 k2a) / N), l = q + 4 m
    static constexpr int B1_TABLE = 16 * 16 * 64;

    int w, l;
    float2 wu[16];                                  // exp(+j 2 pi w m / 256), wave-uniform

    // roots: exp(+j 2 pi x / N), x < N.  extra: LDS table of EXTRA entries,
    // visible to the workgroup after the first transform's X1 barrier.
    __device__ __forceinline__ void init(const float2* __restrict__ roots, float2* extra) {
        w = __builtin_amdgcn_readfirstlane(int(threadIdx.x) >> 6);
        l = int(threadIdx.x) & 63;
#pragma unroll
        for (int m = 0; m < 16; ++m) wu[m] = roots[(w * m * 64) & (N - 1)];
        if (threadIdx.x < EXTRA) {
            const int p = int(threadIdx.x) / TROW, e = int(threadIdx.x) % TROW;
            extra[threadIdx.x] = roots[(((e % 3 + 1) * (4 * p + e / 3)) & 63) * (N / 64)];
        }
    }

    // index of the element in input register m
    __device__ __forceinline__ int in_index(int m) const { return (w << 6) + l + m * NT; }
    // output register r = 4 j + kb2 holds index out_base() + out_off(r)
    __device__ __forceinline__ int out_base() const { return w + 16 * (l >> 2) + 1024 * (l & 3); }
    // smallest / largest out_base() over the wave (wave-uniform)
    __device__ __forceinline__ int out_min() const { return w; }
    __device__ __forceinline__ int out_max() const { return w + 16 * 15 + 1024 * 3; }
    static constexpr int out_off(int r) { return 256 * (r >> 2) + 4096 * (r & 3); }
    static constexpr bool HAS_UPPER = true;     // hi = false leaves out the outputs from HI_OFF on
    static constexpr int HI_OFF = 8192;         // outputs with kb2 >= 2 start here
    static constexpr int LOW_MAX = 256 * 3 + 4096;   // largest out_off below HI_OFF
    // register holding the rr-th smallest output offset (out_off increases with rr)
    static constexpr int visit(int rr) { return ((rr & 3) << 2) | (rr >> 2); }

    template <int S>
    __device__ __forceinline__ void transform(float2 (&v)[16], float2* lds, __amdgpu_buffer_rsrc_t b1tab,
                                              const float2* extra, bool hi = true) const {
        dft16_first(v);
        transform_rest<S>(v, lds, b1tab, extra, hi, [] {});
    }

    // The transform after its first butterflies: v[n] and v[n + 8], n < 8, hold
    // the sum and the difference of inputs n and n + 8.  mid() runs after the
    // transform's last global load is issued: loads it issues (the next input)
    // are not waited for by the transform.
    template <int S, class Mid>
    __device__ __forceinline__ void transform_rest(float2 (&v)[16], float2* lds, __amdgpu_buffer_rsrc_t b1tab,
                                                   const float2* extra, bool hi, Mid mid) const {
        int ln = l;
        asm volatile("" : "+v"(ln));            // recompute lane addressing per call
        // A
        dft16_rest<S>(v);
        __syncthreads();                        // every wave is done with the previous transform's slices
        // X1 write: element (t, k1) -> slice k1, row w, column l.  Slices 8..15
        // lie beyond the 64 KiB reach of a DS immediate offset, so they get a
        // base register of their own (else every store there needs an add).
        {
            float2* p = lds + w * ROW + ln;
            int hi8 = 8 * SLICE;
            asm("" : "+s"(hi8));
            float2* p8 = p + hi8;
#pragma unroll
            for (int k1 = 0; k1 < 8; ++k1) p[k1 * SLICE] = v[k1];
#pragma unroll
            for (int k1 = 0; k1 < 8; ++k1) p8[k1 * SLICE] = v[k1 + 8];
        }
        // B2 twiddles of this lane: the first PRE are loaded before the barrier
        // waits, the rest after X1
        constexpr int PRE = 8;
        const int tboff = (w * 1024 + ln) * 8;
        float2 tb[16];
#pragma unroll
        for (int m = 0; m < PRE; ++m) tb[m] = bload(b1tab, tboff, m * 512);
        __syncthreads();
        float2* sl = lds + w * SLICE;
        // X1 read: wave w gets A[l + 64 m][w]
        {
            const float2* q = sl + ln;
#pragma unroll
            for (int m = 0; m < 16; ++m) v[m] = q[m * ROW];
        }
        // B1, its inputs times the wave-uniform twiddles (the first is 1)
#pragma unroll
        for (int m = 0; m < 8; ++m) {
            const float2 a = m ? cmul(v[m], tw_sign<S>(wu[m])) : v[0];
            bfly_s<S>(a, v[m + 8], wu[m + 8], v[m], v[m + 8]);
        }
        dft16_rest<S>(v);
        // X2: row k2a, column l; lane (k2a', q) reads columns q + 4 m''
        wave_lds_order();
        {
            float2* p = sl + ln;
#pragma unroll
            for (int k2a = 0; k2a < 16; ++k2a) p[k2a * ROW] = v[k2a];
        }
#pragma unroll
        for (int m = PRE; m < 16; ++m) tb[m] = bload(b1tab, tboff, m * 512);
        mid();
        wave_lds_order();
        const int k2 = ln >> 2, q = ln & 3;
        float2* row = sl + k2 * ROW;
        {
            const float2* p = row + q;
#pragma unroll
            for (int m = 0; m < 16; ++m) v[m] = p[4 * m];
        }
        // B2
#pragma unroll
        for (int m = 0; m < 8; ++m)
            bfly_s<S>(cmul(v[m], tw_sign<S>(tb[m])), v[m + 8], tb[m + 8], v[m], v[m + 8]);
        dft16_rest<S>(v);
        // X3: (q, kb1) -> column 4 kb1 + ((q + kb1/4) & 3); lane (k2a, p) reads kb1 = 4 p + j
        wave_lds_order();
#pragma unroll
        for (int a = 0; a < 4; ++a) {
            float2* p = row + ((q + a) & 3) + 16 * a;
#pragma unroll
            for (int b = 0; b < 4; ++b) p[4 * b] = v[4 * a + b];
        }
        wave_lds_order();
#pragma unroll
        for (int qq = 0; qq < 4; ++qq) {
            const float2* p = row + 16 * q + ((qq + q) & 3);
#pragma unroll
            for (int j = 0; j < 4; ++j) v[4 * j + qq] = p[4 * j];
        }
        // B3: inputs 1 .. 3 of each 4-point DFT times their twiddles
        int trow = TROW * q;
        asm("" : "+v"(trow));                   // keep the row base in one register
        const float2* tq = extra + trow;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            float2 s02, d02, s13, d13;
            bfly_s<S>(v[4 * j], v[4 * j + 2], tq[3 * j + 1], s02, d02);
            bfly_s<S>(cmul(v[4 * j + 1], tw_sign<S>(tq[3 * j])), v[4 * j + 3], tq[3 * j + 2], s13, d13);
            const float2 jd = mul_sj<S>(d13);
            v[4 * j] = cadd(s02, s13);
            v[4 * j + 1] = cadd(d02, jd);
            if (hi) {
                v[4 * j + 2] = csub(s02, s13);
                v[4 * j + 3] = csub(d02, jd);
            }
        }
    }
};

}  // namespace dev
}  // namespace acq
