// FSK searching pipeline of Section 3 (steps 1-8) on gfx950, with the FFT
// methods of Section 4.1.
//
//   k_fsk_front     : one workgroup per overlap-save segment of the composed
//                     filters: int16 -> complex and local-oscillator mix (or,
//                     at plan time, the noise-free continuous-phase replica of
//                     a tag's bits), forward 4096-point transform, products
//                     with the spectra of h_BP * h_1 and h_BP * h_0, two inverse
//                     transforms, demodulation d = (|f1|-|f0|)/(|f1|+|f0|),
//                     u = |f1|-|f0|.  Output d and u (block) or d (replica).
//   k_fsk_forward   : overlap-save segments 2s and 2s+1 of the call (numbered
//                     over its blocks) as the real and imaginary parts of one
//                     complex M-point input (slot s), its P = M / Msub decimated
//                     Msub-point transforms, one a workgroup
//   (their combination, and the forward spectra of the templates: the
//    decimation-in-time transform of the acquisition path)
//   k_fsk_first, k_fsk_first_track, k_fsk_phase : the real cross-correlation of
//                     d with each template by overlap-save.  The template d^(c)
//                     is real, so the inverse transform of Z_g conj(D^(c)) / M
//                     holds the correlation of segment 2g in its real part and of
//                     segment 2g+1 in its imaginary part: one complex transform
//                     per two segments.  Two tracking segments with different
//                     templates share a slot too: with Z the slot's spectrum,
//                     X_A = (Z[i] + conj Z[-i]) / 2 and j X_B = (Z[i] -
//                     conj Z[-i]) / 2, so the product is (Z[i] (B_a + B_b) +
//                     conj Z[-i] (B_a - B_b)) / 2 for the conjugate spectra B of
//                     the two templates.  The peak search uses |c|.  An M-point
//                     inverse transform (M up to 2^18) runs as P = M / Msub
//                     phases of an Msub-point transform: for output lag tau =
//                     P u + rho,
//                       G_rho[i'] = exp(+j 2 pi i' rho / M)
//                                   sum_a Y[i' + Msub a] exp(+j 2 pi a rho / P),
//                     Y the spectrum product (first step, k_fsk_first*), then an
//                     Msub-point inverse transform of G_rho (k_fsk_phase).
//                     Keys: bits(|Re c|) << 32 | ~tau.
//   k_fsk_refine    : FP64 sums over +/-3 lags of the peak from the stored d,
//                     u and template (in parts, added in order), re-maximisation,
//                     parabola, w_c, q, p_c, z.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <new>
#include <string>
#include <vector>

#include "acq.h"
#include "arrival.h"
#include "device_common.h"
#include "host_logic.h"
#include "kernels.h"

namespace acq {

using namespace kdev;

namespace {

constexpr int kFrontLog = 12;                 // composed filters applied on 4096-point segments
constexpr int kFrontN = 1 << kFrontLog;
constexpr int kFskPhaseGrid = 256;            // workgroups of the phase transforms: one per CU
// First-step outputs held at a time (complex values, 512 MiB): a search of more
// (template, slot) items runs through them in groups.  Groups small enough for
// the 256 MiB memory-side cache did not pay: a launch of the phase transforms
// costs 15 us before its first transform ends (128 MiB groups: 315 us for the
// 100 ms window's 256 items, 512 MiB: 305 us).
constexpr int64_t kFskGroup = int64_t(1) << 26;
constexpr int kFskPerBlock = 4;               // templates per workgroup of the first step

// One block of an FSK call: the searching window (tag -1: every template) or
// one tracking task (its tag only).  Front-end segments and correlation
// segments are numbered globally over the call's blocks; slot s holds
// correlation segments 2s and 2s+1, which may belong to different blocks.
struct FskTask {
    const int16_t* iq;          // device [n][2]
    int64_t n;                  // samples
    int64_t lags;               // n - n_t + 1 (<= 0: nothing to search)
    int64_t zoff;               // offset of the block's d and u in the plan's arrays
    int32_t tag;                // -1 searching; else the tracked template
    int32_t fseg0, nfseg;       // front-end segments
    int32_t unit0;              // first correlation segment (global number)
    int32_t nseg;               // overlap-save segments of the correlation
};

// One correlation segment of a call: slot s holds units 2s and 2s+1.
struct FskUnit {
    int64_t z0;                 // first sample of the segment in the plan's d
    int32_t left;               // samples from there to the end of its block (at most M)
    int32_t vlim;               // valid lags (0: an absent second unit)
    uint32_t lag0;              // lag of its first output
    int32_t tag;                // tracking: the template
    int32_t key;                // tracking: result index
    int32_t reserved;
};

struct FskTasks {
    const FskTask* t;           // device [count]
    int32_t count;
    int32_t track;              // 1: tracking tasks (one template each)
};

// block holding global front-end segment g, by binary search
__device__ __forceinline__ int fsk_task_of(const FskTasks& tt, int g) {
    int lo = 0, hi = tt.count - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (tt.t[mid].fseg0 <= g) lo = mid; else hi = mid - 1;
    }
    return lo;
}

struct FrontArgs {
    FskTasks tasks;             // blocks (block mode)
    const uint8_t* bits;        // replica: [T][nbits]
    const double* bit_cyc;      // replica: [T][nbits] carrier phase (cycles, in [0,1)) at each bit start
    const float2* G1;           // [kFrontN] DFT(h_BP * h_1) / kFrontN
    const float2* G0;
    const float2* roots;        // [kFrontN] exp(+j 2 pi m / kFrontN), then the pass twiddles
    float2* out;                // replica: [T][out_stride] (d, 0)
    float* out_d;               // block: d at the block's zoff
    float* out_u;               // block: u at the block's zoff
    unsigned long long* keys;   // block: [nkeys] peak keys to clear
    int32_t nkeys;
    int64_t n_in, n_out, out_stride;     // replica mode
    double lo_cyc;              // f_LO / Fs
    float2 lo_step[16];         // exp(-j 2 pi (f_LO / Fs) (NT m)), m < 16 (FP64, rounded once)
    double f1_cyc, f0_cyc;      // tones, cycles per sample
    int32_t nbits, sps, lg, vf, nseg;   // nseg: segments per replica
};

// One workgroup per (template, segment) of the replicas or per global segment
// of the blocks: outputs s*vf .. s*vf + vf - 1 of the causal convolution with
// the composed filters, from inputs s*vf - (lg-1) ..  Four workgroups per CU (128
// VGPRs; the forward spectrum stays in registers through the first inverse
// transform), three when the templates and the blocks shared one kernel: 64 blocks
// of 96,000 samples, 1600 workgroups, 56 us in three rounds, 50.5 us in two.  The
// last butterflies of the second tone's transform and the roots and quotients lie
// within the branch around each output.  Formed without branches they overlap
// (46.8 us), but their products then fuse with the sums: other roundings of d and u
// than before, 5e-10 of the FP64 results.
// REPLICA: the templates, at plan time.
template <bool REPLICA>
__global__ __launch_bounds__(256, 4) void k_fsk_front(FrontArgs a) {
    using E = StockhamEngine<kFrontLog, false>;
    __shared__ float2 lds[E::LDS];
    E eng;
    eng.init(a.roots, nullptr);
    int s, tag = 0;
    const int16_t* iq = nullptr;
    int64_t n_in = a.n_in, n_out = a.n_out, zoff = 0;
    if constexpr (REPLICA) {
        s = int(blockIdx.x) % a.nseg;
        tag = int(blockIdx.x) / a.nseg;
    } else {
        for (int i = int(blockIdx.x) * 256 + int(threadIdx.x); i < a.nkeys; i += int(gridDim.x) * 256) a.keys[i] = 0ull;
        const int b = fsk_task_of(a.tasks, int(blockIdx.x));
        const FskTask tk = a.tasks.t[b];
        s = int(blockIdx.x) - tk.fseg0;
        iq = tk.iq;
        n_in = n_out = tk.n;
        zoff = tk.zoff;
    }
    const int64_t base = int64_t(s) * a.vf - (a.lg - 1);
    float2 x[16];
    if constexpr (REPLICA) {
#pragma unroll
        for (int m = 0; m < 16; ++m) {
            const int64_t p = base + eng.in_index(m);
            float2 v = make_float2(0.f, 0.f);
            if (p >= 0 && p < n_in) {
                const int64_t b = p / a.sps;
                const size_t bi = size_t(tag) * size_t(a.nbits) + size_t(b);
                double cyc = a.bit_cyc[bi] + (a.bits[bi] ? a.f1_cyc : a.f0_cyc) * double(p - b * a.sps);
                cyc -= floor(cyc);                          // exact phase reduction in FP64
                float sn, cs;
                sincospif(2.0f * float(cyc), &sn, &cs);
                v = make_float2(cs, sn);
            }
            x[m] = v;
        }
    } else {
        // LO mix exp(-j 2 pi f_LO p / Fs) at p = p0 + NT m: the phase of p0 is
        // reduced exactly in FP64 once per thread, and register m rotates it
        // by the constant lo_step[m]
        const int64_t p0 = base + eng.in_index(0);
        double cyc = -a.lo_cyc * double(p0);
        cyc -= floor(cyc);
        float sn0, cs0;
        sincospif(2.0f * float(cyc), &sn0, &cs0);
        const float2 e0 = make_float2(cs0, sn0);
        // samples outside the block are zero: buffer loads bounded by the
        // block's samples (those before its start at offset -1, past every
        // bound), so that all 16 are in flight together.  Offsets must not wrap:
        // where a negative one plus the load's immediate offset crosses zero
        // within four lanes, the lanes past it read zero too.
        const int64_t first = base > 0 ? base : 0;
        const int64_t left = n_in - first < kFrontN ? n_in - first : kFrontN;
        const __amdgpu_buffer_rsrc_t ir = make_rsrc(iq + 2 * first, left > 0 ? uint32_t(left) * 4u : 0u);
        uint32_t raw[16];
#pragma unroll
        for (int m = 0; m < 16; ++m)
            raw[m] = __builtin_amdgcn_raw_buffer_load_b32(ir, max(int(base - first) + eng.in_index(m), -1) * 4, 0, 0);
#pragma unroll
        for (int m = 0; m < 16; ++m) {
            const float2 e = m ? cmul(e0, a.lo_step[m]) : e0;
            x[m] = cmul(make_float2(float(int16_t(raw[m] & 0xffffu)), float(int16_t(raw[m] >> 16))), e);
        }
    }
    const __amdgpu_buffer_rsrc_t dummy = make_rsrc(a.roots, 8);   // unused by the Stockham engine
    eng.template transform<-1>(x, lds, dummy, nullptr);
    const __amdgpu_buffer_rsrc_t g1 = make_rsrc(a.G1, kFrontN * 8), g0 = make_rsrc(a.G0, kFrontN * 8);
    const int in0 = eng.in_index(0);                         // in_index(m) = in0 + NT m
    float a1[16];
    float2 w[16];
#pragma unroll
    for (int m = 0; m < 16; ++m) w[m] = cmul(x[m], bload(g1, in0 * 8, E::NT * m * 8));
    eng.template transform<+1>(w, lds, dummy, nullptr);
#pragma unroll
    for (int m = 0; m < 16; ++m) a1[m] = sqrtf(fmaf(w[m].x, w[m].x, w[m].y * w[m].y));
#pragma unroll
    for (int m = 0; m < 16; ++m) w[m] = cmul(x[m], bload(g0, in0 * 8, E::NT * m * 8));
    eng.template transform<+1>(w, lds, dummy, nullptr);
#pragma unroll
    for (int m = 0; m < 16; ++m) {
        const int idx = eng.in_index(m);                     // natural order in and out
        const int64_t o = int64_t(s) * a.vf + idx - (a.lg - 1);
        if (idx >= a.lg - 1 && o < n_out) {
            const float a0 = sqrtf(fmaf(w[m].x, w[m].x, w[m].y * w[m].y));
            const float sum = a1[m] + a0, dif = a1[m] - a0;
            const float d = sum > 0.f ? dif / sum : 0.f;
            if constexpr (REPLICA) {
                a.out[size_t(tag) * size_t(a.out_stride) + size_t(o)] = make_float2(d, 0.f);
            } else {
                a.out_d[zoff + o] = d;
                a.out_u[zoff + o] = dif;
            }
        }
    }
}

// Decimated transforms of the call's slots: work item (slot s, phase r) is the
// Msub-point DFT of the values at i = P n + r of the slot's input, the two
// segments' samples of d as real and imaginary parts (zero past their blocks),
// written to X[s][r Msub + .].  The P items of a slot read interleaved samples
// of one range and are placed on one XCD, as in the acquisition path's forward
// transform.  The samples come straight from d: a packed copy in between cost
// 17 us of its own for 64 blocks of 96,000 samples.
template <class E>
__global__ __launch_bounds__(E::NT, 4) void k_fsk_forward(const FskUnit* __restrict__ units, const float* __restrict__ d,
                                                          int P, int M, int items, const float2* __restrict__ rootsSub,
                                                          const float2* __restrict__ b1tab, float2* __restrict__ X) {
    __shared__ float2 lds[E::LDS];
    __shared__ float2 extra[E::EXTRA];
    E eng;
    eng.init(rootsSub, extra);
    const __amdgpu_buffer_rsrc_t b1 = make_rsrc(b1tab, E::B1_TABLE * 8);
    const int grp = kXcds * P, b = int(blockIdx.x);
    int it = b;
    if (b < items / grp * grp) {
        const int q = b / grp, j = b - q * grp;
        it = (q * kXcds + j % kXcds) * P + j / kXcds;
    }
    const int s = it / P, r = it - s * P;
    const FskUnit ua = units[2 * s], ub = units[2 * s + 1];
    const __amdgpu_buffer_rsrc_t ra = make_rsrc(d + ua.z0, uint32_t(ua.left) * 4u);
    const __amdgpu_buffer_rsrc_t rb = make_rsrc(d + ub.z0, uint32_t(ub.left) * 4u);
    float2 v[16];
#pragma unroll
    for (int m = 0; m < 16; ++m) {
        const int off = (P * eng.in_index(m) + r) * 4;
        v[m].x = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(ra, off, 0, 0));
        v[m].y = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rb, off, 0, 0));
    }
    eng.template transform<-1>(v, lds, b1, extra);
    store_natural(eng, v, lds, X + size_t(s) * size_t(M) + size_t(r) * size_t(E::N));
}

// bank[t][i] = conj(X_t[i]) / M in place
__global__ void k_fsk_conj_scale(float2* bank, int64_t count, float scale) {
    const int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (i < count) {
        const float2 v = bank[i];
        bank[i] = make_float2(v.x * scale, -v.y * scale);
    }
}

// phases[r][i] = exp(+j 2 pi i r / M), i < Msub, r < P
__global__ void k_fsk_phase_roots(const float2* __restrict__ rootsM, int Msub, float2* __restrict__ phases) {
    const int o = int(blockIdx.x) * 256 + int(threadIdx.x);
    phases[o] = rootsM[(o / Msub) * (o % Msub)];
}

// rows of real parts: out[t][i] = in[t][i].x, i < stride, of count values in all
__global__ void k_fsk_real(const float2* __restrict__ in, int64_t in_stride, float* __restrict__ out, int64_t stride,
                           int64_t count) {
    const int64_t o = int64_t(blockIdx.x) * 256 + threadIdx.x;
    if (o < count) out[o] = in[o / stride * in_stride + o % stride].x;
}

__global__ void k_fsk_fill(float2* p, int64_t count) {
    const int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (i < count) p[i] = make_float2(0.f, 0.f);
}

struct FskCorrArgs {
    float2* X;                  // [slots][M] spectra of the packed segment pairs (tracking with P > 1: the
                                // decimated transforms, not yet combined)
    const float2* bank;         // [T][M] conj(DFT_M(d^(c))) / M
    const float2* rootsM;       // [M]
    const float2* phases;       // [P][Msub] exp(+j 2 pi i r / M) (2 < P <= 8)
    const float2* rootsSub;     // [Msub], then the pass twiddles
    const float2* b1tab;
    float2* G;                  // [items of the launch][P][Msub] first-step outputs (P > 1)
    unsigned long long* keys;   // [T] (searching) or [tasks] (tracking)
    float* dump;                // optional [T][lags]: c at every lag (test hook, searching)
    const FskUnit* units;       // device [2 slots]
    int64_t lags;               // lags of the searched block (dump)
    int32_t M, Msub, P, track;
    int32_t t0, nt, s0, ns;     // the launch's templates (searching) and slots; item i: template t0 + i / ns,
                                // slot s0 + i % ns; tracking: slot s0 + i
};

// w[r] = exp(+j 2 pi i r / M), i < Msub, r < P (w[0] unset): from a table [r][i], or for
// P = 16, whose first step is bound by its loads, as powers of the first.  Powers round
// r times: for P = 8 they give 5.92e-7 rms of an output's scale where the table's give
// 5.35e-7, for P = 4 4.94e-7 and 4.78e-7.  (Gathered from rootsM, at i r, they take
// 33 tasks over eight phases 136 us a call; 134 so, 133 with powers.)
template <int P>
__device__ __forceinline__ void phase_twiddles(const FskCorrArgs& a, int i, float2 (&w)[P]) {
    w[1] = a.rootsM[i];
#pragma unroll
    for (int r = 2; r < P; ++r) w[r] = P > 8 ? cmul(w[r - 1], w[1]) : a.phases[r * a.Msub + i];
}

// P-point DFT, P a power of two
template <int P, int S>
__device__ __forceinline__ void dft_p(float2 (&y)[P]) {
#pragma unroll
    for (int r = 0; r < P / 2; ++r) dev::dft2<S>(y[r], y[r + P / 2]);
    dev::dft_rest<P, S>(y);
}

// First step of a search, P > 1: for input index i' of a pair of slots, with
// every template of the workgroup, the P products Y_a = Z[i' + Msub a]
// B[i' + Msub a] and G_rho[i'] = exp(+j 2 pi i' rho / M) sum_a Y_a
// exp(+j 2 pi a rho / P).  It streams the bank in (once for the two slots) and
// G out and is bound by that, so it is a kernel of its own with many more loads
// in flight than the one workgroup of a 2^14-point transform that a CU holds.
// 128 templates, 800,000 samples, M = 2^18: 386 us for both steps in one kernel,
// 305 us so (this one 145 us at 5.6 TB/s).
// (Reading half the bank, each thread taking i' and Msub - i', needs 256
// registers and was slower.)
template <int P>
__global__ __launch_bounds__(256, 2) void k_fsk_first(FskCorrArgs a) {
    const int nib = a.Msub / 256, npair = (a.ns + 1) / 2;
    int rem = int(blockIdx.x);
    const int ip = (rem % nib) * 256 + int(threadIdx.x);
    rem /= nib;
    const int sl = 2 * (rem % npair), ta = (rem / npair) * kFskPerBlock, tb = min(a.nt, ta + kFskPerBlock);
    const bool two = sl + 1 < a.ns;                     // uniform
    const float2* X = a.X + size_t(a.s0 + sl) * size_t(a.M) + ip;
    const size_t second = two ? size_t(a.M) : 0;
    float2 z[2][P], w[P];
#pragma unroll
    for (int q = 0; q < P; ++q) {
        z[0][q] = X[q * a.Msub];
        z[1][q] = X[second + q * a.Msub];
    }
    phase_twiddles<P>(a, ip, w);
    for (int t = ta; t < tb; ++t) {
        const float2* B = a.bank + size_t(a.t0 + t) * size_t(a.M) + ip;
        float2* G = a.G + (size_t(t) * size_t(a.ns) + size_t(sl)) * size_t(a.M) + ip;
        float2 b[P];
#pragma unroll
        for (int q = 0; q < P; ++q) b[q] = B[q * a.Msub];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            if (h && !two) break;
            float2 y[P];
#pragma unroll
            for (int q = 0; q < P; ++q) y[q] = cmul(z[h][q], b[q]);
            dft_p<P, +1>(y);
            G[h * a.M] = y[0];
#pragma unroll
            for (int r = 1; r < P; ++r) G[h * a.M + r * a.Msub] = cmul(y[r], w[r]);
        }
    }
}

// First step of tracking slots, P > 1: combines the slot's decimated transforms
// at i' (and at -i' for two templates) in the same pass, as each slot has one
// item only.
template <int P>
__global__ __launch_bounds__(256, 2) void k_fsk_first_track(FskCorrArgs a) {
    const int nib = a.Msub / 256;
    const int ip = (int(blockIdx.x) % nib) * 256 + int(threadIdx.x);
    const int sl = int(blockIdx.x) / nib;
    const int tga = a.units[2 * (a.s0 + sl)].tag, tgb = a.units[2 * (a.s0 + sl) + 1].tag;
    const float2* F = a.X + size_t(a.s0 + sl) * size_t(a.M);
    const float2* Ba = a.bank + size_t(tga) * size_t(a.M) + ip;
    const float2* Bb = a.bank + size_t(tgb) * size_t(a.M) + ip;
    // Z[i + Msub q], q < P, from the decimated transforms F_r[i]
    auto combine = [&](int i, const float2 (&w)[P], float2 (&z)[P]) {
#pragma unroll
        for (int r = 0; r < P; ++r) z[r] = F[r * a.Msub + i];
#pragma unroll
        for (int r = 1; r < P; ++r) z[r] = cmulc(z[r], w[r]);
        dft_p<P, -1>(z);
    };
    float2 w[P], z[P], y[P];
    phase_twiddles<P>(a, ip, w);
    combine(ip, w, z);
    if (tga == tgb) {                                   // uniform
#pragma unroll
        for (int q = 0; q < P; ++q) y[q] = cmul(z[q], Ba[q * a.Msub]);
    } else {
        // conj Z[-i] for i = i' + Msub q: element P - 1 - q of Msub - i' (element -q of 0 for i' = 0)
        const int im = (a.Msub - ip) & (a.Msub - 1);
        float2 wm[P], zm[P];
        phase_twiddles<P>(a, im, wm);
        combine(im, wm, zm);
#pragma unroll
        for (int q = 0; q < P; ++q) {
            const float2 ba = Ba[q * a.Msub], bb = Bb[q * a.Msub];
            const float2 m0 = zm[(P - q) % P], m1 = zm[P - 1 - q];
            const float2 m = make_float2(ip ? m1.x : m0.x, ip ? -m1.y : -m0.y);
            const float2 r = cadd(cmul(z[q], cadd(ba, bb)), cmul(m, dev::csub(ba, bb)));
            y[q] = make_float2(0.5f * r.x, 0.5f * r.y);
        }
    }
    dft_p<P, +1>(y);
    float2* G = a.G + size_t(sl) * size_t(a.M) + ip;
    G[0] = y[0];
#pragma unroll
    for (int r = 1; r < P; ++r) G[r * a.Msub] = cmul(y[r], w[r]);
}

// Largest |c| of a segment over the wave's outputs against the workgroup's key
// so far (LDS): c = the real (H = 0) or imaginary part of v.  A wave that stays
// below the key forms none, and most do: those that come late see what the
// earlier ones reached.
template <class E, int H>
__device__ __forceinline__ void fsk_segment_peak(const float2 (&v)[16], int omin, int omax, int ob, int ulim, unsigned lag0,
                                                 unsigned step, unsigned long long* best) {
    int lim = ulim - ob;                              // this lane's outputs below this offset are valid lags
    asm volatile("" : "+v"(lim));
    float bp = -1.0f;
    auto mag = [&](int r) { return fabsf(H ? v[r].y : v[r].x); };
    // four registers at a time, in increasing offset: wave-uniform branches for
    // groups without a valid output and for groups without an invalid one
#pragma unroll
    for (int g = 0; g < 16; g += 4) {
        if (omin + E::out_off(E::visit(g)) >= ulim) break;
        if (omax + E::out_off(E::visit(g + 3)) < ulim) {
            asm volatile("" : "+v"(bp));              // (kept a branch: three instructions)
            bp = fmaxf(fmaxf(bp, mag(E::visit(g))), mag(E::visit(g + 1)));
            bp = fmaxf(fmaxf(bp, mag(E::visit(g + 2))), mag(E::visit(g + 3)));
        } else {
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const int r = E::visit(g + k);
                bp = fmaxf(bp, E::out_off(r) < lim ? mag(r) : -1.0f);
            }
        }
    }
    const unsigned long long sofar = __hip_atomic_load(best, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    if (__builtin_amdgcn_ballot_w64(bp >= __uint_as_float(unsigned(sofar >> 32)))) {
        const float wm = wave_fmax(bp);
        int boff = 0;                                 // smallest offset that holds wm
#pragma unroll
        for (int rr = 15; rr >= 0; --rr) {
            const int r = E::visit(rr), off = E::out_off(r);
            boff = off < lim && fabsf(H ? v[r].y : v[r].x) == wm ? off : boff;
        }
        const unsigned long long k = wave_key(bp, wm, lag0 + unsigned(ob + boff) * step);
        if ((threadIdx.x & 63) == 0) atomicMax(best, k);
    }
}

// Phase transforms: work item (item, rho), the Msub-point inverse transform of
// G_rho of the item (P = 1: of the spectrum product, formed here), whose output
// u is lag P u + rho of the slot's two segments.  One workgroup per CU (the
// transform's LDS) runs through a contiguous range of work items, loading the
// next one's input during the transform and keeping the largest key in LDS
// until the result it belongs to changes: an atomic of every work item on its
// template's key was waited for, 14.5 us a work item against 8.
template <class E, int P, bool DUMP>
__global__ __launch_bounds__(E::NT, 4) void k_fsk_phase(FskCorrArgs a) {
    __shared__ float2 lds[E::LDS];
    __shared__ float2 extra[E::EXTRA];
    __shared__ unsigned long long best[2][2];         // [buffer][segment, when they have different results]
    E eng;
    eng.init(a.rootsSub, extra);
    const __amdgpu_buffer_rsrc_t b1 = make_rsrc(a.b1tab, E::B1_TABLE * 8);
    const int64_t items = int64_t(a.track ? a.ns : a.nt * a.ns) * P;
    const int w0 = int(items * blockIdx.x / gridDim.x), w1 = int(items * (blockIdx.x + 1) / gridDim.x);
    if (threadIdx.x < 4) best[threadIdx.x >> 1][threadIdx.x & 1] = 0ull;
    const int voff = eng.in_index(0) * 8;
    // input of work item wi, P > 1
    auto fetch = [&](int wi, float2 (&x)[16]) {
        const __amdgpu_buffer_rsrc_t gr = make_rsrc(a.G + size_t(wi) * size_t(E::N), uint32_t(E::N) * 8u);
#pragma unroll
        for (int m = 0; m < 16; ++m) x[m] = bload(gr, voff, m * E::NT * 8);
    };
    // write a buffer's keys and clear it (every wave is past its last update)
    auto flush = [&](unsigned long long (&b)[2], int ka, int kb) {
        if (threadIdx.x == 0) {
            if (b[0]) atomicMax(&a.keys[ka], b[0]);
            if (b[1]) atomicMax(&a.keys[kb], b[1]);
            b[0] = b[1] = 0ull;
        }
    };
    float2 v[16];
    if constexpr (P > 1) fetch(w0, v);                // the grid is at most the work items: w0 < w1
    int ka = -1, kb = -1, par = 0;                    // results of the keys in best[par]
    for (int wi = w0; wi < w1; ++wi) {
        const int it = wi / P, rho = wi % P;
        const int slot = a.s0 + (a.track ? it : it % a.ns);
        const int t = a.track ? 0 : a.t0 + it / a.ns;
        const FskUnit ua = a.units[2 * slot], ub = a.units[2 * slot + 1];
        const int na = a.track ? ua.key : t, nb = a.track ? ub.key : t;
        const int oa = ka, ob_ = kb;
        const bool change = na != ka || nb != kb;     // uniform
        if (change) {
            ka = na;
            kb = nb;
            par ^= 1;
        }
        if constexpr (P == 1) {
            const float2* Z = a.X + size_t(slot) * size_t(E::N);
            const float2* Ba = a.bank + size_t(a.track ? ua.tag : t) * size_t(E::N);
            const float2* Bb = a.bank + size_t(a.track ? ub.tag : t) * size_t(E::N);
            if (Ba == Bb) {                           // uniform
#pragma unroll
                for (int m = 0; m < 16; ++m) v[m] = cmul(Z[eng.in_index(m)], Ba[eng.in_index(m)]);
            } else {
#pragma unroll
                for (int m = 0; m < 16; ++m) {
                    const int i = eng.in_index(m);
                    const float2 zm = Z[(E::N - i) & (E::N - 1)], ba = Ba[i], bb = Bb[i];
                    const float2 r = cadd(cmul(Z[i], cadd(ba, bb)), cmul(make_float2(zm.x, -zm.y), dev::csub(ba, bb)));
                    v[m] = make_float2(0.5f * r.x, 0.5f * r.y);
                }
            }
        }
        const int ula = ua.vlim > rho ? (ua.vlim - rho + P - 1) / P : 0;
        const int ulb = ub.vlim > rho ? (ub.vlim - rho + P - 1) / P : 0;
        const int omin = eng.out_min();
        const bool hi = omin + E::HI_OFF < max(ula, ulb);
        float2 next[16];
        dft16_first(v);
        eng.template transform_rest<+1>(v, lds, b1, extra, hi, [&] {
            if constexpr (P > 1) fetch(wi + 1 < w1 ? wi + 1 : wi, next);
        });
        if (change && oa >= 0) flush(best[par ^ 1], oa, ob_);
        const int ob = eng.out_base();
        if constexpr (DUMP) {
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int u = ob + E::out_off(r);
                if (u < ula) a.dump[size_t(t) * size_t(a.lags) + size_t(ua.lag0) + size_t(P) * u + rho] = v[r].x;
                if (u < ulb) a.dump[size_t(t) * size_t(a.lags) + size_t(ub.lag0) + size_t(P) * u + rho] = v[r].y;
            }
        }
        fsk_segment_peak<E, 0>(v, omin, eng.out_max(), ob, ula, ua.lag0 + unsigned(rho), unsigned(P), &best[par][0]);
        fsk_segment_peak<E, 1>(v, omin, eng.out_max(), ob, ulb, ub.lag0 + unsigned(rho), unsigned(P), &best[par][na == nb ? 0 : 1]);
        if constexpr (P > 1) {
#pragma unroll
            for (int m = 0; m < 16; ++m) v[m] = next[m];
        }
    }
    __syncthreads();
    flush(best[par], ka, kb);
}

// Results: searching, one item per template of the window; tracking, one item
// per task (its template).
struct FskRefineArgs {
    const float* d;             // the blocks' d (each at its zoff)
    const float* u;
    const float* tmpl;          // [T][tstride] d^(c), zero beyond n_t
    const unsigned long long* keys;     // [items]
    double* partial;            // [items][kFskParts][kFskSums]
    acq_fsk_detection* dets;    // [items]
    int32_t* found;             // [items]
    unsigned* tickets;          // [1 + items] arrivals, zero before and after each call
    acq_fsk_detection* h_out;   // host results of a call of at most kTailItems items, else nullptr
    int32_t* h_count;
    FskTasks tasks;
    int64_t nt, tstride;
    double theta;
};

struct FskItem {
    int tag, block;
    FskTask tk;
};

__device__ __forceinline__ FskItem fsk_item(const FskRefineArgs& a, int item) {
    FskItem r;
    r.block = a.tasks.track ? item : 0;
    r.tk = a.tasks.t[r.block];
    r.tag = a.tasks.track ? r.tk.tag : item;
    return r;
}

// FP64 sums over lags tau*-3 .. tau*+3 around the peak key: w_c, p_c and q at
// each lag and E_c, enough for the re-maximisation over +/-1 and one
// re-centring.  Each (item, part) workgroup sums a fixed chunk of the template
// in a fixed order and the last of an item's to arrive adds the parts in order:
// deterministic.  It writes the item's result, and the last item of a call of at
// most kTailItems the results to the host.
// A thread takes 4 template samples at a time, whose 7 lags use 10 block samples
// (from LDS, in three 16-byte reads of d and of u), and a chunk's loads are all
// in flight before the first is waited for.  (One sample at a time, its loads
// waited for in turn, 47 us for 128 templates of 65,736 samples, with launches for
// the results, their order and two copies after it; 33 us now, the search 444 ->
// 409 us, 64 tracking tasks 263 -> 230 us.)
constexpr int kFskWin = 7;
constexpr int kFskParts = 16;
constexpr int kFskSums = 3 * kFskWin + 1;
constexpr int kFskChunk = 3072;     // template samples of a part staged in LDS at a time, at most

__device__ __forceinline__ void fsk_result(const FskRefineArgs& a, const FskItem& fi, int item, int64_t lam0,
                                           const double* S, const double* A) {
    const int64_t lags = fi.tk.lags;
    const double Ec = S[3 * kFskWin];
    int c = kFskWin / 2;
    bool hit = false;
    for (int pass = 0; pass < 2; ++pass) {
        int wb = c;
        for (int w = c - 1; w <= c + 1; ++w)
            if (A[w] > A[wb] || (A[w] == A[wb] && w < wb)) wb = w;
        const int64_t lam = lam0 + wb;
        hit = (wb == c - 1 && lam > 0) || (wb == c + 1 && lam < lags - 1);
        c = wb;
        if (!hit) break;
    }
    const int64_t lam = lam0 + c;
    unsigned flags = hit ? ACQ_DET_WINDOW_EDGE : 0u;
    const double p0 = A[c];
    const double pm = A[c - 1] < 0.0 ? 0.0 : A[c - 1];
    const double pp = A[c + 1] < 0.0 ? 0.0 : A[c + 1];
    double delta = 0.0;
    if (lam == 0 || lam == lags - 1) {
        flags |= ACQ_DET_NEAR_EDGE;
    } else {
        const double den = pm - 2.0 * p0 + pp;
        if (den < 0.0) {
            delta = 0.5 * (pm - pp) / den;
            delta = delta > 0.5 ? 0.5 : (delta < -0.5 ? -0.5 : delta);
        }
    }
    acq_fsk_detection r;
    r.tag = fi.tag;
    r.block = fi.block;
    r.reserved = 0;
    r.flags = flags;
    r.lag = lam;
    r.toa_samples = double(lam) + delta;
    r.xcorr = S[3 * c];
    r.p = S[3 * c + 1];
    r.q = S[3 * c + 2];
    r.z = (r.q > 0.0 && Ec > 0.0) ? r.xcorr * r.xcorr / (r.q * Ec) : 0.0;
    agent_store_record(&a.dets[item], r);
    agent_store(&a.found[item], (a.theta <= 0.0 || r.z >= a.theta) ? 1 : 0);
}

__global__ __launch_bounds__(256, 4) void k_fsk_refine(FskRefineArgs a) {
    constexpr int NT = 256, NW = NT / 64;
    constexpr int G = kFskChunk / (4 * NT);          // groups of 4 samples per thread and chunk
    constexpr int S = (kFskChunk + 8 + NT - 1) / NT; // staged samples per thread
    __shared__ __align__(16) float s_d[S * NT], s_u[S * NT];
    __shared__ double red[NW][kFskSums];
    __shared__ double sums[kFskSums], amp[kFskWin];
    const int item = int(blockIdx.x) / kFskParts, part = int(blockIdx.x) % kFskParts;
    const int items = int(gridDim.x) / kFskParts;
    const FskItem fi = fsk_item(a, item);
    const int t = int(threadIdx.x), lane = t & 63, wave = t >> 6;
    const unsigned long long key = fi.tk.lags > 0 ? a.keys[item] : 0ull;
    if (key != 0ull) {
        const int64_t lam0 = int64_t(~unsigned(key & 0xffffffffull)) - kFskWin / 2;
        const float* dc = a.tmpl + size_t(fi.tag) * size_t(a.tstride);
        const int64_t ch = ((a.nt + kFskParts - 1) / kFskParts + 3) / 4 * 4;     // whole groups
        const int64_t i0 = min(a.nt, int64_t(part) * ch), i1 = min(a.nt, i0 + ch);
        double wv[kFskWin], pv[kFskWin], qv[kFskWin], ec = 0.0;
#pragma unroll
        for (int w = 0; w < kFskWin; ++w) wv[w] = pv[w] = qv[w] = 0.0;
        const int64_t nch = (ch + kFskChunk - 1) / kFskChunk, cl = (ch + 4 * nch - 1) / (4 * nch) * 4;  // even chunks
        for (int64_t c0 = i0; c0 < i1; c0 += cl) {
            const int len = int(min(i1 - c0, cl));
            float4 cs[G];                            // (the template's rows end in whole groups)
#pragma unroll
            for (int g = 0; g < G; ++g)
                cs[g] = *reinterpret_cast<const float4*>(dc + c0 + min(4 * (t + NT * g), (len - 1) / 4 * 4));
            // block samples from k0 on, by buffer loads bounded by the block: zero
            // outside it (positions before its start at offset -1, as in k_fsk_front)
            const int64_t k0 = lam0 + c0, first = k0 > 0 ? k0 : 0;
            const int64_t left = min(fi.tk.n - first, int64_t(S * NT));
            const uint32_t bytes = left > 0 ? uint32_t(left) * 4u : 0u;
            const __amdgpu_buffer_rsrc_t dr = make_rsrc(a.d + fi.tk.zoff + first, bytes);
            const __amdgpu_buffer_rsrc_t ur = make_rsrc(a.u + fi.tk.zoff + first, bytes);
            const int q0 = int(k0 - first) + t;
            float sd[S], su[S];
#pragma unroll
            for (int q = 0; q < S; ++q) {
                const int at = max(q0 + NT * q, -1) * 4;
                sd[q] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(dr, at, 0, 0));
                su[q] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(ur, at, 0, 0));
            }
            if (c0 != i0) __syncthreads();           // the chunk before has been read
#pragma unroll
            for (int q = 0; q < S; ++q) {
                s_d[t + NT * q] = sd[q];
                s_u[t + NT * q] = su[q];
            }
            __syncthreads();
#pragma unroll
            for (int g = 0; g < G; ++g) {
                const int o = 4 * (t + NT * g);
                if (o >= len) break;
                double zd[12], zu[12];
#pragma unroll
                for (int q = 0; q < 3; ++q) {
                    const float4 vd = *reinterpret_cast<const float4*>(&s_d[o + 4 * q]);
                    const float4 vu = *reinterpret_cast<const float4*>(&s_u[o + 4 * q]);
                    zd[4 * q] = vd.x; zd[4 * q + 1] = vd.y; zd[4 * q + 2] = vd.z; zd[4 * q + 3] = vd.w;
                    zu[4 * q] = vu.x; zu[4 * q + 1] = vu.y; zu[4 * q + 2] = vu.z; zu[4 * q + 3] = vu.w;
                }
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    if (o + e >= len) break;
                    const double c = e == 0 ? cs[g].x : e == 1 ? cs[g].y : e == 2 ? cs[g].z : cs[g].w;
                    ec += c * c;
#pragma unroll
                    for (int w = 0; w < kFskWin; ++w) {
                        wv[w] += c * zd[e + w];
                        pv[w] += c * zu[e + w];
                        qv[w] += zd[e + w] * zd[e + w];
                    }
                }
            }
        }
#pragma unroll
        for (int w = 0; w < kFskWin; ++w) {
            const double r0 = wave_sum(wv[w]), r1 = wave_sum(pv[w]), r2 = wave_sum(qv[w]);
            if (lane == 0) {
                red[wave][3 * w] = r0;
                red[wave][3 * w + 1] = r1;
                red[wave][3 * w + 2] = r2;
            }
        }
        const double es = wave_sum(ec);
        if (lane == 0) red[wave][3 * kFskWin] = es;
        __syncthreads();
        if (t < kFskSums) {
            double v = 0.0;
            for (int q = 0; q < NW; ++q) v += red[q][t];
            agent_store(&a.partial[(size_t(item) * kFskParts + part) * kFskSums + t], v);
        }
        if (!last_arrival(&a.tickets[1 + item], kFskParts)) return;
        if (t < kFskSums) {
            double q[kFskParts], v = 0.0;
#pragma unroll
            for (int p = 0; p < kFskParts; ++p) q[p] = agent_load(&a.partial[(size_t(item) * kFskParts + p) * kFskSums + t]);
#pragma unroll
            for (int p = 0; p < kFskParts; ++p) v += q[p];
            sums[t] = v;
        }
        __syncthreads();
        if (t < kFskWin) {
            const int64_t lam = lam0 + t;
            amp[t] = (lam >= 0 && lam < fi.tk.lags) ? fabs(sums[3 * t]) : -1.0;
        }
        __syncthreads();
        if (t == 0) fsk_result(a, fi, item, lam0, sums, amp);
    } else {
        if (part != 0) return;
        if (t == 0) agent_store(&a.found[item], 0);
    }
    if (!a.h_out || !last_arrival(&a.tickets[0], unsigned(items))) return;
    auto slot = [&](int e) { return agent_load(&a.found[e]) ? e : -1; };
    const int n = compact_records<NT, kTailItems, acq_fsk_detection>(items, a.dets, slot, items, nullptr, a.h_out);
    if (t == 0) *a.h_count = n;
}

// Results in tag order: one workgroup of 1024 threads, runs of tags per
// thread, a scan of the counts gives each run's output offset.
__global__ __launch_bounds__(1024) void k_fsk_compact(const acq_fsk_detection* __restrict__ dets,
                                                      const int32_t* __restrict__ found, int T,
                                                      acq_fsk_detection* __restrict__ out,
                                                      int32_t* __restrict__ count) {
    __shared__ int scan[1024];
    const int t = int(threadIdx.x);
    const int per = (T + 1023) / 1024;
    const int b0 = min(T, t * per), b1 = min(T, b0 + per);
    int c = 0;
    for (int i = b0; i < b1; ++i) c += found[i] ? 1 : 0;
    scan[t] = c;
    __syncthreads();
    for (int off = 1; off < 1024; off <<= 1) {
        const int v = t >= off ? scan[t - off] : 0;
        __syncthreads();
        scan[t] += v;
        __syncthreads();
    }
    int o = scan[t] - c;
    for (int i = b0; i < b1; ++i)
        if (found[i]) out[o++] = dets[i];
    if (t == 1023) *count = scan[t];
}

template <class E, int P>
void launch_fsk_ep(const FskCorrArgs& a, hipStream_t st) {
    const int items = a.track ? a.ns : a.nt * a.ns;
    if constexpr (P > 1) {
        const unsigned nib = unsigned(a.Msub / 256);
        if (a.track)
            hipLaunchKernelGGL((k_fsk_first_track<P>), dim3(nib * unsigned(a.ns)), dim3(256), 0, st, a);
        else
            hipLaunchKernelGGL((k_fsk_first<P>),
                               dim3(nib * unsigned((a.ns + 1) / 2) * unsigned((a.nt + kFskPerBlock - 1) / kFskPerBlock)), dim3(256),
                               0, st, a);
    }
    // P = 1: as many workgroups as items (nothing to load ahead)
    const dim3 grid(unsigned(P > 1 ? std::min(items * P, kFskPhaseGrid) : items));
    if (a.dump)
        hipLaunchKernelGGL((k_fsk_phase<E, P, true>), grid, dim3(E::NT), 0, st, a);
    else
        hipLaunchKernelGGL((k_fsk_phase<E, P, false>), grid, dim3(E::NT), 0, st, a);
}

// M <= 2^14 runs as one phase (P = 1) on the engine of that size; larger M as
// P = M / 2^14 phases on the 2^14-point engine.
hipError_t launch_fsk_correlate(const FskCorrArgs& a, int log2_sub, hipStream_t st) {
    if (a.ns <= 0 || (!a.track && a.nt <= 0)) return hipSuccess;
    if ((log2_sub < 14 && a.P != 1) || (1 << log2_sub) != a.Msub || a.M != a.P * a.Msub) return hipErrorInvalidValue;
    switch (log2_sub) {
        case 10: launch_fsk_ep<StockhamEngine<10>, 1>(a, st); break;
        case 11: launch_fsk_ep<StockhamEngine<11>, 1>(a, st); break;
        case 12: launch_fsk_ep<StockhamEngine<12>, 1>(a, st); break;
        case 13: launch_fsk_ep<StockhamEngine<13>, 1>(a, st); break;
        case 14:
            switch (a.P) {
                case 1: launch_fsk_ep<Fft14, 1>(a, st); break;
                case 2: launch_fsk_ep<Fft14, 2>(a, st); break;
                case 4: launch_fsk_ep<Fft14, 4>(a, st); break;
                case 8: launch_fsk_ep<Fft14, 8>(a, st); break;
                case 16: launch_fsk_ep<Fft14, 16>(a, st); break;
                default: return hipErrorInvalidValue;
            }
            break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

template <class E>
void launch_fsk_forward_e(const FskUnit* units, const float* d, int P, int M, int slots, const float2* rootsSub,
                          const float2* b1tab, float2* X, hipStream_t st) {
    hipLaunchKernelGGL((k_fsk_forward<E>), dim3(unsigned(slots * P)), dim3(E::NT), 0, st, units, d, P, M, slots * P,
                       rootsSub, b1tab, X);
}

hipError_t launch_fsk_forward(const FskUnit* units, const float* d, int P, int M, int log2_sub, int slots,
                              const float2* rootsSub, const float2* b1tab, float2* X, hipStream_t st) {
    if (slots <= 0) return hipSuccess;
    if (M != P << log2_sub) return hipErrorInvalidValue;
    switch (log2_sub) {
        case 10: launch_fsk_forward_e<StockhamEngine<10>>(units, d, P, M, slots, rootsSub, b1tab, X, st); break;
        case 11: launch_fsk_forward_e<StockhamEngine<11>>(units, d, P, M, slots, rootsSub, b1tab, X, st); break;
        case 12: launch_fsk_forward_e<StockhamEngine<12>>(units, d, P, M, slots, rootsSub, b1tab, X, st); break;
        case 13: launch_fsk_forward_e<StockhamEngine<13>>(units, d, P, M, slots, rootsSub, b1tab, X, st); break;
        case 14: launch_fsk_forward_e<Fft14>(units, d, P, M, slots, rootsSub, b1tab, X, st); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

// ------------------------------------------------------------------ host side
struct FskGeometry {
    int64_t lg = 0, nt = 0, M = 0, Msub = 0, V = 0, vf = 0, max_seg = 0, max_front_seg = 0, bytes = 0;
    int64_t slots = 0;          // packed segment pairs a call may use
    int64_t group = 0;          // first-step outputs held at a time (complex values, a multiple of M; 0: P = 1)
    int P = 1, log2_sub = 0;
    int max_tasks = 16;         // tracking tasks per call
    int items = 0;              // results per call: max(templates, tasks)
};

int fsk_geometry(const acq_fsk_config* c, FskGeometry* g) {
    if (!c) return fail(ACQ_ERR_INVALID_ARG, "null configuration");
    if (!(c->sample_rate_hz > 0.0) || !std::isfinite(c->lo_hz) || !std::isfinite(c->f1_hz) ||
        !std::isfinite(c->f0_hz) || !std::isfinite(c->threshold))
        return fail(ACQ_ERR_INVALID_ARG, "sample rate must be positive and frequencies finite");
    if (!c->bp_taps || !c->bits) return fail(ACQ_ERR_INVALID_ARG, "null taps or bits");
    if (c->bp_len < 1 || c->bp_len > 1024) return fail(ACQ_ERR_INVALID_ARG, "bp_len outside [1, 1024]");
    if (c->mf_len < 1 || c->mf_len > 64) return fail(ACQ_ERR_INVALID_ARG, "mf_len outside [1, 64]");
    if (c->num_tags < 1 || c->num_bits < 1) return fail(ACQ_ERR_INVALID_ARG, "num_tags and num_bits must be >= 1");
    if (c->max_block_len < 1) return fail(ACQ_ERR_INVALID_ARG, "max_block_len must be >= 1");
    g->lg = int64_t(c->bp_len) + c->mf_len - 1;
    g->nt = int64_t(c->num_bits) * c->mf_len + g->lg - 1;
    g->vf = kFrontN - g->lg + 1;
    constexpr int64_t kMaxM = int64_t(1) << 18;
    int64_t M = c->fft_len;
    if (M == 0) {
        M = 1024;
        while (M <= g->nt && M < kMaxM) M <<= 1;      // smallest power of two > n_t ...
        if (M < kMaxM && M - g->nt + 1 < g->nt / 2) M <<= 1;   // ... doubled when few lags remain
        // ... or, from 2^17 (templates of the paper's length), doubled when
        // that needs fewer transform points for the plan's blocks: one window
        // of max_block_len samples, or, when the plan is sized for tracking
        // tasks, max_track_tasks blocks of equal length
        if (M >= (int64_t(1) << 17) && M > g->nt && 2 * M <= kMaxM) {
            const int64_t tasks = c->max_track_tasks > 0 ? c->max_track_tasks : 1;
            const int64_t len = (c->max_block_len + tasks - 1) / tasks;
            auto points = [&](int64_t m) {
                const int64_t lags = std::max<int64_t>(len - g->nt + 1, 1), v = m - g->nt + 1;
                return tasks * ((lags + v - 1) / v + 1) / 2 * m;       // segments two to a transform
            };
            if (points(2 * M) < points(M)) M *= 2;
        }
    }
    if (M < 1024 || M > kMaxM || (M & (M - 1)))
        return fail(ACQ_ERR_UNSUPPORTED, "fft_len must be a power of two in [2^10, 2^18]");
    if (M <= g->nt) return fail(ACQ_ERR_UNSUPPORTED, "template longer than the correlation segment (at most 2^18 - 1)");
    g->M = M;
    g->Msub = std::min<int64_t>(M, int64_t(1) << 14);
    g->P = int(M / g->Msub);
    g->log2_sub = 0;
    while ((int64_t(1) << g->log2_sub) < g->Msub) ++g->log2_sub;
    g->V = M - g->nt + 1;
    const int64_t lags = c->max_block_len - g->nt + 1;
    g->max_seg = lags > 0 ? (lags + g->V - 1) / g->V : 0;
    g->max_front_seg = (c->max_block_len + g->vf - 1) / g->vf;
    if (c->max_track_tasks < 0 || c->max_track_tasks > 65536)
        return fail(ACQ_ERR_INVALID_ARG, "max_track_tasks outside [0, 65536]");
    g->max_tasks = c->max_track_tasks > 0 ? c->max_track_tasks : 16;
    // a searching window uses ceil(max_seg / 2) slots; tracking blocks of total
    // length <= max_block_len have at most max_block_len / V + one segment per
    // task, two to a slot (the bound below keeps room for one slot per task)
    g->slots = (g->max_seg + 1) / 2 + g->max_tasks + 1;
    g->items = std::max<int>(c->num_tags, g->max_tasks);
    const int64_t T = c->num_tags;
    const int64_t slots = g->slots;
    // every item of a call, (template, slot) or tracking slot, or a group of them
    g->group = g->P > 1 ? std::min<int64_t>(std::max<int64_t>(T * ((g->max_seg + 1) / 2), slots),
                                            std::max<int64_t>(1, kFskGroup / M)) * M : 0;
    g->bytes = c->max_block_len * 8 + slots * M * 8 + g->group * 8 + slots * 2 * int64_t(sizeof(FskUnit)) +
               T * M * 8 + T * (g->nt + 4) * 4 + T * c->num_bits * 9 + int64_t(g->items) * (kFskParts * kFskSums * 8 + 64) +
               kFrontN * 8 * 2 + transform_roots_len(kFrontN) * 8 + M * 8 * (g->P > 2 && g->P <= 8 ? 2 : 1) + transform_roots_len(g->Msub) * 8 + T * (8 + 4 + 2 * int64_t(sizeof(acq_fsk_detection)));
    return ACQ_OK;
}

// composed filter h_BP * h_b, FP64
std::vector<double> composed(const acq_fsk_config* c, double f_hz) {
    const int lb = c->bp_len, lm = c->mf_len;
    std::vector<double> g(size_t(2 * (lb + lm - 1)), 0.0);
    const double two_pi = 6.283185307179586476925286766559;
    for (int k = 0; k < lm; ++k) {
        // h_b[k] = exp(-j 2 pi f (lm-1-k) / Fs), phase reduced in cycles
        double cyc = -f_hz * double(lm - 1 - k) / c->sample_rate_hz;
        cyc -= std::floor(cyc);
        const double hr = std::cos(two_pi * cyc), hi = std::sin(two_pi * cyc);
        for (int i = 0; i < lb; ++i) {
            const double br = c->bp_taps[2 * i], bi = c->bp_taps[2 * i + 1];
            g[size_t(2 * (i + k))] += br * hr - bi * hi;
            g[size_t(2 * (i + k) + 1)] += br * hi + bi * hr;
        }
    }
    return g;
}

// DFT_kFrontN(g) / kFrontN in FP64 (direct sum, exact index reduction), as FP32 pairs
std::vector<float> filter_spectrum(const std::vector<double>& g) {
    const int64_t lg = int64_t(g.size() / 2);
    const std::vector<double> roots = unit_roots64(kFrontN);        // (cos, sin)(2 pi m / N)
    std::vector<float> out(size_t(2 * kFrontN));
    for (int64_t k = 0; k < kFrontN; ++k) {
        double re = 0.0, im = 0.0;
        for (int64_t i = 0; i < lg; ++i) {
            const int64_t e = (i * k) % kFrontN;
            const double cr = roots[size_t(2 * e)], ci = -roots[size_t(2 * e + 1)];   // exp(-j 2 pi i k / N)
            re += g[size_t(2 * i)] * cr - g[size_t(2 * i + 1)] * ci;
            im += g[size_t(2 * i)] * ci + g[size_t(2 * i + 1)] * cr;
        }
        out[size_t(2 * k)] = float(re / kFrontN);
        out[size_t(2 * k + 1)] = float(im / kFrontN);
    }
    return out;
}

}  // namespace
}  // namespace acq

using acq::BlockDesc;
using acq::BlockTable;

struct acq_fsk_plan_s {
    acq_fsk_config cfg{};
    acq::FskGeometry g;
    hipStream_t stream = nullptr;
    float2* d_G1 = nullptr;             // [kFrontN]
    float2* d_G0 = nullptr;
    float2* d_rootsF = nullptr;         // unit roots and pass twiddles of the front end's transform
    uint8_t* d_bits = nullptr;          // [T][nbits]
    double* d_bitcyc = nullptr;         // [T][nbits]
    float* d_tmpl = nullptr;            // [T][tstride] d^(c), zero beyond n_t
    int64_t tstride = 0;                // n_t in whole groups of 4
    float2* d_bank = nullptr;           // [T][M] conj(DFT_M(d^(c))) / M
    float* d_d = nullptr;               // [max_block_len] demodulated d
    float* d_u = nullptr;               // [max_block_len] u
    float2* d_X = nullptr;              // [slots][M] spectra of the packed segment pairs of d
    float2* d_G = nullptr;              // [group] first-step outputs of the correlation
    double* d_partial = nullptr;        // [T][parts][sums] refinement partial sums
    float2* d_rootsM = nullptr;
    float2* d_phases = nullptr;         // [P][Msub] phase twiddles (2 < P <= 8)
    float2* d_rootsSub = nullptr;
    float2* d_b1tab = nullptr;
    BlockDesc* d_tdescs = nullptr;      // [T] templates as blocks of the forward transform
    int32_t* d_tcounts = nullptr;       // [2]
    unsigned long long* d_keys = nullptr;
    acq_fsk_detection* d_dets = nullptr;
    acq_fsk_detection* d_out = nullptr;
    int32_t* d_found = nullptr;
    int32_t* d_count = nullptr;
    unsigned* d_tickets = nullptr;      // [1 + items] refinement arrivals
    acq::FskTask* d_tasks = nullptr;        // [max_tasks] blocks of a call, then (right after the call's
                                            // blocks) [2 slots] its correlation segments
    acq::FskTask* h_tasks = nullptr;        // pinned, the same
    acq_fsk_detection* h_out = nullptr;     // pinned [items]
    int32_t* h_count = nullptr;             // pinned [1]
    bool profiling = false;
    hipEvent_t ev[ACQ_FSK_NUM_KERNELS][2] = {};
};

namespace {

#define FSK_HIP(call)                                                                          \
    do {                                                                                       \
        hipError_t e_ = (call);                                                                \
        if (e_ != hipSuccess)                                                                  \
            return acq::fail(e_ == hipErrorOutOfMemory ? ACQ_ERR_OOM : ACQ_ERR_DEVICE,         \
                             std::string(#call) + ": " + hipGetErrorString(e_));               \
    } while (0)

template <typename T>
hipError_t dalloc(T** p, size_t count) {
    return hipMalloc(reinterpret_cast<void**>(p), sizeof(T) * (count ? count : 1));
}

// Event pair around one launch when profiling is on.
struct FskTimer {
    acq_fsk_plan_s* p;
    int id;
    FskTimer(acq_fsk_plan_s* plan, int kernel) : p(plan), id(kernel) {
        if (p->profiling) (void)hipEventRecord(p->ev[id][0], p->stream);
    }
    ~FskTimer() {
        if (p->profiling) (void)hipEventRecord(p->ev[id][1], p->stream);
    }
};

void free_fsk(acq_fsk_plan_s* p) {
    if (!p) return;
    for (auto& pair : p->ev)
        for (hipEvent_t e : pair)
            if (e) (void)hipEventDestroy(e);
    void* dev[] = {p->d_G1, p->d_G0, p->d_rootsF, p->d_bits, p->d_bitcyc, p->d_tmpl, p->d_bank, p->d_d, p->d_u, p->d_X, p->d_G, p->d_partial,
                   p->d_rootsM, p->d_phases, p->d_rootsSub, p->d_b1tab, p->d_tdescs, p->d_tcounts, p->d_keys,
                   p->d_dets, p->d_out, p->d_found, p->d_count, p->d_tickets};
    for (void* d : dev)
        if (d) (void)hipFree(d);
    if (p->h_out) (void)hipHostFree(p->h_out);
    if (p->h_tasks) (void)hipHostFree(p->h_tasks);
    if (p->d_tasks) (void)hipFree(p->d_tasks);
    if (p->h_count) (void)hipHostFree(p->h_count);
    delete p;
}

// Replica mode writes `out` ([T][M]); block mode processes the call's blocks
// (device task table, fsegs front-end segments in all) into the plan's d, u.
hipError_t launch_front(acq_fsk_plan_s* p, const acq::FskTasks& tasks, int fsegs, bool replica, float2* out,
                        int nkeys) {
    const acq_fsk_config& c = p->cfg;
    acq::FrontArgs a{};
    a.tasks = tasks;
    a.bits = p->d_bits;
    a.bit_cyc = p->d_bitcyc;
    a.G1 = p->d_G1;
    a.G0 = p->d_G0;
    a.roots = p->d_rootsF;
    a.out = out;
    a.out_d = p->d_d;
    a.out_u = p->d_u;
    a.keys = p->d_keys;
    a.nkeys = nkeys;
    a.n_in = int64_t(c.num_bits) * c.mf_len;
    a.n_out = p->g.nt;
    a.out_stride = p->g.M;
    a.lo_cyc = c.lo_hz / c.sample_rate_hz;
    {
        using E = acq::kdev::StockhamEngine<acq::kFrontLog, false>;
        for (int m = 0; m < 16; ++m) {
            double cyc = -a.lo_cyc * double(int64_t(E::NT) * m);
            cyc -= std::floor(cyc);
            a.lo_step[m] = make_float2(float(std::cos(2.0 * M_PI * cyc)), float(std::sin(2.0 * M_PI * cyc)));
        }
    }
    a.f1_cyc = c.f1_hz / c.sample_rate_hz;
    a.f0_cyc = c.f0_hz / c.sample_rate_hz;
    a.nbits = c.num_bits;
    a.sps = c.mf_len;
    a.lg = int(p->g.lg);
    a.vf = int(p->g.vf);
    a.nseg = int((a.n_out + p->g.vf - 1) / p->g.vf);
    const unsigned grid = replica ? unsigned(a.nseg) * unsigned(c.num_tags) : unsigned(fsegs);
    if (grid == 0) return hipSuccess;
    if (replica)
        hipLaunchKernelGGL(acq::k_fsk_front<true>, dim3(grid), dim3(256), 0, p->stream, a);
    else
        hipLaunchKernelGGL(acq::k_fsk_front<false>, dim3(grid), dim3(256), 0, p->stream, a);
    return hipGetLastError();
}

acq::FwdArgs fwd_args(acq_fsk_plan_s* p, const BlockTable& bt, float2* X, int64_t V) {
    acq::FwdArgs fa{};
    fa.blocks = bt;
    fa.X = X;
    fa.Xh = nullptr;
    fa.exps = nullptr;
    fa.cls_cyc = nullptr;            // no residual offsets
    fa.ncls = 1;
    fa.rootsM = p->d_rootsM;
    fa.rootsSub = p->d_rootsSub;
    fa.b1tab = p->d_b1tab;
    fa.V = V;
    fa.xstride = p->g.M;             // unpadded [slots][M]
    fa.xpad = 0;
    fa.spc = p->g.P;
    fa.M = int(p->g.M);
    fa.Msub = int(p->g.Msub);
    return fa;
}

int build_fsk(acq_fsk_plan_s* p, const acq_fsk_config* cfg) {
    const acq::FskGeometry& g = p->g;
    const acq_fsk_config& c = *cfg;
    const size_t T = size_t(c.num_tags), NB = size_t(c.num_bits), M = size_t(g.M);
    hipStream_t st = p->stream;
    FSK_HIP(dalloc(&p->d_G1, size_t(acq::kFrontN)));
    FSK_HIP(dalloc(&p->d_G0, size_t(acq::kFrontN)));
    FSK_HIP(dalloc(&p->d_rootsF, size_t(acq::transform_roots_len(acq::kFrontN))));
    FSK_HIP(dalloc(&p->d_bits, T * NB));
    FSK_HIP(dalloc(&p->d_bitcyc, T * NB));
    p->tstride = (g.nt + 3) / 4 * 4;
    FSK_HIP(dalloc(&p->d_tmpl, T * size_t(p->tstride)));
    float2* wave = nullptr;                         // [T][M] (d^(c), 0), zero beyond n_t, while the plan is made
    FSK_HIP(dalloc(&wave, T * M));
    struct WaveFree {
        float2* p;
        ~WaveFree() { (void)hipFree(p); }
    } wave_free{wave};
    FSK_HIP(dalloc(&p->d_bank, T * M));
    const size_t slots = size_t(g.slots);
    const size_t items = size_t(g.items);
    FSK_HIP(dalloc(&p->d_d, size_t(c.max_block_len)));
    FSK_HIP(dalloc(&p->d_u, size_t(c.max_block_len)));
    FSK_HIP(dalloc(&p->d_X, slots * M));
    FSK_HIP(dalloc(&p->d_G, size_t(g.group)));
    const size_t table_bytes = sizeof(acq::FskTask) * size_t(g.max_tasks) + sizeof(acq::FskUnit) * 2 * slots;
    FSK_HIP(hipMalloc(reinterpret_cast<void**>(&p->d_tasks), table_bytes));
    FSK_HIP(hipHostMalloc(reinterpret_cast<void**>(&p->h_tasks), table_bytes));
    FSK_HIP(dalloc(&p->d_rootsM, M));
    const bool phases = g.P > 2 && g.P <= 8;
    if (phases) FSK_HIP(dalloc(&p->d_phases, M));
    FSK_HIP(dalloc(&p->d_rootsSub, size_t(acq::transform_roots_len(g.Msub))));
    const std::vector<float> b1 = g.log2_sub == 14 ? acq::fft14_b1_table() : std::vector<float>(2, 0.f);
    FSK_HIP(dalloc(&p->d_b1tab, b1.size() / 2));
    FSK_HIP(dalloc(&p->d_tdescs, T));
    FSK_HIP(dalloc(&p->d_tcounts, 2));
    FSK_HIP(dalloc(&p->d_keys, items));
    FSK_HIP(dalloc(&p->d_partial, items * size_t(acq::kFskParts) * size_t(acq::kFskSums)));
    FSK_HIP(dalloc(&p->d_dets, items));
    FSK_HIP(dalloc(&p->d_out, items));
    FSK_HIP(dalloc(&p->d_found, items));
    FSK_HIP(dalloc(&p->d_count, 1));
    FSK_HIP(dalloc(&p->d_tickets, items + 1));
    FSK_HIP(acq::launch_fill_i32(reinterpret_cast<int*>(p->d_tickets), int64_t(items) + 1, p->stream));
    FSK_HIP(hipHostMalloc(reinterpret_cast<void**>(&p->h_out), sizeof(acq_fsk_detection) * items));
    FSK_HIP(hipHostMalloc(reinterpret_cast<void**>(&p->h_count), sizeof(int32_t)));

    // tables: composed filter spectra, unit roots, replica bit phases (FP64 on the host)
    const std::vector<float> G1 = acq::filter_spectrum(acq::composed(&c, c.f1_hz));
    const std::vector<float> G0 = acq::filter_spectrum(acq::composed(&c, c.f0_hz));
    const std::vector<float> rootsF = acq::transform_roots(acq::kFrontN);
    const std::vector<float> rootsM = acq::unit_roots(g.M);
    const std::vector<float> rootsSub = acq::transform_roots(g.Msub);
    std::vector<double> bitcyc(T * NB);
    std::vector<uint8_t> bits(T * NB);
    for (size_t t = 0; t < T; ++t) {
        long double acc = 0.0L;                   // cycles at the bit start, reduced as it grows
        for (size_t b = 0; b < NB; ++b) {
            const uint8_t bit = c.bits[t * NB + b] ? 1 : 0;
            bits[t * NB + b] = bit;
            bitcyc[t * NB + b] = double(acc);
            acc += (long double)(bit ? c.f1_hz : c.f0_hz) * (long double)c.mf_len / (long double)c.sample_rate_hz;
            acc -= std::floor(acc);
        }
    }
    FSK_HIP(hipMemcpyAsync(p->d_G1, G1.data(), G1.size() * sizeof(float), hipMemcpyHostToDevice, st));
    FSK_HIP(hipMemcpyAsync(p->d_G0, G0.data(), G0.size() * sizeof(float), hipMemcpyHostToDevice, st));
    FSK_HIP(hipMemcpyAsync(p->d_rootsF, rootsF.data(), rootsF.size() * sizeof(float), hipMemcpyHostToDevice, st));
    FSK_HIP(hipMemcpyAsync(p->d_rootsM, rootsM.data(), rootsM.size() * sizeof(float), hipMemcpyHostToDevice, st));
    if (phases) {
        hipLaunchKernelGGL(acq::k_fsk_phase_roots, dim3(unsigned(M / 256)), dim3(256), 0, st, p->d_rootsM, int(g.Msub),
                           p->d_phases);
        FSK_HIP(hipGetLastError());
    }
    FSK_HIP(hipMemcpyAsync(p->d_rootsSub, rootsSub.data(), rootsSub.size() * sizeof(float), hipMemcpyHostToDevice,
                           st));
    FSK_HIP(hipMemcpyAsync(p->d_b1tab, b1.data(), b1.size() * sizeof(float), hipMemcpyHostToDevice, st));
    FSK_HIP(hipMemcpyAsync(p->d_bits, bits.data(), bits.size(), hipMemcpyHostToDevice, st));
    FSK_HIP(hipMemcpyAsync(p->d_bitcyc, bitcyc.data(), bitcyc.size() * sizeof(double), hipMemcpyHostToDevice, st));

    // replica templates d^(c) (zero beyond n_t), then their spectra
    const int64_t tcount = int64_t(T * M);
    hipLaunchKernelGGL(acq::k_fsk_fill, dim3(unsigned((tcount + 255) / 256)), dim3(256), 0, st, wave, tcount);
    FSK_HIP(hipGetLastError());
    FSK_HIP(launch_front(p, acq::FskTasks{}, 0, true, wave, 0));
    std::vector<BlockDesc> descs(T);
    for (size_t t = 0; t < T; ++t) {
        BlockDesc d{};
        d.x = wave + t * M;
        d.n = g.nt;
        d.lags = 1;
        d.seg0 = int32_t(t);
        d.nseg = 1;
        d.tag = -1;
        descs[t] = d;
    }
    const int32_t counts[2] = {int32_t(T), int32_t(T)};
    FSK_HIP(hipMemcpyAsync(p->d_tdescs, descs.data(), T * sizeof(BlockDesc), hipMemcpyHostToDevice, st));
    FSK_HIP(hipMemcpyAsync(p->d_tcounts, counts, sizeof(counts), hipMemcpyHostToDevice, st));
    BlockTable bt{};
    bt.descs = p->d_tdescs;
    bt.counts = p->d_tcounts;
    const acq::FwdArgs fa = fwd_args(p, bt, p->d_bank, g.M);
    FSK_HIP(acq::launch_forward(fa, int(T) * g.P, int(T), 0, 0, g.log2_sub, ACQ_FP32, st));
    hipLaunchKernelGGL(acq::k_fsk_conj_scale, dim3(unsigned((tcount + 255) / 256)), dim3(256), 0, st, p->d_bank, tcount,
                       float(1.0 / double(g.M)));
    FSK_HIP(hipGetLastError());
    // the refinement reads d^(c) alone: half the bytes, 16 at a time
    hipLaunchKernelGGL(acq::k_fsk_real, dim3(unsigned((int64_t(T) * p->tstride + 255) / 256)), dim3(256), 0, st, wave,
                       int64_t(M), p->d_tmpl, p->tstride, int64_t(T) * p->tstride);
    FSK_HIP(hipGetLastError());
    FSK_HIP(hipStreamSynchronize(st));
    return ACQ_OK;
}

int check_iq(acq_fsk_plan_s* p, const int16_t* iq, int64_t n) {
    if (!p) return acq::fail(ACQ_ERR_INVALID_ARG, "null plan");
    if (n < 0) return acq::fail(ACQ_ERR_INVALID_ARG, "negative block length");
    if (n > p->cfg.max_block_len) return acq::fail(ACQ_ERR_BLOCK_TOO_LONG, "block longer than max_block_len");
    if (n > 0 && !iq) return acq::fail(ACQ_ERR_INVALID_ARG, "null block");
    if (reinterpret_cast<uintptr_t>(iq) % 4 != 0) return acq::fail(ACQ_ERR_INVALID_ARG, "block must be 4-byte aligned");
    return ACQ_OK;
}

}  // namespace

extern "C" {

int acq_fsk_plan_geometry(const acq_fsk_config* cfg, acq_fsk_geometry* out) {
    if (!out) return acq::fail(ACQ_ERR_INVALID_ARG, "null output");
    acq::FskGeometry g;
    const int rc = acq::fsk_geometry(cfg, &g);
    if (rc != ACQ_OK) return rc;
    out->template_len = g.nt;
    out->fft_len = g.M;
    out->valid_per_segment = g.V;
    out->filter_len = g.lg;
    out->front_fft_len = acq::kFrontN;
    out->device_bytes = g.bytes;
    acq::clear_error();
    return ACQ_OK;
}

int acq_fsk_plan(const acq_fsk_config* cfg, void* stream, acq_fsk_plan_t* out) {
    if (!out) return acq::fail(ACQ_ERR_INVALID_ARG, "null output");
    *out = nullptr;
    acq::FskGeometry g;
    int rc = acq::fsk_geometry(cfg, &g);
    if (rc != ACQ_OK) return rc;
    acq_fsk_plan_s* p = new (std::nothrow) acq_fsk_plan_s();
    if (!p) return acq::fail(ACQ_ERR_OOM, "host allocation failed");
    p->cfg = *cfg;
    p->g = g;
    p->stream = static_cast<hipStream_t>(stream);
    rc = build_fsk(p, cfg);
    p->cfg.bits = nullptr;           // copied to the device; the caller keeps its buffers
    p->cfg.bp_taps = nullptr;
    if (rc != ACQ_OK) {
        free_fsk(p);
        return rc;
    }
    *out = p;
    acq::clear_error();
    return ACQ_OK;
}

int acq_fsk_release(acq_fsk_plan_t p) {
    if (p) {
        (void)hipStreamSynchronize(p->stream);
        free_fsk(p);
    }
    return ACQ_OK;
}

int acq_fsk_demod(acq_fsk_plan_t p, const int16_t* iq, int64_t n, float* d, float* u) {
    int rc = check_iq(p, iq, n);
    if (rc != ACQ_OK) return rc;
    if (n > 0 && (!d || !u)) return acq::fail(ACQ_ERR_INVALID_ARG, "null output");
    if (n == 0) return ACQ_OK;
    acq::FskTask& tk = p->h_tasks[0];
    tk = acq::FskTask{};
    tk.iq = iq;
    tk.n = n;
    tk.tag = -1;
    tk.nfseg = int((n + p->g.vf - 1) / p->g.vf);
    FSK_HIP(hipMemcpyAsync(p->d_tasks, p->h_tasks, sizeof(acq::FskTask), hipMemcpyHostToDevice, p->stream));
    FSK_HIP(launch_front(p, acq::FskTasks{p->d_tasks, 1, 0}, tk.nfseg, false, nullptr, 0));
    FSK_HIP(hipMemcpyAsync(d, p->d_d, sizeof(float) * size_t(n), hipMemcpyDeviceToDevice, p->stream));
    FSK_HIP(hipMemcpyAsync(u, p->d_u, sizeof(float) * size_t(n), hipMemcpyDeviceToDevice, p->stream));
    FSK_HIP(hipStreamSynchronize(p->stream));
    acq::clear_error();
    return ACQ_OK;
}

int acq_fsk_template(acq_fsk_plan_t p, int32_t tag, float* out) {
    if (!p || !out) return acq::fail(ACQ_ERR_INVALID_ARG, "null argument");
    if (tag < 0 || tag >= p->cfg.num_tags) return acq::fail(ACQ_ERR_INVALID_ARG, "tag outside [0, num_tags)");
    FSK_HIP(hipMemcpyAsync(out, p->d_tmpl + size_t(tag) * size_t(p->tstride), sizeof(float) * size_t(p->g.nt),
                           hipMemcpyDeviceToDevice, p->stream));
    FSK_HIP(hipStreamSynchronize(p->stream));
    acq::clear_error();
    return ACQ_OK;
}

}  // extern "C"

namespace {

// Steps 1-7 and the peak keys on the plan's stream for the call's blocks,
// staged in h_tasks[0 .. nblocks) with iq, n and tag set (tag -1: searching,
// one block).  Fills the rest of each entry, copies the table and launches.
// dump (device [T][lags], searching only) gets c at every lag.  Returns the
// result items (templates or tasks) in *items.
int enqueue_fsk(acq_fsk_plan_s* p, int nblocks, bool track, float* dump, int* items) {
    const acq::FskGeometry& g = p->g;
    const int T = p->cfg.num_tags;
    hipStream_t st = p->stream;
    int64_t zoff = 0;
    int fsegs = 0, units = 0;
    for (int b = 0; b < nblocks; ++b) {
        acq::FskTask& tk = p->h_tasks[b];
        tk.lags = tk.n - g.nt + 1;
        tk.zoff = zoff;
        tk.nseg = tk.lags > 0 ? int((tk.lags + g.V - 1) / g.V) : 0;
        tk.nfseg = tk.lags > 0 ? int((tk.n + g.vf - 1) / g.vf) : 0;
        tk.fseg0 = fsegs;
        tk.unit0 = units;
        zoff += tk.n;
        fsegs += tk.nfseg;
        units += tk.nseg;
    }
    const int slots = (units + 1) / 2;              // correlation segments 2s and 2s+1 share slot s
    if (zoff > p->cfg.max_block_len) return acq::fail(ACQ_ERR_BLOCK_TOO_LONG, "blocks longer than max_block_len in all");
    if (slots > g.slots) return acq::fail(ACQ_ERR_BLOCK_TOO_LONG, "blocks need more segments than the plan holds");
    *items = track ? nblocks : T;
    // the correlation segments follow the blocks in the table
    acq::FskUnit* hu = reinterpret_cast<acq::FskUnit*>(p->h_tasks + nblocks);
    for (int b = 0; b < nblocks; ++b) {
        const acq::FskTask& tk = p->h_tasks[b];
        for (int64_t s = 0; s < tk.nseg; ++s) {
            acq::FskUnit& u = hu[tk.unit0 + s];
            u = acq::FskUnit{};
            u.z0 = tk.zoff + s * g.V;
            u.left = int32_t(std::min<int64_t>(tk.n - s * g.V, g.M));
            u.vlim = int32_t(std::min<int64_t>(tk.lags - s * g.V, g.V));
            u.lag0 = uint32_t(s * g.V);
            u.tag = tk.tag;
            u.key = b;
        }
    }
    if (units & 1) {                                // the last slot's absent second segment
        hu[units] = hu[units - 1];
        hu[units].left = hu[units].vlim = 0;
    }
    FSK_HIP(hipMemcpyAsync(p->d_tasks, p->h_tasks,
                           sizeof(acq::FskTask) * size_t(nblocks) + sizeof(acq::FskUnit) * 2 * size_t(slots),
                           hipMemcpyHostToDevice, st));
    const acq::FskUnit* du = reinterpret_cast<const acq::FskUnit*>(p->d_tasks + nblocks);
    acq::FskTasks tt{p->d_tasks, nblocks, track ? 1 : 0};
    if (slots == 0) return ACQ_OK;                  // no lags: no key is read
    {
        FskTimer kt(p, ACQ_FSK_KERNEL_FRONT);
        FSK_HIP(launch_front(p, tt, fsegs, false, nullptr, *items));
    }
    {
        FskTimer kt(p, ACQ_FSK_KERNEL_FORWARD);
        FSK_HIP(acq::launch_fsk_forward(du, p->d_d, g.P, int(g.M), g.log2_sub, slots, p->d_rootsSub, p->d_b1tab,
                                        p->d_X, st));
        if (!track && g.P > 1) {                    // tracking combines in its first step
            BlockTable bt{};
            bt.one.nseg = slots;
            FSK_HIP(acq::launch_forward_combine(fwd_args(p, bt, p->d_X, g.M), slots, ACQ_FP32, st));
        }
    }
    acq::FskCorrArgs ca{};
    ca.X = p->d_X;
    ca.bank = p->d_bank;
    ca.rootsM = p->d_rootsM;
    ca.rootsSub = p->d_rootsSub;
    ca.b1tab = p->d_b1tab;
    ca.G = p->d_G;
    ca.keys = p->d_keys;
    ca.dump = dump;
    ca.units = du;
    ca.lags = p->h_tasks[0].lags;
    ca.M = int(g.M);
    ca.Msub = int(g.Msub);
    ca.P = g.P;
    ca.track = track ? 1 : 0;
    ca.phases = p->d_phases;
    {
        FskTimer kt(p, ACQ_FSK_KERNEL_CORRELATE);
        // groups of items whose first-step outputs fit the plan's buffer: all
        // slots with some of the templates, or some of the slots
        const int most = g.P > 1 ? int(g.group / g.M) : INT32_MAX;
        const int ns = std::min(slots, most);
        int nt = track ? 1 : std::min(T, std::max(1, most / ns));
        if (!track) nt = (T + (T + nt - 1) / nt - 1) / ((T + nt - 1) / nt);       // even groups
        for (int s0 = 0; s0 < slots; s0 += ns)
            for (int t0 = 0; t0 < (track ? 1 : T); t0 += nt) {
                ca.s0 = s0;
                ca.ns = std::min(ns, slots - s0);
                ca.t0 = t0;
                ca.nt = track ? 1 : std::min(nt, T - t0);
                FSK_HIP(acq::launch_fsk_correlate(ca, g.log2_sub, st));
            }
    }
    return ACQ_OK;
}

// Step 8 for the call's result items, compaction and the copy to the host.
int finish_fsk(acq_fsk_plan_s* p, int nblocks, bool track, int items, acq_fsk_detection* out, int32_t capacity,
               int32_t* n_found) {
    const acq::FskGeometry& g = p->g;
    hipStream_t st = p->stream;
    acq::FskRefineArgs ra{};
    ra.d = p->d_d;
    ra.u = p->d_u;
    ra.tmpl = p->d_tmpl;
    ra.keys = p->d_keys;
    ra.partial = p->d_partial;
    ra.dets = p->d_dets;
    ra.found = p->d_found;
    ra.tasks = acq::FskTasks{p->d_tasks, nblocks, track ? 1 : 0};
    ra.nt = g.nt;
    ra.tstride = p->tstride;
    ra.theta = p->cfg.threshold;
    ra.tickets = p->d_tickets;
    // few results are ordered and sent to the host by the refinement launch itself
    const bool tail = items <= acq::kTailItems;
    ra.h_out = tail ? p->h_out : nullptr;
    ra.h_count = p->h_count;
    {
        FskTimer kt(p, ACQ_FSK_KERNEL_REFINE);
        hipLaunchKernelGGL(acq::k_fsk_refine, dim3(unsigned(items) * acq::kFskParts), dim3(256), 0, st, ra);
        FSK_HIP(hipGetLastError());
    }
    if (!tail) {
        hipLaunchKernelGGL(acq::k_fsk_compact, dim3(1), dim3(1024), 0, st, p->d_dets, p->d_found, items, p->d_out,
                           p->d_count);
        FSK_HIP(hipGetLastError());
        FSK_HIP(hipMemcpyAsync(p->h_count, p->d_count, sizeof(int32_t), hipMemcpyDeviceToHost, st));
        FSK_HIP(hipMemcpyAsync(p->h_out, p->d_out, sizeof(acq_fsk_detection) * size_t(items), hipMemcpyDeviceToHost,
                               st));
    }
    FSK_HIP(hipStreamSynchronize(st));
    const int32_t found = *p->h_count;
    *n_found = found;
    const int32_t ncopy = found < capacity ? found : capacity;
    if (ncopy > 0) std::memcpy(out, p->h_out, sizeof(acq_fsk_detection) * size_t(ncopy));
    if (found > capacity) return acq::fail(ACQ_ERR_TRUNCATED, "more detections than capacity");
    acq::clear_error();
    return ACQ_OK;
}

}  // namespace

extern "C" {

int acq_fsk_set_profiling(acq_fsk_plan_t p, int on) {
    if (!p) return acq::fail(ACQ_ERR_INVALID_ARG, "null plan");
    if (on && !p->ev[0][0])
        for (auto& pair : p->ev)
            for (hipEvent_t& e : pair) FSK_HIP(hipEventCreate(&e));
    p->profiling = on != 0;
    return ACQ_OK;
}

int acq_fsk_last_kernel_times(acq_fsk_plan_t p, double* ms, int32_t n) {
    if (!p || !ms || n < ACQ_FSK_NUM_KERNELS) return acq::fail(ACQ_ERR_INVALID_ARG, "bad arguments");
    if (!p->profiling) return acq::fail(ACQ_ERR_INVALID_ARG, "profiling is off");
    for (int k = 0; k < ACQ_FSK_NUM_KERNELS; ++k) {
        float t = 0.f;
        FSK_HIP(hipEventElapsedTime(&t, p->ev[k][0], p->ev[k][1]));
        ms[k] = t;
    }
    return ACQ_OK;
}

int acq_fsk_xcorr(acq_fsk_plan_t p, const int16_t* iq, int64_t n, float* out) {
    int rc = check_iq(p, iq, n);
    if (rc != ACQ_OK) return rc;
    if (n < p->g.nt) return acq::fail(ACQ_ERR_INVALID_ARG, "block shorter than a template");
    if (!out) return acq::fail(ACQ_ERR_INVALID_ARG, "null output");
    p->h_tasks[0] = acq::FskTask{};
    p->h_tasks[0].iq = iq;
    p->h_tasks[0].n = n;
    p->h_tasks[0].tag = -1;
    int items = 0;
    rc = enqueue_fsk(p, 1, false, out, &items);
    if (rc != ACQ_OK) return rc;
    FSK_HIP(hipStreamSynchronize(p->stream));
    acq::clear_error();
    return ACQ_OK;
}

int acq_fsk_detect(acq_fsk_plan_t p, const int16_t* iq, int64_t n, acq_fsk_detection* out, int32_t capacity,
                   int32_t* n_found) {
    int rc = check_iq(p, iq, n);
    if (rc != ACQ_OK) return rc;
    if (!n_found) return acq::fail(ACQ_ERR_INVALID_ARG, "null n_found");
    if (capacity < 0 || (capacity > 0 && !out)) return acq::fail(ACQ_ERR_INVALID_ARG, "bad output buffer");
    *n_found = 0;
    if (n < p->g.nt) {
        acq::clear_error();
        return ACQ_OK;
    }
    p->h_tasks[0] = acq::FskTask{};
    p->h_tasks[0].iq = iq;
    p->h_tasks[0].n = n;
    p->h_tasks[0].tag = -1;
    int items = 0;
    rc = enqueue_fsk(p, 1, false, nullptr, &items);
    if (rc != ACQ_OK) return rc;
    return finish_fsk(p, 1, false, items, out, capacity, n_found);
}

int acq_fsk_track(acq_fsk_plan_t p, const acq_fsk_task* tasks, int32_t ntasks, acq_fsk_detection* out,
                  int32_t capacity, int32_t* n_found) {
    if (!p) return acq::fail(ACQ_ERR_INVALID_ARG, "null plan");
    if (!tasks || !n_found) return acq::fail(ACQ_ERR_INVALID_ARG, "null argument");
    if (capacity < 0 || (capacity > 0 && !out)) return acq::fail(ACQ_ERR_INVALID_ARG, "bad output buffer");
    if (ntasks < 1 || ntasks > p->g.max_tasks) return acq::fail(ACQ_ERR_INVALID_ARG, "ntasks outside [1, max_track_tasks]");
    int64_t total = 0;
    for (int32_t b = 0; b < ntasks; ++b) {
        const int rc = check_iq(p, tasks[b].iq, tasks[b].n);
        if (rc != ACQ_OK) return rc;
        if (tasks[b].tag < 0 || tasks[b].tag >= p->cfg.num_tags)
            return acq::fail(ACQ_ERR_INVALID_ARG, "task tag outside [0, num_tags)");
        total += tasks[b].n;
    }
    if (total > p->cfg.max_block_len) return acq::fail(ACQ_ERR_BLOCK_TOO_LONG, "tasks longer than max_block_len in all");
    *n_found = 0;
    for (int32_t b = 0; b < ntasks; ++b) {
        p->h_tasks[b] = acq::FskTask{};
        p->h_tasks[b].iq = tasks[b].iq;
        p->h_tasks[b].n = tasks[b].n;
        p->h_tasks[b].tag = tasks[b].tag;
    }
    int items = 0;
    const int rc = enqueue_fsk(p, ntasks, true, nullptr, &items);
    if (rc != ACQ_OK) return rc;
    return finish_fsk(p, ntasks, true, items, out, capacity, n_found);
}

}  // extern "C"
