// HIP kernels of the acquisition path (gfx950).
//
//   k_forward_*    : overlap-save segment j, X_j = DFT_M(x[jV .. jV+M)) with a zero
//                    tail, as spc decimated Msub-point transforms (one workgroup
//                    each) combined by one radix-spc decimation-in-time step; beside them
//                    the FP64 sums of |x|^2 (mean block power Pxhat)
//   k_bank         : replica spectra conj(DFT_Msub(chip code)) / M, plan time
//   k_correlate    : the hot loop, in correlate.hip
//   k_refine       : FP64 re-correlation around each tag's peak, re-maximisation,
//                    parabolic vertex, z and energy; detections in tag order
//   k_compact      : detections in tag order, of searches of many items
//
#include <hip/hip_runtime.h>

#include <algorithm>

#include "arrival.h"
#include "device_common.h"
#include "host_logic.h"
#include "kernels.h"

namespace acq {

using namespace kdev;

namespace {

// ------------------------------------------------------------------ block power
// Partial sums of block b in parts[b][*]: part p sums the p-th chunk of the
// block (chunks of at least kPowerMinChunk samples, so a block of n samples
// fills the first power_parts(n) <= kPowerParts parts and no more are read).
// Item p * blocks + b, p < the parts of the longest block the plan takes;
// workgroups stride over the items, and every item is summed in the same
// order whichever workgroup takes it, so the sums are deterministic.
constexpr int kPowerMaxGrid = 1024;
constexpr int64_t kPowerMinChunk = 4096;

__host__ __device__ __forceinline__ int64_t power_chunk(int64_t n) {
    const int64_t c = (n + kPowerParts - 1) / kPowerParts;
    return c > kPowerMinChunk ? c : kPowerMinChunk;
}

__host__ __device__ __forceinline__ int power_parts(int64_t n) {
    return n > 0 ? int((n + power_chunk(n) - 1) / power_chunk(n)) : 0;
}

// Workgroups of NT threads that sum the parts.  A part is summed by 256
// threads (four waves), so a workgroup takes NT / 256 parts at a time, or a
// smaller one a part's waves in turn; 8 samples of each thread are in flight
// together.
template <int NT>
__host__ __device__ constexpr int power_per_group() { return NT > 256 ? NT / 256 : 1; }

template <int NT>
__device__ __forceinline__ void sum_block_power(const BlockTable& bt, const PowerArgs& a, int wg) {
    __shared__ double red[4 * power_per_group<NT>()];
    constexpr int NW = NT / 64, PP = power_per_group<NT>(), PW = NW < 4 ? NW : 4;   // waves of a part
    const int lane = int(threadIdx.x) & 63, wave = int(threadIdx.x) >> 6;
    const int nb = bt.nblocks();
    const int items = nb * a.max_parts;
    // part-major order: the low parts of every block come first and spread
    // over distinct workgroups
    for (int it0 = wg * PP; it0 < items; it0 += a.groups * PP) {
        const int it = it0 + wave / PW;
        const int b = it % nb, part = it / nb;
        const bool in = it < items;
        const BlockDesc d = bt.get(in ? b : 0);
        const int64_t chunk = power_chunk(d.n);
        const int64_t beg = int64_t(part) * chunk;
        const int64_t end = beg + chunk < d.n ? beg + chunk : d.n;
        const bool some = in && beg < d.n;           // uniform over the wave
        for (int vw = wave % PW; vw < 4; vw += PW) {
            double acc = 0.0;
            if (some) {
                constexpr int U = 8;
                for (int64_t i = beg + vw * 64 + lane; i < end; i += 256 * U) {
                    float2 v[U];
#pragma unroll
                    for (int u = 0; u < U; ++u) v[u] = d.x[min(i + 256 * u, end - 1)];
#pragma unroll
                    for (int u = 0; u < U; ++u)
                        if (i + 256 * u < end)
                            acc += double(v[u].x) * double(v[u].x) + double(v[u].y) * double(v[u].y);
                }
            }
            acc = wave_sum(acc);
            if (lane == 0) red[(wave / PW) * 4 + vw] = acc;
        }
        __syncthreads();
        if (some && wave % PW == 0 && lane == 0) {
            const double* r = red + (wave / PW) * 4;
            agent_store(&a.parts[size_t(b) * kPowerParts + part], (r[0] + r[1]) + (r[2] + r[3]));
        }
        __syncthreads();
    }
}

__global__ void k_fill_i32(int* p, int64_t count) {
    const int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (i < count) p[i] = 0;
}

// mean block power from the fixed-order partial sums
// (agent loads: they may have been stored by this launch)
__device__ __forceinline__ double block_mean_power(const double* parts, int64_t n) {
    // the parts are added in index order; loads go out 32 at a time so that a
    // single thread does not wait for each one in turn
    constexpr int kBatch = 32;
    double s = 0.0;
    const int np = power_parts(n);
    int i = 0;
    for (; i + kBatch <= np; i += kBatch) {
        double v[kBatch];
#pragma unroll
        for (int j = 0; j < kBatch; ++j) v[j] = agent_load(&parts[i + j]);
#pragma unroll
        for (int j = 0; j < kBatch; ++j) s += v[j];
    }
    for (; i < np; ++i) s += agent_load(&parts[i]);
    return n > 0 ? s / double(n) : 0.0;
}

// ------------------------------------------------------------------ per-block statistics
// From the block power, for every block b of the table: the power-of-two
// prescale of 16-bit storage, 2^-e with e = round(log2(sqrt(M * Pxhat))) (so
// typical |X| is near 1); the power at the detection threshold, theta * L *
// Pxhat (the z >= theta test on FP32 powers); and whether the block holds a
// non-finite sample (then Pxhat is not finite: |x|^2 of a finite complex64
// value cannot overflow FP64 and every term is >= 0, so no cancellation).
// One workgroup strides over the blocks and counts the non-finite ones.
template <int NT>
__device__ __forceinline__ void block_stats(const BlockTable& bt, const PowerArgs& a) {
    __shared__ int s_bad;
    if (threadIdx.x == 0) s_bad = 0;
    __syncthreads();
    const int nb = bt.nblocks();
    for (int b = int(threadIdx.x); b < nb; b += NT) {
        const BlockDesc d = bt.get(b);
        const double px = block_mean_power(a.parts + size_t(b) * kPowerParts, d.n);
        a.parts[size_t(b) * kPowerParts] = px;
        const bool fin = isfinite(px);
        a.exps[b] = fin && px > 0.0 ? int(rint(0.5 * log2(double(a.M) * px))) : 0;
        const double th = d.theta * double(a.L) * px;
        a.pthr[b] = fin && px > 0.0 && th <= 3.0e38 ? float(th) : __builtin_huge_valf();
        a.bad[b] = fin ? 0 : 1;
        if (!fin) atomicAdd(&s_bad, 1);
    }
    __syncthreads();
    if (threadIdx.x == 0) a.nbad[0] = s_bad;
}

// Workgroup `wg` of a launch's a.groups power workgroups: its share of the
// block power, of the clearing of the search's peak keys, crossing counts and
// refinement tickets, and, in the last one to arrive, the statistics.
template <int NT>
__device__ __forceinline__ void power_group(const BlockTable& bt, const PowerArgs& a, int wg) {
    for (int64_t i = int64_t(wg) * NT + threadIdx.x; i < a.nclear; i += int64_t(a.groups) * NT) {
        a.keys[i] = 0ull;
        a.cross[i] = 0u;
        a.tickets[i] = 0u;
        if (i == 0) a.tickets[a.nclear] = 0u;
    }
    sum_block_power<NT>(bt, a, wg);
    if (!last_arrival(a.ticket, unsigned(a.groups))) return;
    block_stats<NT>(bt, a);
}

// ------------------------------------------------------------------ forward spectra
// One workgroup per global segment g (looping when the grid is smaller):
// X_g = DFT_M of the segment held in slot g (segment g - seg0 of its block, or
// the listed segment when only some segments are searched), in two kernels:
//
// k_forward_sub: work item (g, r), r < spc: the Msub-point DFT of the decimated
//   samples x[base + spc*i + r] (zero beyond the block), F_r, written to
//   X_g[r*Msub + i].  One workgroup per item (a loop over items for batches).
// k_forward_combine: the radix-spc decimation-in-time step, in place per i:
//   X_g[i + q*Msub] = F_0[i] + sum_{r>=1} exp(-j 2 pi (i + q*Msub) r / M) F_r[i],
//   accumulated in FP32 in increasing r; 16-bit plans store the result scaled
//   and packed in the 16-bit copy instead.  Each spectrum sits at offset xpad
//   of its slot, with its last xpad entries copied before it and its first
//   xpad after it (rotated reads need no wrap-around).
// The launch's first a.power.groups workgroups sum the block power and form the
// statistics beside the transforms (as launches of their own, 4.5 and 2.6 us
// and two launch gaps for one block of 131,072 samples; the transforms take
// 10.6 us with or without them).
// PREMIX: exact bins, whose classes have residual offsets (a kernel of its own:
// its phase reductions cost the other one registers).
template <class E, bool PREMIX>
__global__ __launch_bounds__(E::NT) void k_forward_sub(FwdArgs a) {
    __shared__ float2 lds[E::LDS];
    __shared__ float2 extra[E::EXTRA];
    const int wg = int(blockIdx.x) - a.power.groups, wgs = int(gridDim.x) - a.power.groups;
    if (wg < 0) {
        power_group<E::NT>(a.blocks, a.power, int(blockIdx.x));
        return;
    }
    E eng;
    eng.init(a.rootsSub, extra);
    const __amdgpu_buffer_rsrc_t b1 = make_rsrc(a.b1tab, E::B1_TABLE * 8);
    const int per_seg = a.ncls * a.spc;
    const int items = a.blocks.total_seg() * per_seg;
    // the per_seg items of a segment read interleaved samples of one input
    // range: with one item per workgroup, place them on one XCD (workgroups
    // go to the XCDs in turn), so that its L2 fetches the range once.  Within
    // each group of kXcds * per_seg workgroups, workgroup j takes item
    // k = j / kXcds of segment j % kXcds of the group.
    const int grp = kXcds * per_seg;
    const bool xcd_map = wgs >= items && per_seg > 1;
    for (int b = wg; b < items; b += wgs) {
        int it = b;
        if (xcd_map && b < items / grp * grp) {
            const int q = b / grp, j = b - q * grp;
            it = (q * kXcds + j % kXcds) * per_seg + j / kXcds;
        }
        const int g = it / per_seg, rem = it - g * per_seg, c = rem / a.spc, r = rem - c * a.spc;
        const int bi = a.blocks.block_of_segment(g);
        const BlockDesc d = a.blocks.get(bi);
        const int64_t base = int64_t(a.blocks.segment(g, d)) * a.V;
        const double cyc = PREMIX ? a.cls_cyc[c] : 0.0;          // residual offset of the class
        // the segment's samples, zero past the block's end: buffer loads bounded
        // by the samples left, so that all 16 are in flight together (a branch
        // around each load waits for them one by one)
        const int64_t left = d.n - base < a.M ? d.n - base : a.M;
        const __amdgpu_buffer_rsrc_t xr =
            make_rsrc(wave_uniform(d.x + base), uint32_t(__builtin_amdgcn_readfirstlane(int(left))) * 8u);
        float2 v[16];
#pragma unroll
        for (int m = 0; m < 16; ++m) v[m] = bload(xr, (a.spc * eng.in_index(m) + r) * 8, 0);
        if (PREMIX && cyc != 0.0) {                // x * exp(-j 2 pi cyc idx), phase reduced in FP64
            int n0 = eng.in_index(0);              // (opaque: 16 indices held over the loop spilled)
            asm volatile("" : "+v"(n0));
#pragma unroll
            for (int m = 0; m < 16; ++m) {
                const int64_t idx = base + a.spc * (n0 + m * (E::N / 16)) + r;
                double ph = cyc * double(idx);
                ph -= floor(ph);
                float sn, cs;
                sincospif(2.0f * float(ph), &sn, &cs);
                v[m] = make_float2(fmaf(v[m].x, cs, v[m].y * sn), fmaf(v[m].y, cs, -v[m].x * sn));
            }
        }
        eng.template transform<-1>(v, lds, b1, extra);
        float2* F = a.X + (size_t(g) * size_t(a.ncls) + size_t(c)) * size_t(a.xstride) + size_t(a.xpad) +
                    size_t(r) * size_t(a.Msub);
        store_natural(eng, v, lds, F);
    }
}

// 256 threads per workgroup, one i per thread; a workgroup's 256 i lie in one
// slot (Msub is a multiple of 256).  Workgroups past the slots in use exit.
// SPC (= a.spc) is a template argument so the spc inputs stay in registers.
// The twiddle of phase r is the r-th power of exp(-j 2 pi io / M): one table
// load per output, then products (exact table values for spc <= 2).
template <int PREC, int SPC>
__global__ __launch_bounds__(256) void k_forward_combine(FwdArgs a) {
    using St = dev::Storage<PREC>;
    const int per_slot = a.Msub / 256;
    const int g = int(blockIdx.x) / per_slot;           // spectra slot: segment * ncls + class
    if (g >= a.blocks.total_seg() * a.ncls) return;
    const int i = (int(blockIdx.x) - g * per_slot) * 256 + int(threadIdx.x);
    float2* X = a.X + size_t(g) * size_t(a.xstride) + size_t(a.xpad);
    float xs = 1.0f;
    if constexpr (PREC != ACQ_FP32) xs = ldexpf(1.0f, -a.exps[a.blocks.block_of_segment(g / a.ncls)]);
    float2 F[SPC];
#pragma unroll
    for (int r = 0; r < SPC; ++r) F[r] = X[r * a.Msub + i];
    // 16 phases (the FSK path's 2^18-point segments): X[i + q Msub] is the
    // 16-point DFT over r of F_r[i] exp(-j 2 pi i r / M)
    if constexpr (SPC == 16) {
        const float2 w1 = a.rootsM[i];
        float2 w = w1;
#pragma unroll
        for (int r = 1; r < SPC; ++r) {
            F[r] = cmulc(F[r], w);
            if (r + 1 < SPC) w = cmul(w, w1);
        }
        dev::dft16<-1>(F);
    }
#pragma unroll
    for (int q = 0; q < SPC; ++q) {
        const int io = i + q * a.Msub;
        float2 c = F[0];
        if constexpr (SPC == 16) {
            c = F[q];
        } else if constexpr (SPC > 1) {
            const float2 w1 = a.rootsM[io];
            float2 w = w1;
#pragma unroll
            for (int r = 1; r < SPC; ++r) {
                c = cadd(c, cmulc(F[r], w));
                if (r + 1 < SPC) w = cmul(w, w1);
            }
        }
        // the spectrum, and its wrap-around copy when io is within xpad of an end
        if constexpr (PREC == ACQ_FP32) {
            X[io] = c;
            if (io < a.xpad) X[a.M + io] = c;
            if (io >= a.M - a.xpad) X[io - a.M] = c;
        } else {
            typename St::T* Xh = reinterpret_cast<typename St::T*>(a.Xh) + size_t(g) * size_t(a.xstride) +
                                 size_t(a.xpad);
            const typename St::T h = St::pack(make_float2(c.x * xs, c.y * xs));
            Xh[io] = h;
            if (io < a.xpad) Xh[a.M + io] = h;
            if (io >= a.M - a.xpad) Xh[io - a.M] = h;
        }
    }
}

// ------------------------------------------------------------------ replica bank
// bank[t][i] = 2^bank_exp * conj(DFT_Msub(chips_t))[i] / M in the storage format
template <class E, int PREC>
__global__ __launch_bounds__(E::NT) void k_bank(const int8_t* __restrict__ chips, int C,
                                                void* __restrict__ bank,
                                                const float2* __restrict__ rootsSub,
                                                const float2* __restrict__ b1tab, int M, int bank_exp) {
    using St = dev::Storage<PREC>;
    __shared__ float2 lds[E::LDS];
    __shared__ float2 extra[E::EXTRA];
    E eng;
    eng.init(rootsSub, extra);
    const __amdgpu_buffer_rsrc_t b1 = make_rsrc(b1tab, E::B1_TABLE * 8);
    const int tag = blockIdx.x;
    float2 v[16];
#pragma unroll
    for (int m = 0; m < 16; ++m) {
        const int ip = eng.in_index(m);
        v[m] = make_float2(ip < C ? float(chips[size_t(tag) * C + ip]) : 0.f, 0.f);
    }
    eng.template transform<-1>(v, lds, b1, extra);
    const float s = ldexpf(1.0f, bank_exp) / float(M);   // exact: powers of two
    const int ob = eng.out_base();
    typename St::T* out = reinterpret_cast<typename St::T*>(bank) + size_t(tag) * bank_stride(E::N);
#pragma unroll
    for (int m = 0; m < 16; ++m) {
        const int i = ob + E::out_off(m);
        if (i <= E::N / 2) out[i] = St::pack(make_float2(v[m].x * s, -v[m].y * s));   // the rest is the mirror
    }
}

// ------------------------------------------------------------------ refine
constexpr int kMaxWin = 2 * kMaxRefineRadius + 3;

// FP64 refinement of each (block, tag) peak key, one launch.  The window of W =
// 2R + 3 lags is centred on the key's lag and its samples are split into
// kRefineParts parts; an item's workgroups take a.parts_each of them each and add
// the re- and im-sums of the mixed samples against the tag's replica and the
// sample energy under it for every lag of the window, and the last of them to
// arrive adds the parts in order, re-maximises over the inner 2R+1 lags and
// writes the detection.  When the maximum sits on the inner edge it takes the
// window re-centred there once more first, part by part in the same order (the
// two kernels of a second pass cost each search two launches; the powers of the
// two passes' centres differ by the rounding of the search, so few items do).
// The last item of a small search writes the detections in (block, tag) order
// as well, also to the host (k_compact and two copies otherwise).
// Against two passes of two kernels, the compaction and its copies, with the
// power in launches of its own: a search of 1 code in 131,072 samples 89.7 ->
// 60.6 us, of 13 codes in 5 bins of 100,003 samples 118 -> 91 us, 9 tracking
// tasks 133 -> 98 us.  The kernel against the two passes', 16,384 samples each: 64
// items 22 -> 18 us, 256 42 -> 36, 4096 418 -> 356, 16,384 1.49 -> 1.21 ms (with 16
// workgroups of one part for every item 18, 51, 656 and 2.59 ms: an item's share
// is then smaller than what a workgroup pays besides).
// Registers decide how many workgroups hide each other's loads and sums: 32-bit
// indices (a window has fewer than 2^18 samples), the exact bins' phases in a
// kernel of their own, and one copy of the sums for both passes leave 95 of them
// at radius 1 (121 with two copies and 64-bit indices).
// The mix exp(-j 2 pi m_k i / M) is an FP64 table entry at (m_k i) mod M (M a
// power of two, so the reduction is exact), or the exact bin's FP64 phase.
struct RefineItem {
    int bi, tag;
    size_t slot;
    BlockDesc d;
};

__device__ __forceinline__ bool refine_item(const RefineArgs& a, int item, RefineItem* r) {
    const int per = a.track ? 1 : a.T;
    r->bi = item / per;
    if (r->bi >= a.blocks.nblocks()) return false;
    r->d = a.blocks.get(r->bi);
    r->tag = a.track ? r->d.tag : item % per;
    if (r->tag < 0 || r->tag >= a.T) return false;
    r->slot = size_t(r->bi) * a.T + r->tag;
    return true;
}

constexpr int kRefineMaxChips = 1 << 14;  // the longest code of any transform length
// chips under one part: (C spc + W - 1) / kRefineParts samples rounded up, and W - 1 more
constexpr int kRefineChipsLds = kRefineMaxChips / kRefineParts + 2 * kMaxWin + 4;

constexpr int kRefineThreads = 256;

// Sums of part `part` of an item's window around `center`: sum t in thread t < 3W.
// (One after the other is safe: a barrier lies between any two uses of the LDS.)
template <int WMAX, bool EXACT>
__device__ __forceinline__ double refine_sums(const RefineArgs& a, const RefineItem& it, int part, int k,
                                              int64_t center) {
    __shared__ int8_t s_chips[kRefineChipsLds];
    __shared__ double red[kRefineThreads / 64][3 * WMAX];
    constexpr int NT = kRefineThreads, NW = NT / 64;
    const BlockDesc& d = it.d;
    const int R = a.radius, L = int(a.L);
    const int W = 2 * R + 3;                 // <= WMAX, which the launcher picks
    const int t = int(threadIdx.x), lane = t & 63, wave = t >> 6;
    const int64_t lam0 = center - R - 1;
    // samples e of the window (lag lam0's first is e = 0) inside the block, split into parts
    const int e_lo = lam0 < 0 ? int(-lam0) : 0;
    const int e_hi = int(min(int64_t(L) + W - 1, d.n - lam0));
    const int ch = (e_hi - e_lo + kRefineParts - 1) / kRefineParts;
    const int p0 = e_lo + part * ch, p1 = min(e_hi, p0 + ch);
    // the part's chips (replica samples e - w, w < W)
    const int8_t* chips = a.chips + size_t(it.tag) * size_t(a.C);
    const int c0 = max(0, (p0 - W + 1) >> a.log2_spc);
    const int c1 = min(a.C, ((p1 - 1) >> a.log2_spc) + 1);
    for (int q = c0 + t; q < c1; q += NT) s_chips[q - c0] = chips[q];
    __syncthreads();
    // table index (m_k i) mod M in 32 bits (M a power of two)
    const unsigned mrot = unsigned(a.rot_signed[k]), mmask = unsigned(a.M) - 1u, i0 = unsigned(lam0);
    const double fk = a.cyc[k];
    const float2* x = d.x + lam0;
    double cr[WMAX], ci[WMAX], en[WMAX];
#pragma unroll
    for (int w = 0; w < WMAX; ++w) cr[w] = ci[w] = en[w] = 0.0;
    constexpr int U = WMAX > 5 ? 1 : 4;      // a thread's samples loaded together
    for (int e0 = p0 + t; e0 < p1; e0 += U * NT) {
        float2 xs[U];
        double2 ts[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int e = min(e0 + u * NT, p1 - 1);
            xs[u] = x[unsigned(e)];
            if constexpr (!EXACT) ts[u] = a.roots64[(mrot * (i0 + unsigned(e))) & mmask];
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int e = e0 + u * NT;
            if (e >= p1) break;
            const double xr = xs[u].x, xi = xs[u].y;
            double2 cs;
            if constexpr (EXACT) {              // exp(-j 2 pi (f_k / Fs) i), phase reduced in FP64
                double ph = fk * double(lam0 + e);
                ph -= floor(ph);
                sincospi(2.0 * ph, &cs.y, &cs.x);
            } else {
                cs = ts[u];
            }
            const double mr = xr * cs.x + xi * cs.y;      // x * exp(-j 2 pi m i / M)
            const double mi = xi * cs.x - xr * cs.y;
            const double pw = xr * xr + xi * xi;
#pragma unroll
            for (int w = 0; w < WMAX; ++w) {
                const int nn = e - w;
                if (w < W && nn >= 0 && nn < L) {
                    const double sg = double(s_chips[(nn >> a.log2_spc) - c0]);
                    cr[w] += mr * sg;
                    ci[w] += mi * sg;
                    en[w] += pw;
                }
            }
        }
    }
#pragma unroll
    for (int w = 0; w < WMAX; ++w) {
        const double r0 = wave_sum(cr[w]), r1 = wave_sum(ci[w]), r2 = wave_sum(en[w]);
        if (lane == 0) {
            red[wave][3 * w] = r0;
            red[wave][3 * w + 1] = r1;
            red[wave][3 * w + 2] = r2;
        }
    }
    __syncthreads();
    double v = 0.0;
    if (t < 3 * W)
        for (int q = 0; q < NW; ++q) v += red[q][t];
    return v;
}

// Window position of the largest power (the centre, then the lowest lag, at a
// tie), and whether the window may continue past it.
__device__ __forceinline__ int refine_best(const RefineArgs& a, const RefineItem& it, int64_t center, const double* P,
                                           bool* hit) {
    const int W = 2 * a.radius + 3;
    int wb = a.radius + 1;
    for (int w = 1; w <= W - 2; ++w)
        if (P[w] > P[wb] || (P[w] == P[wb] && w < wb)) wb = w;
    const int64_t lam = center - a.radius - 1 + wb;
    *hit = (wb == 1 && lam > 0) || (wb == W - 2 && lam < it.d.lags - 1);
    return wb;
}

// The detection record of an item whose largest power is at window position wb.
__device__ __forceinline__ void refine_record(const RefineArgs& a, const RefineItem& it, int k, int64_t lam, int wb,
                                              bool hit, const double* sums, const double* P) {
    const BlockDesc& d = it.d;
    unsigned flags = hit ? ACQ_DET_WINDOW_EDGE : 0u;
    const double p0 = P[wb];
    const double pm = P[wb - 1] < 0.0 ? 0.0 : P[wb - 1];
    const double pp = P[wb + 1] < 0.0 ? 0.0 : P[wb + 1];
    double delta = 0.0;
    if (lam == 0 || lam == d.lags - 1) {
        flags |= ACQ_DET_NEAR_EDGE;
    } else {
        const double den = pm - 2.0 * p0 + pp;
        if (den < 0.0) {
            delta = 0.5 * (pm - pp) / den;
            delta = delta > 0.5 ? 0.5 : (delta < -0.5 ? -0.5 : delta);
        }
    }
    const double px = a.parts[size_t(it.bi) * kPowerParts];      // the mean power (block_stats)
    const double z = px > 0.0 ? p0 / (double(a.L) * px) : 0.0;
    const bool suppressed = a.check_finite && a.bad[it.bi];
    acq_detection r;
    r.tag = it.tag;
    r.bin = k;
    r.lag = lam;
    r.toa_samples = double(lam) + delta;
    r.freq_hz = a.freqs[k];
    r.peak_power = p0;
    r.z = z;
    const double energy = sums[3 * wb + 2];
    r.energy = energy;
    r.block_power = px;
    // relative power and SNR (Section 3 step 8's power and SNR sums)
    const double Ld = double(a.L);
    r.power = p0 / (Ld * Ld);
    const double s2 = (energy - p0 / Ld) / Ld;
    r.snr = s2 > 0.0 ? r.power / s2 : __builtin_huge_val();
    r.block = it.bi;
    r.flags = flags;
    r.crossings = int64_t(a.cross[it.slot]);
    agent_store_record(&a.dets[it.slot], r);
    agent_store(&a.found[it.slot], z >= d.theta && !suppressed ? 1 : 0);
}

// The detections of a search of at most kTailItems items, in order, to a.out and
// the host (as k_compact does).
__device__ __forceinline__ void compact_tail(const RefineArgs& a, int items) {
    auto slot = [&](int e) {
        RefineItem it;
        return refine_item(a, e, &it) && agent_load(&a.found[it.slot]) ? int(it.slot) : -1;
    };
    const int n = compact_records<kRefineThreads, kTailItems>(items, a.dets, slot, a.capacity, a.out, a.h_out);
    if (threadIdx.x == 0) {
        *a.count = n;
        if (a.h_out) {
            a.h_count[0] = n;
            a.h_count[1] = *a.nbad;
        }
    }
}

template <int WMAX, bool EXACT>
__global__ __launch_bounds__(kRefineThreads, WMAX > 5 ? (EXACT ? 2 : 3) : EXACT ? 4 : 5) void k_refine(RefineArgs a) {
    __shared__ double sums[3 * WMAX], P[WMAX];
    const int groups = kRefineParts / a.parts_each;    // workgroups of an item
    const int item = int(blockIdx.x) / groups, first = int(blockIdx.x) % groups * a.parts_each;
    const int items = a.blocks.nblocks() * (a.track ? 1 : a.T);
    if (item >= items) return;               // a batch smaller than the plan's capacity
    RefineItem it;
    const bool known = refine_item(a, item, &it);      // false: a tracking task of no tag
    const unsigned long long key = known && it.d.lags > 0 ? a.keys[it.slot] : 0ull;
    if (key != 0ull) {
        const unsigned idx = ~unsigned(key & 0xffffffffull);
        const int k = int(idx % unsigned(a.K)), t = int(threadIdx.x), W = 2 * a.radius + 3;
        int64_t center = int64_t(idx / unsigned(a.K));
        int q0 = first, q1 = first + a.parts_each, wb = 0;
        bool hit = false;
        for (int pass = 0; pass < 2; ++pass) {
            const bool split = q1 - q0 < kRefineParts;
            double* partial = a.partial + size_t(item) * kRefineParts * size_t(3 * WMAX) + t;
            double tot = 0.0;                          // sum t over the parts, in their order
            for (int q = q0; q < q1; ++q) {
                const double v = refine_sums<WMAX, EXACT>(a, it, q, k, center);
                if (split && t < 3 * W) agent_store(&partial[q * (3 * WMAX)], v);
                tot += v;
            }
            if (split) {
                if (!last_arrival(&a.tickets[1 + item], unsigned(groups))) return;
                tot = 0.0;
                if (t < 3 * W) {
                    double v[kRefineParts];
#pragma unroll
                    for (int q = 0; q < kRefineParts; ++q) v[q] = agent_load(&partial[q * (3 * WMAX)]);
#pragma unroll
                    for (int q = 0; q < kRefineParts; ++q) tot += v[q];
                }
            }
            if (t < 3 * W) sums[t] = tot;
            __syncthreads();
            if (t < W) {
                const int64_t lam = center - a.radius - 1 + t;
                const double re = sums[3 * t], im = sums[3 * t + 1];
                P[t] = (lam >= 0 && lam < it.d.lags) ? re * re + im * im : -1.0;
            }
            __syncthreads();
            wb = refine_best(a, it, center, P, &hit);  // every thread the same
            if (!hit || pass) break;
            center += wb - a.radius - 1;
            q0 = 0;
            q1 = kRefineParts;
        }
        if (threadIdx.x == 0) refine_record(a, it, k, center - a.radius - 1 + wb, wb, hit, sums, P);
    } else {                                 // no valid lag was searched for this tag
        if (first != 0) return;
        if (known && threadIdx.x == 0) agent_store(&a.found[it.slot], 0);
    }
    if (a.tail && last_arrival(&a.tickets[0], unsigned(items))) compact_tail(a, items);
}

// Detections in (block, tag) order.  One workgroup: each thread takes a
// contiguous run of candidates, counts its detections, an exclusive scan over
// the threads gives its first output slot, and it copies its run in order.
// Candidates are every (block, tag), or (block, its tag) for tracking tasks.
constexpr int kCompactThreads = 1024;

__global__ __launch_bounds__(kCompactThreads) void k_compact(BlockTable bt, const acq_detection* __restrict__ dets,
                                                             const int32_t* __restrict__ found, int T, int track,
                                                             acq_detection* __restrict__ out, int32_t capacity,
                                                             int32_t* __restrict__ count) {
    __shared__ int scan[kCompactThreads];
    const int t = int(threadIdx.x);
    const int nb = bt.nblocks();
    const int64_t n = track ? int64_t(nb) : int64_t(nb) * T;
    const int64_t per = (n + kCompactThreads - 1) / kCompactThreads;
    const int64_t e0 = min(n, int64_t(t) * per), e1 = min(n, e0 + per);
    auto slot = [&](int64_t e) -> int64_t {
        if (!track) return e;
        const int tag = bt.get(int(e)).tag;
        return tag >= 0 && tag < T ? e * T + tag : -1;
    };
    int c = 0;
    for (int64_t e = e0; e < e1; ++e) {
        const int64_t s = slot(e);
        c += s >= 0 && found[s] ? 1 : 0;
    }
    scan[t] = c;
    __syncthreads();
    for (int off = 1; off < kCompactThreads; off <<= 1) {     // inclusive Hillis-Steele scan
        const int v = t >= off ? scan[t - off] : 0;
        __syncthreads();
        scan[t] += v;
        __syncthreads();
    }
    int o = scan[t] - c;
    for (int64_t e = e0; e < e1 && o < capacity; ++e) {
        const int64_t s = slot(e);
        if (s >= 0 && found[s]) out[o++] = dets[s];
    }
    if (t == kCompactThreads - 1) *count = scan[t];
}

}  // namespace

// ------------------------------------------------------------------ launchers
hipError_t launch_fill_i32(int* p, int64_t count, hipStream_t st) {
    if (count <= 0) return hipSuccess;
    const int64_t blocks = (count + 255) / 256;
    hipLaunchKernelGGL(k_fill_i32, dim3(unsigned(blocks)), dim3(256), 0, st, p, count);
    return hipGetLastError();
}

template <class E>
static hipError_t fwd_e(FwdArgs a, int grid, int power_blocks, int64_t power_len, hipStream_t st) {
    a.power.groups = 0;
    if (power_blocks > 0) {
        constexpr int PP = power_per_group<E::NT>();
        a.power.max_parts = std::max(power_parts(power_len), 1);
        const int64_t items = int64_t(power_blocks) * a.power.max_parts;
        // (and at most 2048 entries to clear a workgroup, as far as that goes)
        a.power.groups = int(std::min<int64_t>(std::max((items + PP - 1) / PP, (a.power.nclear + 2047) / 2048),
                                               kPowerMaxGrid / PP));
        grid += a.power.groups;
    }
    if (a.premix)
        hipLaunchKernelGGL((k_forward_sub<E, true>), dim3(grid), dim3(E::NT), 0, st, a);
    else
        hipLaunchKernelGGL((k_forward_sub<E, false>), dim3(grid), dim3(E::NT), 0, st, a);
    return hipGetLastError();
}

template <int PREC>
static hipError_t combine_p(const FwdArgs& a, dim3 grid, hipStream_t st) {
    if constexpr (PREC == ACQ_FP32) {
        if (a.spc == 16) {                  // the FSK path's 2^18-point segments (16 phases of 2^14)
            hipLaunchKernelGGL((k_forward_combine<PREC, 16>), grid, dim3(256), 0, st, a);
            return hipSuccess;
        }
    }
    switch (a.spc) {
        case 1: hipLaunchKernelGGL((k_forward_combine<PREC, 1>), grid, dim3(256), 0, st, a); break;
        case 2: hipLaunchKernelGGL((k_forward_combine<PREC, 2>), grid, dim3(256), 0, st, a); break;
        case 3: hipLaunchKernelGGL((k_forward_combine<PREC, 3>), grid, dim3(256), 0, st, a); break;
        case 4: hipLaunchKernelGGL((k_forward_combine<PREC, 4>), grid, dim3(256), 0, st, a); break;
        case 5: hipLaunchKernelGGL((k_forward_combine<PREC, 5>), grid, dim3(256), 0, st, a); break;
        case 6: hipLaunchKernelGGL((k_forward_combine<PREC, 6>), grid, dim3(256), 0, st, a); break;
        case 7: hipLaunchKernelGGL((k_forward_combine<PREC, 7>), grid, dim3(256), 0, st, a); break;
        case 8: hipLaunchKernelGGL((k_forward_combine<PREC, 8>), grid, dim3(256), 0, st, a); break;
        default: return hipErrorInvalidValue;
    }
    return hipSuccess;
}

hipError_t launch_forward_combine(const FwdArgs& a, int slots, int prec, hipStream_t st) {
    if (slots <= 0) return hipSuccess;
    if (a.Msub % 256 || a.spc < 1 || (a.spc > 8 && !(a.spc == 16 && prec == ACQ_FP32))) return hipErrorInvalidValue;
    const dim3 cgrid(unsigned(slots) * unsigned(a.Msub / 256));
    hipError_t e;
    switch (prec) {
        case ACQ_FP32: e = combine_p<ACQ_FP32>(a, cgrid, st); break;
        case ACQ_FP16: e = combine_p<ACQ_FP16>(a, cgrid, st); break;
        case ACQ_BF16: e = combine_p<ACQ_BF16>(a, cgrid, st); break;
        default: return hipErrorInvalidValue;
    }
    return e == hipSuccess ? hipGetLastError() : e;
}

hipError_t launch_forward(const FwdArgs& a, int grid, int combine_slots, int power_blocks, int64_t power_len,
                          int log2_sub, int prec, hipStream_t st) {
    if (grid <= 0 && power_blocks <= 0) return hipSuccess;
    if ((1 << log2_sub) != a.Msub || a.Msub % 256 || a.spc < 1 || (a.spc > 8 && !(a.spc == 16 && prec == ACQ_FP32)))
        return hipErrorInvalidValue;
    if (a.xpad < 0 || a.xpad > a.M / 2 || a.xstride < int64_t(a.M) + 2 * int64_t(a.xpad)) return hipErrorInvalidValue;
    hipError_t e;
    switch (log2_sub) {
        case 10: e = fwd_e<StockhamEngine<10>>(a, grid, power_blocks, power_len, st); break;
        case 11: e = fwd_e<StockhamEngine<11>>(a, grid, power_blocks, power_len, st); break;
        case 12: e = fwd_e<StockhamEngine<12>>(a, grid, power_blocks, power_len, st); break;
        case 13: e = fwd_e<StockhamEngine<13>>(a, grid, power_blocks, power_len, st); break;
        case 14: e = fwd_e<Fft14>(a, grid, power_blocks, power_len, st); break;
        default: return hipErrorInvalidValue;
    }
    if (e != hipSuccess) return e;
    return launch_forward_combine(a, combine_slots, prec, st);
}

template <class E>
static hipError_t bank_e(const int8_t* chips, int T, int C, void* bank, const float2* rootsSub,
                         const float2* b1tab, int M, int bank_exp, int prec, hipStream_t st) {
    switch (prec) {
        case ACQ_FP32:
            hipLaunchKernelGGL((k_bank<E, ACQ_FP32>), dim3(T), dim3(E::NT), 0, st, chips, C, bank, rootsSub, b1tab, M,
                               bank_exp);
            break;
        case ACQ_FP16:
            hipLaunchKernelGGL((k_bank<E, ACQ_FP16>), dim3(T), dim3(E::NT), 0, st, chips, C, bank, rootsSub, b1tab, M,
                               bank_exp);
            break;
        case ACQ_BF16:
            hipLaunchKernelGGL((k_bank<E, ACQ_BF16>), dim3(T), dim3(E::NT), 0, st, chips, C, bank, rootsSub, b1tab, M,
                               bank_exp);
            break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_bank(const int8_t* chips, int T, int C, void* bank, const float2* rootsSub,
                       const float2* b1tab, int Msub, int M, int bank_exp, int log2_sub, int prec,
                       hipStream_t st) {
    if ((1 << log2_sub) != Msub || C > Msub) return hipErrorInvalidValue;
    switch (log2_sub) {
        case 10: return bank_e<StockhamEngine<10>>(chips, T, C, bank, rootsSub, b1tab, M, bank_exp, prec, st);
        case 11: return bank_e<StockhamEngine<11>>(chips, T, C, bank, rootsSub, b1tab, M, bank_exp, prec, st);
        case 12: return bank_e<StockhamEngine<12>>(chips, T, C, bank, rootsSub, b1tab, M, bank_exp, prec, st);
        case 13: return bank_e<StockhamEngine<13>>(chips, T, C, bank, rootsSub, b1tab, M, bank_exp, prec, st);
        case 14: return bank_e<Fft14>(chips, T, C, bank, rootsSub, b1tab, M, bank_exp, prec, st);
        default: return hipErrorInvalidValue;
    }
}

// Parts that a workgroup of k_refine takes, one after the other.  Few items need
// all 16 workgroups each to fill the chip (64 items of 16,384 samples 18 us; with 4
// parts a workgroup 26, with all 16, 71); of many, each workgroup pays its start,
// its stores to the item's last one and the arrival again (4096 items 510 us; with
// 4 parts 382, 8 364, 16 356).  The lines lie about where the times cross: over 16
// to 16,384 items of 1024 and 16,384 samples the rule is 3 % off the best of 1, 2, 4,
// 8 and 16 on average, 18 % at the worst (80 items), at radius 8 3 and 15 %.
static int refine_parts_each(int items) {
    return items < 96 ? 1 : items < 192 ? 2 : items < 1024 ? 4 : items < 4096 ? 8 : 16;
}

hipError_t launch_refine(RefineArgs a, int max_blocks, hipStream_t st) {
    if (a.radius < 0 || a.radius > kMaxRefineRadius || a.C > kRefineMaxChips || (a.M & (a.M - 1)) || (1 << a.log2_spc) != a.spc ||
        !a.partial || !a.tickets)
        return hipErrorInvalidValue;
    const int items = max_blocks * (a.track ? 1 : a.T);
    if (a.tail && (items > kTailItems || !a.out || !a.count)) return hipErrorInvalidValue;
    a.parts_each = refine_parts_each(items);
    const dim3 grid(unsigned(items) * unsigned(kRefineParts / a.parts_each));
    auto go = [&](auto kern) { hipLaunchKernelGGL(kern, grid, dim3(kRefineThreads), 0, st, a); };
    if (a.radius <= 1)
        a.exact ? go(k_refine<5, true>) : go(k_refine<5, false>);
    else
        a.exact ? go(k_refine<kMaxWin, true>) : go(k_refine<kMaxWin, false>);
    return hipGetLastError();
}

hipError_t launch_compact(const BlockTable& bt, const acq_detection* dets, const int32_t* found, int T, int track,
                          acq_detection* out, int32_t capacity, int32_t* count, hipStream_t st) {
    hipLaunchKernelGGL(k_compact, dim3(1), dim3(kCompactThreads), 0, st, bt, dets, found, T, track, out, capacity,
                       count);
    return hipGetLastError();
}

}  // namespace acq
