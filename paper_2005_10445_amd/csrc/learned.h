// Proposal stage: STFT power map, 1-D CNN (inference and training), window
// scores and the proposal-to-segment mapping.  Launch interface used by
// cnn.hip.
//
// Rows are frames of a batch of equal-length blocks: row r is frame r mod F of
// block r / F.  Activations are row-major [rows][channels]; convolutions pad
// with zeros at each block's edges.
#pragma once

#include <hip/hip_runtime.h>
#include <cstdint>

namespace acq {
namespace learned {

constexpr int kWin = 256;          // STFT length
constexpr int kHop = 128;          // STFT hop
constexpr int kSpan = 128;         // window-score length (frames)
constexpr int kCh = 64;            // channels of every conv layer
constexpr int kTaps = 5;
constexpr int kLayers = 4;
constexpr int kMaxTx = 32;         // transmissions per synthetic block
constexpr int kDilation[kLayers] = {1, 2, 4, 8};

inline int64_t num_frames(int64_t n) { return n < kWin ? 0 : (n - kWin) / kHop + 1; }

// FP32 parameter vector: per layer l, W_l[5][cin_l][64] then b_l[64]; then the
// head wh[64] and bh.  The bf16 copies hold, per layer, W_l in the order that the
// matrix instructions read their B operand in, once with the outputs as the columns
// of the forward product (k: the inputs) and once with the inputs as those of the
// input gradient's (k: the outputs): per tap and 32-deep k step the 16-column tiles,
// each its 64 lanes' 8 values (conv_operand in learned_kernels.hip).
struct NetLayout {
    int cin[kLayers];
    int64_t w_off[kLayers], b_off[kLayers], wh_off, bh_off, total;
    int64_t bf_off[kLayers], bf_total;
};
NetLayout net_layout(int cin0);

// One transmission of a synthetic training block (sample-level model of the
// tag-bank workload: BPSK chips held spc samples, on-grid carrier offset,
// amplitude from the per-sample SNR, integer delay).
struct SynthTx {
    int64_t delay;              // first sample
    double cycles_per_sample;   // f / Fs
    float amp;                  // sqrt(SNR), noise power 1
    float phase0;               // carrier phase at sample 0, cycles
    uint32_t code;              // chip stream id
    uint32_t pad;
};

// Sample source of the STFT: a device block, or synthetic blocks generated on
// the fly (Philox4x32-10 noise and chips, Box-Muller normals).
struct BlockSource {
    const float2* x;            // device samples of block 0 (x[b * stride + n]) or nullptr
    int64_t stride;
    const SynthTx* tx;          // [block][kMaxTx] when x == nullptr
    const int32_t* ntx;         // [block]
    uint32_t seed_lo, seed_hi;  // generator key
    int64_t block0;             // stream id of block 0
    int32_t chip_len;           // samples per transmission L
    int32_t spc;
};

// Median state of one block for the radix selection over FP32 bit patterns.
struct MedianState {
    uint32_t prefix;
    uint32_t rank;
};

// Scratch of the median: zero before the first launch, left so by every
// launch_median.
constexpr int64_t kMedianDigit = 2048;      // histogram words of one digit
struct MedianScratch {
    uint32_t* hist;             // [blocks][kMedianDigit]
    int32_t blocks;             // histograms held: a call of fewer blocks gives each several copies
    unsigned* tickets;          // [block]
    MedianState* state;         // [block]
};

// Powers P[block][F][256] and the median's first digit; launch_median (on the
// same blocks and scratch) selects the rest.
hipError_t launch_stft(const BlockSource& src, int nblocks, int64_t F, const float* hann, const float2* tw,
                       float* P, const MedianScratch& ms, hipStream_t st);
hipError_t launch_median(const float* P, int nblocks, int64_t per_block, const MedianScratch& ms, float* med,
                         hipStream_t st);
// h_med: block 0's median, to host memory (nullptr: no)
hipError_t launch_map(const float* P, int nblocks, int64_t F, const float* med, void* map, bool bf16,
                      float* h_med, hipStream_t st);
// Samples of synthetic block 0 of `src` (src.x == nullptr) into out[n].
hipError_t launch_synth(const BlockSource& src, int64_t n, float2* out, hipStream_t st);
hipError_t launch_labels(const SynthTx* tx, const int32_t* ntx, int nblocks, int64_t F, int L, float* labels,
                         hipStream_t st);

// Forward of one conv layer: out = relu(conv(in) + b).
hipError_t launch_conv_forward(const void* in, int cin, const void* wt, const float* bias, void* out,
                               int64_t rows, int64_t F, int d, bool bf16, hipStream_t st);
// Input gradient of layer l (cin = 64): dprev[r][c] = sum_i sum_o W[i][c][o] dA[r - d(i-2)][o],
// dA = dH * (H > 0).
hipError_t launch_conv_dinput(const float* dH, const void* H, const void* w, float* dprev, int64_t rows,
                              int64_t F, int d, bool bf16, hipStream_t st);
// Weight and bias gradients of one layer, dW[i][c][o] = sum_r in[r + d(i-2)][c] dA[r][o],
// db[o] = sum_r dA[r][o]: the bf16 form leaves the sums of *chunks row chunks in
// `part` (FP32, at least dweight_part_elems(cin, rows) values, which grow with the rows).
int64_t dweight_part_elems(int cin, int64_t max_rows);
hipError_t launch_conv_dweight(const void* in, int cin, const float* dH, const void* H, float* part,
                               int64_t part_elems, int32_t* chunks, int64_t rows, int64_t F, int d, hipStream_t st);
hipError_t launch_conv_dweight_ref(const float* in, int cin, const float* dH, const float* H, float* dW, float* db,
                                   int64_t rows, int64_t F, int d, hipStream_t st);
// Head logits y[r] = bh + h4[r] . wh; with labels also dH4 = dy wh^T and, of each
// of head_groups(rows) row groups, the sums dwh = h4^T dy, dbh = sum dy and of the
// loss terms: part[kHeadSums][groups].
constexpr int kHeadSums = kCh + 2;
int64_t head_groups(int64_t rows);
hipError_t launch_head(const void* h4, const float* theta, int64_t wh_off, float* y, const float* labels,
                       float pos_weight, float inv_rows, float* dH4, float* part, int64_t rows, bool bf16,
                       hipStream_t st);
// Partial sums added up in a fixed order: the head's and, where part is not null,
// the layers', to grad and, if not null, out; the loss to host memory.
struct GradSums {
    const float* head;
    int64_t head_groups, wh_off;
    const float* part[kLayers];
    int64_t w_off[kLayers];     // of the layer's weights, the bias after them
    int32_t cin[kLayers], nchunks[kLayers];
};
hipError_t launch_grad_reduce(const GradSums& a, float* grad, float* out, float* h_loss, hipStream_t st);
hipError_t launch_adam(float* theta, float* grad, float* m, float* v, int64_t n, float lr, float b1, float b2,
                       float eps, int t, const NetLayout& lay, uint16_t* w_bf, uint16_t* wt_bf, hipStream_t st);
hipError_t launch_fill_f32(float* p, int64_t n, hipStream_t st);
hipError_t launch_fill_u32(uint32_t* p, int64_t n, hipStream_t st);

// Frames of one block whose window score c[f] = sum_{i=-63}^{64} y[f+i] is at or
// above kappa, their lag ranges and the segment list.  h_info (host memory) =
// {proposed frames, segments}.  mask: kProposeWords words, zero before the first
// launch and left so.
constexpr int kMaxSegList = 4096;
constexpr int kProposeWords = kMaxSegList / 32 + 2;
hipError_t launch_propose(const float* y, int64_t F, float kappa, int64_t n, int64_t L, int64_t V,
                          int32_t max_segments, uint32_t* mask, int32_t* segs, int32_t* h_info, hipStream_t st);

}  // namespace learned
}  // namespace acq
