// Internal launch interface between the C-ABI layer (api.hip) and the kernel files.
// Every launcher enqueues on `st` and returns the hipError_t of its last launch.
#pragma once
#include "profile.h"
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include <atomic>

namespace int8t {

// Raises a kernel's dynamic-LDS limit (the default is 64 KB) the first time it is launched on a
// device; `done` is the call site's own bit mask of the devices already served.
inline hipError_t raise_dynamic_lds(const void* fn, int bytes, std::atomic<unsigned long long>& done) {
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    const unsigned long long bit = 1ull << (dev & 63);
    if (done.load(std::memory_order_acquire) & bit) return hipSuccess;
    e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
    if (e == hipSuccess) done.fetch_or(bit, std::memory_order_release);
    return e;
}


constexpr int kMaxPartials = 1024;   // per-block partial results of an absmax pass
constexpr int kAbsmaxPartials = 256;  // ... of which an absmax pass writes at most this many (its block count)

// Partial sums of Eq.6 left by one block: A = sum g*q, G = sum g^2, B = sum q^2.
struct DevPartial {
    double A;
    double G;
    unsigned long long B;
};

// ---- quantize.hip ---------------------------------------------------------------------------
// max|x| per block -> part[0..nparts); returns the number of partials through *nparts.
// sumsq: nullptr, or kMaxPartials doubles that receive per-block sums of squares; then the pass
// also clears the nzero 64-bit words at zero (the clip search's accumulators and ticket)
hipError_t launch_absmax(const float* x, size_t n, float* part, int* nparts, hipStream_t st, double* sumsq = nullptr,
                         unsigned long long* zero = nullptr, int nzero = 0);

struct QuantArgs {
    const float* x;
    int d0, d1, d2, d3;          // logical dims: N,C,H,W or K,Cg,R,S
    const float* clip;           // device scalar or nullptr (then absmax partials are reduced)
    const float* absmax_part;
    int nparts;
    int stochastic;
    uint64_t seed;
    int8_t* q;
    float* scale;
    DevPartial* devpart;         // nullptr: no deviation
};
// several tensors per launch (round-to-nearest, no deviation output)
constexpr int kMaxBatch = 8;
struct AbsmaxBatchItem {
    const float* x;
    size_t n;
    float* part;                 // this tensor's partials
    int nblocks;                 // its blocks inside the launch
    // the tensor of a clip search (at most one, the last item): its blocks also leave the sums of squares and clear
    // the search's accumulators, as absmax_kernel<true> does
    double* sumsq;
    unsigned long long* zero;
    int nzero;
    // > 0: not a maximum but column sums: x is a matrix of n / cols rows, part receives its `cols` sums (absmax_colsum_blocks() blocks)
    int cols;
};
// The item that holds a block of a batched launch.  The first blocks of all items stand side by side at the front of the kernel's
// arguments (0x7fffffff where there is no item): one load, where walking the items is a chain of them, each a round trip to memory.
template <int COUNT>
__device__ __forceinline__ int batch_item(const int (&block0)[COUNT], int block) {
    int i = 0;
#pragma unroll
    for (int k = 1; k < COUNT; ++k) i += block >= block0[k] ? 1 : 0;
    return i;
}
struct AbsmaxBatch {
    int block0[kMaxBatch + 1];   // first block of every item: batch_item()
    int count;
    AbsmaxBatchItem it[kMaxBatch + 1];
};
struct QuantBatchItem {
    const float* x;
    int d0, d1, d2, d3;
    const float* clip;
    const float* absmax_part;
    int nparts;
    int8_t* q;
    float* scale;
    int kind;                    // 0 activations, 1 weights, 2 planar, 3 activations of at most 4 channels with their space-to-depth codes
    int gx, gy, gz;              // its virtual grid inside the launch
    int stoch;                   // Eq.3 instead of Eq.1
    uint32_t seed_lo, seed_hi;   // seed_key_x(seed), seed_key_a(seed): the draw's two keys
};
struct QuantBatch {
    int block0[kMaxBatch];       // as in AbsmaxBatch
    int count;
    QuantBatchItem it[kMaxBatch];
};
int absmax_blocks(size_t n);
int absmax_colsum_blocks(int cols);
void quant_grid(int kind, const int d[4], int* gx, int* gy, int* gz);
hipError_t launch_absmax_batch(const AbsmaxBatch& b, int total_blocks, hipStream_t st);
// s2d: where an item of kind 3 puts the space-to-depth codes (s2d.hip)
hipError_t launch_quantize_batch(const QuantBatch& b, int total_blocks, hipStream_t st, int8_t* s2d = nullptr);
int quant_blocks_act(int N, int Cp, int HW);
int quant_blocks_planar(size_t n);
int quant_blocks_wgt(int K, int Cg, int R, int S);
hipError_t launch_quantize_act(const QuantArgs& a, hipStream_t st);
hipError_t launch_quantize_planar(const QuantArgs& a, hipStream_t st);
hipError_t launch_quantize_wgt(const QuantArgs& a, hipStream_t st);
hipError_t launch_deviation_finish(const DevPartial* part, int nparts, double* dev_out, hipStream_t st);

// ---- dsgc.hip -------------------------------------------------------------------------------
struct DsgcWs {
    float* absmax_part;          // kMaxPartials floats
    unsigned long long* acc;     // dsgc_acc_words() 64-bit accumulators, then the ticket word; cleared by the absmax pass
    unsigned int* ticket;
    double* partG;               // [kMaxPartials]: per-block sums of g^2 from the absmax pass
};
// 64-bit accumulator words of the sweep: 32 sets x 64 candidates x {sum H*m, sum L*m, sum m^2}
constexpr size_t kDsgcAccWords = (size_t)32 * 64 * 3;
size_t dsgc_acc_words();             // == kDsgcAccWords
hipError_t launch_dsgc(const float* g, size_t n, const float* ratios, int n_cand, int stochastic,
                       uint64_t seed, const DsgcWs& ws, int nparts_absmax, float* clip_out,
                       double* dev_out, double* dev_all_out, hipStream_t st);

// Division by a number the host knows: q = floor(n / d) for 0 <= n < 2^31 as a high product and a shift.  With l = ceil(log2 d) and
// m = floor(2^(31+l) / d) + 1 (below 2^32 for d >= 2), m d exceeds 2^(31+l) by at most 2^l, so n m / 2^(31+l) lies at or above
// n / d by less than n / 2^31 / d < 1 / d.  d = 1: m = 0 stands for it.
struct FastDiv {
    uint32_t m, s;
};
inline FastDiv fast_div(unsigned d) {
    if (d <= 1) return FastDiv{0u, 0u};
    unsigned l = 0;
    while ((1ull << l) < d) ++l;
    return FastDiv{(uint32_t)((1ull << (31 + l)) / d + 1), l - 1};
}
__host__ __device__ __forceinline__ int div_by(int n, const FastDiv& f) {
    return f.m ? (int)((uint32_t)(((unsigned long long)(uint32_t)n * f.m) >> 32) >> f.s) : n;
}

// ---- conv_igemm.hip (dense forward and backward-data) -----------------------------------------
struct IgemmArgs {
    const int8_t* act;           // NHWC codes, channel pitch Ca
    const int8_t* wgt;           // [rows][R][S][Ca]
    const float* sa;
    const float* sb;
    float* out;                  // [N][rows][OH*OW]
    int32_t* acc;                // nullable, same order
    int N, rows, Ca;             // Ca: padded reduction channels (multiple of 16)
    int IH, IW, OH, OW, R, S;
    int stride_h, stride_w, pad_h, pad_w;
    int dgrad;                   // 0: ih = oh*stride + r - pad;  1: ih = (oh + pad - r)/stride
    int C;                       // forward: channels in use (<= Ca); lets the launch recognise a layer for s2d.hip
    int8_t* s2d;                 // nullable scratch of igemm_s2d_bytes() bytes for the rewritten codes
    int s2d_ready;               // those of the input are there already
    int cell;                    // filled by launch_igemm(): 0, or 1 + the only residue class that has taps (cell form, conv_igemm.hip)
    int cls_h, cls_w;            // filled by launch_igemm(): strides of the residue classes a strided backward-data pass splits its pixels into (1 = not split)
    int32_t* partial;            // nullable scratch [ksplit][N][rows][OH*OW] of a split reduction
    size_t partial_bytes;
    int ksplit;                  // filled by launch_igemm(): blocks per output tile along the reduction
    int variant;                 // ConvVariant: VAR_AUTO, or the kernel the caller selected for this layer
    FastDiv by_rtiles, by_image, by_row;     // filled with the grid of the wide tiles: row tiles, columns per image and per image row (pixels, or cells)
    int colrun;                  // filled by launch_igemm(): column tiles an XCD takes in a run, 0 = every eighth tile
    // Quantization fused into the forward pass of a 1 x 1, stride-1, unpadded layer (launch_igemm_fused):
    const float* xf;             // fp32 activations N,C,H,W (act is not read)
    const float* xclip;          // clip value of a, or nullptr: max|a| from xabs_part[0..xabs_nparts)
    const float* xabs_part;
    int xabs_nparts;
    int8_t* xq_out;              // nullable: the codes of a (N,H,W,Ca), written by the first row tile
    float* sx_out;               // the scale of a
};
// Kernel variants of the dense passes (values of INT8T_VARIANT_* in include/int8t.h).
enum ConvVariant : int {
    VAR_AUTO = 0,
    VAR_BAND = 1,          // forward / backward-data: filter bank resident on chip (conv_band.hip)
    VAR_TILE = 2,          // 64/128 x 128 tiles through registers, reduction whole
    VAR_TILE_SPLIT = 3,    // ... reduction split over several blocks per tile
    VAR_WIDE128 = 4,       // 128 x 256 tiles, operands straight into an LDS ring of 3 stages
    VAR_WIDE256 = 5,       // 256 x 256 tiles, ring of 2 stages of 128 reduction bytes
    VAR_WGRAD_FEWER = 6,   // backward-weight: half the reduction shares of the cost model's choice
    VAR_WGRAD_MORE = 7,    // backward-weight: twice as many
    VAR_WGRAD_IMAGES = 8,  // backward-weight: operands of 16 images per pixel, transposed in registers (conv_wgrad.hip)
    VAR_WGRAD_LINES = 9,   // backward-weight: operands of 32 image lines per position, transposing LDS reads (conv_wgrad_lines.hip)
    VAR_WIDE_SQ128 = 10,   // forward / backward-data: 128 x 128 tiles, ring of 3 stages, three blocks per compute unit
    VAR_WIDE_SQ128_DEEP = 11,   // ... 2 stages of 128 reduction bytes, two blocks per compute unit
    VAR_WIDE_128X64 = 12,       // ... 128 x 64 tiles: layers with few columns
    VAR_WIDE_CELLS = 13,        // backward-data under stride 2 x 2: 128 rows x 64 cells of 2 x 2 pixels, the four pixel classes in one block
    VAR_COUNT
};
int igemm_ksplit(const IgemmArgs& a);   // largest split a launch of this layer may use (1 = none): sizes the scratch
// whether `variant` can run this layer (VAR_AUTO always can); resolved = the variant VAR_AUTO stands for
bool igemm_variant_ok(const IgemmArgs& a, int variant);
int igemm_auto_variant(const IgemmArgs& a, bool allow_split = true);   // allow_split: the caller's scratch holds the partial sums of a split reduction
bool igemm_splits(const IgemmArgs& a);   // whether launch_igemm() would run the split reduction on its own choice
// Forward pass of a layer s2d.hip covers: rewrites the geometry and returns the scratch bytes of the
// rewritten input and filter codes (0: does not apply, the geometry is left alone).
size_t igemm_s2d(IgemmArgs* a);
hipError_t launch_igemm(const IgemmArgs& a, hipStream_t st);
// Blocks of the 128 x bn tiles of igemm_dma_tile over a pass that is not split by pixel classes (0: it is); fills what
// launch_igemm() would.
unsigned igemm_plain_blocks(IgemmArgs* a, int bm, int bn);
// Forms of a strided backward-data pass on 128 x 64 tiles, and the one the pass takes by itself; fills the geometry, returns the blocks
enum StridedForm { STRIDED_PLAIN, STRIDED_CLASSES, STRIDED_CELL, STRIDED_CELLS };
unsigned igemm_strided_blocks(IgemmArgs* a, int* form);
// forward pass that quantizes fp32 activations in its load path; 1 x 1 filter, stride 1, no padding
hipError_t launch_igemm_fused(const IgemmArgs& a, hipStream_t st);
// conv_band.hip: LDS-resident variant for small filter banks; false = shape not covered
// (dry_run: only say whether the shape is covered, launch nothing)
bool launch_band(const IgemmArgs& a, hipStream_t st, hipError_t* err, bool dry_run = false);

// ---- s2d.hip ----------------------------------------------------------------------------------
// A stride-2 layer with at most 4 input channels (the stem of an image network) as the stride-1
// layer on the space-to-depth image: pixel (h', w') holds the 2 x 2 block of pixels (2h' + dy,
// 2w' + dx) as channel (2 dy + dx) * C + c.  Input row 2p + r - pad = 2 (p + r' - ph) + dy with
// ph = ceil(pad / 2) and r = 2 r' + dy - eh, eh = 2 ph - pad: the R x S filter becomes a
// ceil((R+eh)/2) x ceil((S+ew)/2) one whose taps outside the original filter are zero.  The 16-byte
// pixel granule then carries 4 C channels instead of C, and the taps shrink fourfold.  The output
// pixels stay the same.  An odd image gets a last block row / column whose missing pixels are zero, as
// the padding around the image is.
struct S2dGeo {
    int ph, pw, eh, ew, R2, S2;
};
inline bool s2d_applies(int C, int stride_h, int stride_w) { return stride_h == 2 && stride_w == 2 && C <= 4; }
inline S2dGeo s2d_geometry(int R, int S, int pad_h, int pad_w) {
    S2dGeo g;
    g.ph = (pad_h + 1) / 2;
    g.pw = (pad_w + 1) / 2;
    g.eh = 2 * g.ph - pad_h;
    g.ew = 2 * g.pw - pad_w;
    g.R2 = (R + g.eh + 1) / 2;
    g.S2 = (S + g.ew + 1) / 2;
    return g;
}
// input codes [N][H][W][16] -> [N][ceil(H/2)][ceil(W/2)][16] and, unless w is nullptr, filter codes [K][R][S][16] -> [K][R2][S2][16]
hipError_t launch_s2d_repack(const int8_t* x, int8_t* xs, int N, int H, int W, int C, const int8_t* w, int8_t* ws, int K, int R, int S,
                             const S2dGeo& g, hipStream_t st);

// ---- conv_wgrad.hip (dense backward-weight) ---------------------------------------------------
struct WgradArgs {
    const int8_t* x;             // NHWC codes of a, pitch Cp
    const int8_t* dy;            // NHWC codes of g_z, pitch Kp
    const float* sa;
    const float* sb;
    float* dw;                   // [K][C][R][S]
    int32_t* acc;                // nullable
    int32_t* partial;            // scratch [splits][ceil(K / 4)][R*S*Cp][4 filters]
    int N, C, Cp, H, W, K, Kp, P, Q, R, S;
    int stride_h, stride_w, pad_h, pad_w;
    // filled by wgrad_plan():
    int TB, CS;                  // taps per block, 32-channel slabs per wave
    int pk;                      // 1: a tensor of 16 channels, four taps per block packed side by side into the 64 columns
    int BP, BQ, ntp, ntq;        // output-pixel tile and tiles per image
    int ngrp, chunks, splits;    // groups of 16 images, reduction chunks, split-K factor
    int ktiles, ctiles, tapgroups;
    int xt_slots;                // 16-byte granules of the staged input window
    FastDiv by_tiles, by_taps, by_ctiles, by_splits, by_lines;     // image lines: output tiles (of a patch), tap groups, channel tiles (of a patch), splits, lines per image
    size_t lds_bytes;
    // set by the caller, who knows the buffers: one share on image lines, whose tiles are written as the result (dw and acc overlap nothing the pass reads)
    int direct;
    // filled by wgrad_s2d() when it rewrites the geometry above into the space-to-depth form:
    int s2d;                     // 1: C, Cp, H, W, R, S, strides and pads describe the rewritten problem
    int oC, oR, oS, oH, oW, eh, ew;   // the layer's own channels, filter and image; tap r = 2 r' + dy - eh, s = 2 s' + dx - ew
    int8_t* xs;                  // scratch: the input codes in space-to-depth form, [N][H][W][16]
    int xs_ready;                // they are there already (the forward pass made them)
    int variant;                 // VAR_AUTO or a VAR_WGRAD_*: set before wgrad_plan()
    int lines;                   // filled by wgrad_plan(): 1 = wgrad_lines_kernel runs (TB = taps along the line)
    int xgk, xgc;                // ... and its patches of output tiles per XCD: xgk x xgc = 8, or 0 0: tiles dealt by share
    float t_chunk, t_partial;    // ... and its estimates, us: a chunk of a share, a share's partial tiles
};
// Rewrites the geometry into the space-to-depth form (s2d.hip) when it applies.  Returns the bytes of
// the rewritten input codes (0: does not apply, the geometry is left alone).  Call before wgrad_plan().
size_t wgrad_s2d(WgradArgs* a);
void wgrad_plan(WgradArgs* a);   // needs the geometry fields above the first comment
hipError_t launch_wgrad(const WgradArgs& a, hipStream_t st);
hipError_t launch_wgrad_reduce(const WgradArgs& a, hipStream_t st);     // its second launch: the shares' partial tiles -> dw
// conv_wgrad_lines.hip: the kernel for stride-1 filters with 1, 3, 5 or 7 taps along an image axis
bool wgrad_lines_applies(const WgradArgs& a);    // geometry as wgrad_plan() takes it (after wgrad_s2d())
// lines are image rows and the taps of a block run along W (else: columns, along H)
__host__ __device__ inline bool wgrad_lines_along_w(int R, int S) { return S > 1 || R == 1; }
void wgrad_plan_lines(WgradArgs* a);
hipError_t launch_wgrad_lines(const WgradArgs& a, hipStream_t st);
unsigned wgrad_grid(const WgradArgs& a);         // blocks of wgrad_kernel
unsigned wgrad_lines_grid(const WgradArgs& a);
bool wgrad_lines_s2(const WgradArgs& a);         // the stride-2 form: 3x3 filters, stride 2 x 2
// Partial tiles of the shares: four filters side by side, which a lane of a matrix product holds in four neighbouring registers (one 16-byte
// store instead of four of 4 bytes: the address path of a compute unit takes 16 cycles for either.  us for the pass, channel by
// channel / so: 7x1, 160 -> 192, 17 x 17, batch 64: 23.3, 19.7; 3x3, 96 channels, 35 x 35, batch 32: 18.1, 16.5; 3x3, 64 channels, 56 x 56, batch 64: 21.5, 20.2; 1x1, 1024 -> 256, 14 x 14, batch 128: 26.3, 25.1).
__host__ __device__ inline size_t wgrad_partial_elems(const WgradArgs& a) { return (size_t)((a.K + 3) / 4 * 4) * a.R * a.S * a.Cp; }      // of one share
inline size_t wgrad_partial_bytes(const WgradArgs& a) { return (a.splits * wgrad_partial_elems(a) * 4 + 255) & ~(size_t)255; }

// Whether the pass runs as one share on image lines, in the layer's own geometry, and its tiles are better written as the result
// (WgradArgs::direct) than reduced: neighbouring lanes then store R S floats apart, the taps along the line as a run, where a reduction writes
// whole filters but takes a launch.  us, as the result / with the reduction:
//   3x3   64 -> 64 (0.15 MB of weights) 6.6, 8.9   640 -> 384 (8.8 MB) 12.7, 14.7
//   5x5   33 -> 48 (0.16 MB) 7.5, 8.8   40 -> 64 (0.26 MB) 9.3, 8.7   64 -> 64 (0.4 MB) 12.7, 8.6   256 -> 128 (3.3 MB) 15.8, 13.8   320 -> 256 (8.2 MB) 22.1, 24.0
//   7x7   16 -> 64 (0.2 MB) 7.9, 9.1    33 -> 48 (0.31 MB) 10.0, 9.3    64 -> 64 (0.8 MB) 18.7, 10.0   256 -> 128 (6.4 MB) 22.3, 14.4   640 -> 384 (48 MB) 69.5, 50.5
inline bool wgrad_single_share(const WgradArgs& a) {
    const int RS = a.R * a.S;
    const long long bytes = 4ll * RS * a.C * a.K;
    return a.lines && !a.s2d && a.splits == 1 && (RS <= 9 || bytes <= 200000 || (RS <= 25 && bytes >= 6000000));
}

// which kernel VAR_AUTO stands for: true = wgrad_lines_kernel
bool wgrad_auto_lines(const WgradArgs& a);
// Share z runs on XCD z mod 8 with all its output tiles (they read the same lines of both tensors, and every XCD fills
// its own L2) when the shares go round the XCDs evenly enough: the grid holds a multiple of 8 shares, the extra ones
// exit at once, and the XCDs with one share more take 8 / splits longer (at most 1/7 here).  Without it the tiles of a
// share land on all 8 XCDs and each L2 fetches the share's lines again (256 x 128 -> 128 3x3 at 28 x 28: 68 -> 47 us).
__host__ __device__ inline bool wgrad_xcd_mapping(int splits) {
    return splits >= 8 && (((splits + 7) & ~7) - splits) * 7 <= splits;
}

// ---- conv_trio.hip (the three dense passes of a layer in one launch) ---------------------------
// Column width of the implicit-GEMM tiles with which the passes share a launch, 0: they run one by one.  w: after wgrad_plan();
// fwd: nullptr where only the two backward passes run.
struct TrioTile {
    int bn;          // columns of the 128-row tiles, 0: the passes run one by one
    bool rows64;     // 64 x 128 tiles for the passes of at most 64 rows
};
TrioTile conv_trio_tile(const IgemmArgs* fwd, const IgemmArgs& bwd, const WgradArgs& w);
bool conv_trio_fwd_apart(const IgemmArgs& fwd, const IgemmArgs& bwd);    // the forward pass is better launched ahead, by itself
hipError_t launch_conv_trio(const IgemmArgs* fwd, const IgemmArgs& bwd, const WgradArgs& w, TrioTile tile, hipStream_t st);

// The same for passes whose filter bank stays on chip (conv_band_trio.hip): 0: they run one by one; 2: the two backward passes
// share a launch, the forward pass (if any) runs ahead; 3: all three
int conv_band_trio(const IgemmArgs* fwd, const IgemmArgs& bwd, const WgradArgs& w);
hipError_t launch_conv_band_trio(const IgemmArgs* fwd, const IgemmArgs& bwd, const WgradArgs& w, hipStream_t st);
constexpr int kBandTrioKernels = 16;

bool conv_trio_strided(const IgemmArgs* fwd, const IgemmArgs& bwd, const WgradArgs& w);      // whether the passes of a strided layer share one
hipError_t launch_conv_trio_strided(const IgemmArgs* fwd, const IgemmArgs& bwd, const WgradArgs& w, hipStream_t st);

// ---- conv_infer.hip (1x1 forward pass from the fp32 tensors, no codes written) -----------------
struct InferArgs {
    const float *x, *w;
    const float *part_x, *part_w;    // absmax partials of a and W
    int np_x, np_w;
    float* y;
    int N, C, K, HW;
    int tiles_img, tiles;            // tiles of 128 pixels, launch_infer_1x1()
};
bool infer_1x1_applies(const InferArgs& a);
hipError_t launch_infer_1x1(const InferArgs& a, hipStream_t st);

// ---- conv_dw.hip (depthwise, planar codes) ----------------------------------------------------
struct DwArgs {
    const int8_t* a;             // planar codes, input of the gather ([N][C][IH][IW])
    const int8_t* b;             // fwd/bwd-data: weights [C][R][S]; bwd-weight: dy codes [N][C][P][Q]
    const float* sa;
    const float* sb;
    float* out;
    int32_t* acc;                // nullable
    int32_t* partial;            // bwd-weight scratch [chunks][C*R*S]
    int chunks;                  // bwd-weight: shares of the batch, dw_wgrad_shape()
    int threads;                 // bwd-weight: block size, dw_wgrad_shape()
    int cg;                      // bwd-weight: consecutive channels per block (1: a block per channel), dw_wgrad_shape()
    int N, C, IH, IW, OH, OW, R, S;
    int stride_h, stride_w, pad_h, pad_w;
    int dgrad;
};
// conv_dw_fused.hip: quantization and convolutions of a 3x3 depthwise layer, from the fp32 tensors (x: codes of a and W and the
// forward pass; g: codes of g_z and the backward passes; either may be nullptr, the codes are inputs then)
struct DwFused {
    const float *x, *w, *g;
    int8_t *xq, *wq, *gq;
    const float *part_x, *part_w;    // absmax partials of a and W
    int np_x, np_w;
    const float* clip;               // of g_z
    uint32_t key_x, key_a;
    float *sx, *sw, *sg;
    float *y, *dx;
    int32_t *y_acc, *dx_acc;         // nullable
    int32_t* partial;                // [shares][C][9]
    int N, C, H, W;
    int cg, slot, shares, pitch;     // launch shape, launch_dw_fused()
};
int dw_threads(int OH, int OW, bool quads);       // block size by plane size (quads: four results per task)
int dw_wgrad_threads(int P, int Q, int R, int S, int stride_h, int stride_w);
int dw_wgrad_chunks(int N, int C, int threads);
// launch shape of the depthwise backward-weight pass (its scratch is chunks * C * R * S int32)
void dw_wgrad_shape(int N, int C, int IH, int IW, int P, int Q, int R, int S, int stride_h, int stride_w,
                    int* threads, int* chunks, int* cg);
hipError_t launch_dw_conv(const DwArgs& a, hipStream_t st);
hipError_t launch_dw_wgrad(const DwArgs& a, hipStream_t st);
hipError_t launch_dw_wgrad_reduce(const DwArgs& a, hipStream_t st);
// whether a 3x3 layer under stride 1 and "same" padding is one for it; launch: false, nothing launched, where it is not
bool dw_fused_applies(int H, int W, const DwArgs& wgrad);
bool launch_dw_fused(const DwFused& a, const DwArgs& wgrad, hipStream_t st, hipError_t* err);
// the three passes of a layer (fwd: nullptr where only the two backward ones run) in one launch; false: not a layer for it,
// nothing launched
bool dw_trio_applies(const DwArgs& pass, const DwArgs& wgrad);
bool launch_dw_trio(const DwArgs* fwd, const DwArgs& bwd, const DwArgs& wgrad, hipStream_t st, hipError_t* err);

}  // namespace int8t
