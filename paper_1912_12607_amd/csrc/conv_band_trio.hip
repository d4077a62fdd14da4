// The passes of a layer whose filter bank stays on chip (conv_band.h) in one launch with its backward-weight pass.
//
// Bound: the bands write fp32 results at the rate of HBM and wait for it, backward-weight reads codes that lie in the caches and
// waits for its stages; one after the other, each also ends on its slowest block with the chip half empty.  Backward-weight's blocks
// come first (they live longest: a block of bands that starts late has few of them), two blocks per compute unit as alone.
// Alternating blocks of both kinds from the start was slower (1.003 and 0.972 against 0.917 and 0.928, see conv_band_trio()), and so were
// more, shorter blocks of bands (0.940, 0.951).
#include <algorithm>

#include "conv_band.h"
#include "conv_wgrad_lines.h"
#include "conv_wgrad_tile.h"

namespace int8t {

namespace {
struct BandTrioBlocks {
    unsigned wgrad, wgrad8, fwd, bwd;        // backward-weight's blocks, and rounded up to the 8 XCDs; the forward and backward-data passes'
};
// what a walk needs beside the pass itself
struct BandWalk {
    int BP, nbands_h, nbands;
    BandRegTab tab;
};
// (The LDS body keeps its 12 staging slots.  6 where no window takes more would need ten instantiations more; with 12 / with 6, us for two and three
// passes: 1x1, 24 -> 144, 56 x 56, batch 64: 23.2 49.1, 21.4 48.2; 1x3, 8 -> 16, 109 x 109, batch 26: 19.7 28.2, 18.3 26.0; 1x1, 16 -> 32,
// 112 x 112, batch 64: 38.4 58.0, 36.6 55.8; 5x5, 3x3 and 7x1 on 16, 16 and 8 channels the same.)
template <bool DGRAD, int NKS, int MT>
__device__ __forceinline__ void band_pass(const IgemmArgs& a, const BandWalk& p, int block, int nblocks) {
    if constexpr (NKS > 0) band_reg_walk<DGRAD, NKS>(a, p.BP, p.nbands_h, p.nbands, p.tab, block, nblocks);
    else band_walk<DGRAD, MT, 1, true>(a, p.BP, p.nbands_h, p.nbands, block, nblocks);
}
constexpr int bt_wt(int ST) { return ST == 1 ? 2 : 1; }
constexpr int bt_gp(int ST) { return ST == 1 ? 4 : ST == 5 ? 6 : 8; }
}  // namespace

// NKS > 0: the register-weight body, else the LDS body with MT row tiles; ST: taps along backward-weight's lines, 0: image granules.
template <int NKS, int MT, int ST>
__global__ __launch_bounds__(256, 2) void conv_band_trio_kernel(const IgemmArgs f, const IgemmArgs b, const WgradArgs w, const BandWalk fp,
                                                                const BandWalk bp, const BandTrioBlocks n) {
    const unsigned block = blockIdx.x;
    if (block < n.wgrad8) {
        if (block >= n.wgrad) return;
        if constexpr (ST == 0) wgrad_tile<1, 1>(w, block);
        else wgrad_lines_tile<ST, bt_wt(ST), bt_wt(ST), bt_gp(ST)>(w, block);
    } else if (block < n.wgrad8 + n.fwd) {
        band_pass<false, NKS, MT>(f, fp, (int)(block - n.wgrad8), (int)n.fwd);
    } else {
        band_pass<true, NKS, MT>(b, bp, (int)(block - n.wgrad8 - n.fwd), (int)n.bwd);
    }
}

namespace {
bool band_auto(const IgemmArgs& a, BandPlan* p) {
    return a.variant == VAR_AUTO && a.stride_h == 1 && a.stride_w == 1 && igemm_auto_variant(a) == VAR_BAND && band_plan(a, p) &&
           (p->nks || (p->ntw == 1 && p->uni));
}
bool same_body(const BandPlan& a, const BandPlan& b) { return a.nks == b.nks && (a.nks || a.mt == b.mt); }
// taps along backward-weight's lines, 0: image granules, -1: a form without instantiation
int wgrad_form(const WgradArgs& w) {
    if (w.variant != VAR_AUTO || w.s2d) return -1;
    if (w.lines) return w.stride_h == 1 && w.stride_w == 1 ? w.TB : -1;
    return w.TB == 1 && w.CS == 1 && !w.pk ? 0 : -1;
}
typedef void (*kern_t)(const IgemmArgs, const IgemmArgs, const WgradArgs, const BandWalk, const BandWalk, const BandTrioBlocks);
kern_t band_trio_kernel(int nks, int mt, int st, int* slot) {
    static const struct { int nks, mt, st; kern_t k; } table[] = {
        {2, 0, 0, conv_band_trio_kernel<2, 0, 0>},   {2, 0, 1, conv_band_trio_kernel<2, 0, 1>},   {4, 0, 0, conv_band_trio_kernel<4, 0, 0>},
        {4, 0, 1, conv_band_trio_kernel<4, 0, 1>},   {9, 0, 3, conv_band_trio_kernel<9, 0, 3>},   {18, 0, 3, conv_band_trio_kernel<18, 0, 3>},
        {0, 1, 0, conv_band_trio_kernel<0, 1, 0>},   {0, 1, 1, conv_band_trio_kernel<0, 1, 1>},   {0, 1, 3, conv_band_trio_kernel<0, 1, 3>},
        {0, 1, 5, conv_band_trio_kernel<0, 1, 5>},   {0, 1, 7, conv_band_trio_kernel<0, 1, 7>},   {0, 2, 0, conv_band_trio_kernel<0, 2, 0>},
        {0, 2, 1, conv_band_trio_kernel<0, 2, 1>},   {0, 2, 3, conv_band_trio_kernel<0, 2, 3>},   {0, 2, 5, conv_band_trio_kernel<0, 2, 5>},
        {0, 2, 7, conv_band_trio_kernel<0, 2, 7>}};
    static_assert(sizeof(table) / sizeof(table[0]) <= kBandTrioKernels, "slots");
    for (unsigned i = 0; i < sizeof(table) / sizeof(table[0]); ++i)
        if (table[i].nks == nks && (nks || table[i].mt == mt) && table[i].st == st) {
            *slot = (int)i;
            return table[i].k;
        }
    return nullptr;
}
}  // namespace

// Layers that conv_trio_tile() leaves apart: their bands are walked by resident blocks, which its 128-row tiles cannot match.  Over 60 random
// ones the two backward passes take 0.917 of the time one by one (1.03 at most), the three passes 0.928 (1.06 at most), us for two and
// three passes apart and here:
//   3x3, 64 channels, 56 x 56, batch 64       38.3   59.1     34.4   47.4     1x1, 64 channels, 56 x 56, batch 64      32.4   48.2   22.1   42.2
//   1x1, 24 -> 144, 56 x 56, batch 64         28.7   61.9     24.7   58.1     3x3, 32 channels, 56 x 56, batch 256     75.6  112.4   64.6   95.2
//   3x3, 40 -> 60, 31 x 31, batch 200         38.8   62.8     33.6   57.9     1x3, 8 -> 16, 109 x 109, batch 26        29.7   43.8   23.9   33.3
// With more codes and input gradient than the last-level cache of 256 MB holds beside other data, HBM bounds both kinds of blocks, and side by
// side they share it worse.  Time here over the time apart, 8 to 14 layers with batches that give the stated MB (geometric mean, and the
// worst layer; two sets of buffers in turn):
//   MB             60          120         180         210         240         270         290         340         500
//   two passes   0.94 1.01   0.95 1.09   0.94 1.01   0.93 1.02   0.96 1.11   1.01 1.14   1.04 1.16   1.05 1.17   1.06 1.16
//   three        0.87 1.00   0.91 0.99   0.96 1.01   0.98 1.02   0.99 1.04   1.00 1.09   1.02 1.11   1.03 1.07   1.03 1.09
// (1x1, 64 channels, 56 x 56, two passes, us apart and here: 180 MB 0.85 of the time, 290 MB 83.3, 96.7; 1x1, 64 -> 256 at 56 x 56, 463 MB:
// 142.7, 146.1.)
int conv_band_trio(const IgemmArgs* fwd, const IgemmArgs& bwd, const WgradArgs& w) {
    BandPlan d, f;
    int slot;
    const int st = wgrad_form(w);
    const size_t pixels = (size_t)bwd.N * bwd.OH * bwd.OW;
    if (4 * pixels * bwd.rows + pixels * (size_t)w.Cp + (size_t)w.N * w.P * w.Q * w.Kp > 220000000u) return 0;
    if (st < 0 || !band_auto(bwd, &d) || !band_trio_kernel(d.nks, d.mt, st, &slot)) return 0;
    return fwd && band_auto(*fwd, &f) && same_body(f, d) ? 3 : 2;
}

hipError_t launch_conv_band_trio(const IgemmArgs* fwd, const IgemmArgs& bwd, const WgradArgs& w, hipStream_t st) {
    BandPlan d, f;
    if (!band_plan(bwd, &d)) return hipErrorInvalidValue;
    f = d;
    if (fwd && !band_plan(*fwd, &f)) return hipErrorInvalidValue;
    int slot = 0;
    const kern_t k = band_trio_kernel(d.nks, d.mt, wgrad_form(w), &slot);
    if (!k) return hipErrorInvalidValue;
    BandTrioBlocks n;
    n.wgrad = w.lines ? wgrad_lines_grid(w) : wgrad_grid(w);
    n.wgrad8 = (n.wgrad + 7) & ~7u;
    n.fwd = fwd ? (unsigned)std::min(f.nbands, 512) : 0;
    n.fwd = (n.fwd + 7) & ~7u;         // (backward-data's blocks start on an XCD boundary; blocks without a band do nothing)
    n.bwd = (unsigned)std::min(d.nbands, 512);
    const BandWalk fw{f.BP, f.nbands_h, f.nbands, f.tab}, dw{d.BP, d.nbands_h, d.nbands, d.tab};
    const size_t lds = std::max({d.lds, f.lds, w.lds_bytes});
    static std::atomic<unsigned long long> attr_done[kBandTrioKernels];
    const hipError_t e = raise_dynamic_lds(reinterpret_cast<const void*>(k), (int)BAND_LDS_MAX, attr_done[slot]);
    if (e != hipSuccess) return e;
    {
        KernelTimer kt(KID_CONV_BAND_TRIO, st);
        launch_timed(kt, k, dim3(n.wgrad8 + n.fwd + n.bwd), dim3(256), lds, st, fwd ? *fwd : bwd, bwd, w, fw, dw, n);
    }
    const hipError_t el = hipGetLastError();
    return el != hipSuccess ? el : launch_wgrad_reduce(w, st);
}

}  // namespace int8t
