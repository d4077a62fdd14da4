// The implicit-GEMM tile whose operands are fetched by buffer loads straight into LDS, and the residue classes of a strided
// backward-data pass: shared by the kernels that run it alone (conv_igemm.hip) and beside other passes (conv_trio.hip).
#pragma once
#include "device_common.h"
#include "kernels.h"
#include "lds_dma.h"

namespace int8t {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v16i __attribute__((ext_vector_type(16)));

// Strided backward-data by residue classes.  The input pixels (h, w) with h % stride_h == ch and
// w % stride_w == cw all receive the same filter taps: r = r0 + stride_h * tr, s = s0 + stride_w * ts,
// and for pixel h = ch + stride_h * i the tap tr reads gradient row i + bh - tr.  In the class's own
// coordinates (i, j, tr, ts) that is a stride-1 backward-data pass over nr x ns taps, so a tile whose
// columns are pixels of ONE class spends no matrix-core work on the taps that never reach it (a
// tile of neighbouring pixels multiplies stride_h * stride_w - 1 zeros for every useful product).
// A class without taps (1x1 filter, stride 2: three pixels in four) gets zeros.
struct DgradClass {
    int ch, cw;        // residues of the class
    int OHc, OWc;      // pixels of the class per image: rows, columns
    int r0, s0, nr, ns;
    int bh, bw;
};
// CS: the strides, where they are known to be CS x CS.
template <int CS = 0>
__device__ __forceinline__ DgradClass dgrad_class(const IgemmArgs& a, int cls) {
    DgradClass c;
    const int csh = CS ? CS : a.cls_h, csw = CS ? CS : a.cls_w;     // the stride, or 1 where that direction is not split
    c.ch = cls / csw;
    c.cw = cls - c.ch * csw;
    c.OHc = (a.OH - c.ch + csh - 1) / csh;
    c.OWc = (a.OW - c.cw + csw - 1) / csw;
    c.r0 = (c.ch + a.pad_h) % csh;
    c.s0 = (c.cw + a.pad_w) % csw;
    c.nr = c.r0 < a.R ? (a.R - c.r0 + csh - 1) / csh : 0;
    c.ns = c.s0 < a.S ? (a.S - c.s0 + csw - 1) / csw : 0;
    c.bh = (c.ch + a.pad_h - c.r0) / csh;
    c.bw = (c.cw + a.pad_w - c.s0) / csw;
    return c;
}

// When only ONE class has taps (a 1x1 filter under a stride) the other pixels are zero, and the pass
// is bound by writing them.  "Cell" form (CELL, stride 2 x 2 and an even row length): the columns are
// the 2 x 2 cells of pixels, the tile runs the one class's taps, and the epilogue writes each cell
// whole -- the value at the class's pixel, zeros around it -- as two 8-byte stores, so that a lane
// stores neighbouring floats and a wave whole cache lines.  T = float (result) or int (partial sums,
// accumulators); `o` is the cell's top left element (even: 8-byte aligned).
template <typename T, typename T2>
__device__ __forceinline__ void store_cell(T* __restrict__ dst, size_t o, int OW, bool second_row, int ch, int cw, T v) {
    const T z = (T)0;
    T2 top, bot;
    top.x = (ch == 0 && cw == 0) ? v : z;
    top.y = (ch == 0 && cw == 1) ? v : z;
    bot.x = (ch == 1 && cw == 0) ? v : z;
    bot.y = (ch == 1 && cw == 1) ? v : z;
    *reinterpret_cast<T2*>(dst + o) = top;
    if (second_row) *reinterpret_cast<T2*>(dst + o + OW) = bot;
}

// ---------------------------------------------------------------------------------------------
// Wide-tile variants for the layers bound by the matrix cores: (64*WM) rows x 256 columns per
// block of 2*WM waves (each 64 x 128), operands fetched by buffer loads that write straight into
// LDS (no staging registers), NSTAGE LDS buffers in a ring with the loads running NSTAGE-1 stages
// ahead of the MFMAs, one barrier per stage.  A stage is KG 16-byte granules of the reduction per
// row: KG = 8 makes every row's share of a stage one full 128-byte cache line.  A wave-wide load
// fills 64 consecutive 16-byte slots, lane l the slot base + l; which (row, granule) that slot
// holds follows from the slot index, so each lane simply fetches the granule that belongs there.
// Out-of-range rows, ragged columns, padding taps and the reduction tail carry an offset beyond the
// buffer descriptor: the hardware then writes zeros.
//   <WM=2, KG=4, NSTAGE=3>: 128 x 256, 72 KB of LDS, two blocks per compute unit
//   <WM=4, KG=8, NSTAGE=2>: 256 x 256, 128 KB of LDS, one block of eight waves per compute unit
//   <WM=2, KG=4, NSTAGE=3, BNT=128>: 128 x 128 (waves of 64 x 64), 48 KB of LDS, three blocks per compute unit: for
//   layers whose larger tiles would leave most compute units without one
//   <WM=2, KG=8, NSTAGE=2, BNT=128>: the same tile with 128-byte stages (64 KB, two blocks): half the barriers per MFMA,
//   better where the reduction is long
//   <WM=2, KG=8, NSTAGE=2, BNT=64>: 128 x 64 (waves of 64 x 32), 48 KB: twice the tiles for layers with few columns
//   (7 x 7 and 8 x 8 images), which otherwise leave more than half of the compute units idle
// ---------------------------------------------------------------------------------------------
// What a stage of 128 bytes costs, us, by the times of 1x1 passes of 128 filters on 512 to 4096 channels (4 to 32 stages), before the offsets
// were worked out a stage ahead and operands and loads took turns / so: 128 x 64 tile with 32 blocks 0.46, 0.32, with 256 blocks 0.62, 0.57;
// 128 x 128 tile with 16 and 128 blocks 0.67, 0.45 and 0.76, 0.61.  (The matrix products of a stage, 8 and 16 of 32 cycles per wave, are 0.11 and
// 0.21 us at 2.4 GHz; the rest is the chain of loads, operand reads and the barrier.)  us per pass alone: 3x3, 256 channels, 14 x 14,
// batch 64: 17.7 -> 15.6; 1x1, 1024 -> 256, 14 x 14, batch 128, forward 16.5 -> 14.7; fully connected 2048 -> 1000, batch 256, forward
// 14.7 -> 11.5; 3x3 under stride 2, 128 channels, 56 x 56, backward-data 35.1 -> 33.0.  Over 620 forward and backward-data passes of random layers 0.94 of the
// time: 0.87 - 0.93 where the channels are whole stages; elsewhere 0.93 - 0.95 up to two blocks per compute unit and 0.97 - 1.0 above, where the arithmetic
// of the lanes and loads of two half lines per pixel bound (3x3, 850 -> 1024, 12 x 12, batch 32, 576 tiles: 65, 78; the others 1.13 at most).  Dealing
// the loads out between the products gains 2 - 3 % there and costs 3 % below two blocks per compute unit.
//   ALLC (with CLS and CELL, stride 2 x 2, every class with taps): the columns are the 2 x 2 cells of pixels and the
//   block runs the four classes one after the other, each into accumulators of its own, then writes every cell
//   whole -- two neighbouring floats per lane and image row, whole cache lines per wave -- where the per-class
//   form writes every other float of a line from four different blocks and pays a block's fixed cost per class.
//   STG (plain forms, planes of whole 16-byte groups): the results leave through LDS, see the epilogue.
//   NWN: waves along the columns.  4 with WM = 1: 64 x 128 tiles for passes of at most 64 rows.
template <bool DGRAD, int WM, int KG, int NSTAGE, bool CLS = false, bool CELL = false, int BNT = IGD_BN, bool ALLC = false, bool STG = false, int NWN = 2>
__device__ __forceinline__ void igemm_dma_tile(const IgemmArgs& a, const unsigned block) {
    static_assert(!STG || (!CLS && WM * NWN == 4), "staged results: plain forms of the tiles of four waves");
    static_assert(DGRAD || !CLS, "residue classes exist in the backward-data pass only");
    static_assert(CLS || !CELL, "the cell form is a residue-class form");
    static_assert(!ALLC || (CLS && CELL && BNT == 64), "all classes per block: cell columns, 64 of them");
    constexpr int BM = 64 * WM, BN = BNT, CW = BN / NWN, MI = 2, NJ = CW / 32, NW = NWN * WM;      // CW: columns of a wave
    constexpr int NC = ALLC ? 4 : 1;                    // classes a block runs
    constexpr int STAGE_SLOTS = (BM + BN) * KG;         // 16-byte slots per stage: A tile, then B tile
    constexpr int RPL = 64 / KG;                        // tile rows covered by one wave-wide load
    constexpr int NLA = BM * KG / 64 / NW;              // A loads per wave and stage
    constexpr int NLB = BN * KG / 64 / NW;              // B loads per wave and stage
    constexpr int NL = NLA + NLB;
    static_assert(NSTAGE == 2 || NL == 6 || NL == 4, "vmcnt waits below are written for these");
    extern __shared__ __attribute__((aligned(16))) uint4 ring[];   // [NSTAGE][STAGE_SLOTS]
    raise_wave_priority();

    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = tid >> 6;
    const int wm = wave % WM, wn = wave / WM;

    const int OHWfull = a.OH * a.OW;
    const int Cg16 = a.Ca >> 4;
    const int gfull = a.R * a.S * Cg16;
    // Workgroups are dealt to the 8 XCDs round-robin (workgroup b runs on XCD b % 8).  Column tile
    // ct = 8 * (i / rtiles) + xcd, row tile i % rtiles, i = b / 8: all row tiles of a column tile --
    // they read the same pixels -- run on one XCD and share its L2, as do the column tiles of an XCD
    // that read the same filter rows.  The grid is padded to whole groups of 8 column tiles.
    // CLS: the residue classes of a column tile follow each other on the same XCD as well (they read
    // the same gradient pixels and write interleaved floats of the same cache lines).
    const int rtiles = (a.rows + BM - 1) / BM;
    const int wg_i = (int)(block >> 3);
    const int row_group = div_by(wg_i, a.by_rtiles);
    int cgroup = row_group;
    DgradClass dc;
    if (CLS) {
        if (CELL) {
            dc = dgrad_class<ALLC ? 2 : 0>(a, ALLC ? 0 : a.cell - 1);
            dc.OHc = (a.OH + a.cls_h - 1) / a.cls_h;      // cells, not pixels of the class
            dc.OWc = (a.OW + a.cls_w - 1) / a.cls_w;
        } else {
            const int ncls = a.cls_h * a.cls_w;
            const int g = cgroup / ncls;
            dc = dgrad_class(a, cgroup - g * ncls);
            cgroup = g;
        }
    }
    const int OWc = CLS ? dc.OWc : a.OW;
    const int OHW = CLS ? dc.OHc * dc.OWc : OHWfull;     // columns per image
    const int ncols = a.N * OHW;
    // (a class's columns are known here only)
    auto image_of = [&](int col) { return CLS && !CELL ? col / OHW : div_by(col, a.by_image); };
    auto row_of = [&](int pix) { return CLS && !CELL ? pix / OWc : div_by(pix, a.by_row); };
    int nr = CLS ? dc.nr : a.R, ns = CLS ? dc.ns : a.S;  // (ALLC: of the class being run)
    int gtot = nr * ns * Cg16;
    int nsteps = (gtot + KG - 1) / KG;
    // colrun (igemm_colrun): an XCD takes a run of column tiles instead of every eighth.
    const int ctile = a.colrun ? (int)(block & 7) * a.colrun + cgroup : (cgroup << 3) + (int)(block & 7);
    if (ctile * BN >= ncols) return;
    const int rowbase = (wg_i - row_group * rtiles) * BM;
    const int colbase = ctile * BN;

    const v4i wr = igd_rsrc(a.wgt, (uint32_t)((size_t)a.rows * gfull * 16));
    const v4i xr = igd_rsrc(a.act, (uint32_t)((size_t)a.N * a.IH * a.IW * a.Ca));
    // LDS byte address of this wave's first A / B load slot in buffer 0 (wave-uniform)
    const uint32_t lds_a0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(size_t)(ring + 64 * wave));
    const uint32_t lds_b0 = lds_a0 + BM * KG * 16;

    // ---- loader state: this wave issues A loads {wave + NW*i} and B loads {wave + NW*i}.  Load
    // number wl covers tile rows RPL*wl .. RPL*wl + RPL-1; lane -> (row, granule) through the swizzle.
    const int lrow = lane / KG;                              // row inside the load's row group
    // granule held by this lane's slot: the inverse of igd_slot().  KG = 4: a load covers 16 rows from a
    // multiple of 16, bits 2..3 of the row are those of lrow.  KG = 8: a load covers 8 rows from
    // 8 * (wave + NW * i); with NW even, bit 3 of the row is the wave's parity for every i.
    static_assert(KG == 4 || (NW & 1) == 0, "the swizzle of the 8-granule tile needs an even wave count");
    const int gsw = KG == 4 ? ((lane & 3) ^ ((lrow >> 2) & 3)) : ((lane & 7) ^ (((lrow >> 1) & 3) | ((wave & 1) << 2)));
    uint32_t aoff[NLA];                                      // byte offset of (row, granule 0) or OOB
#pragma unroll
    for (int i = 0; i < NLA; ++i) {
        const int row = rowbase + RPL * (wave + NW * i) + lrow;
        aoff[i] = row < a.rows ? (uint32_t)row * (uint32_t)gfull * 16u : IGD_OOB;
    }
    int bh[NLB], bw[NLB];                                    // a column beyond the last: a row that no tap brings inside the image
    int boh[NLB], bow[NLB];                                  // (ALLC) the column's cell, to which each class adds its offset
    uint32_t bimg[NLB];                                      // byte offset of the column's image
    uint32_t bbase[NLB];                                     // ... of the pixel that tap (0,0) reads, modulo 2^32 (it may lie outside the image)
    constexpr int kFar = 0x40000000;
    // byte offset of pixel (y, x) in an image, modulo 2^32: y may be kFar, whose offset nothing uses
    auto pixel = [&](int y, int x) { return ((uint32_t)y * (uint32_t)a.IW + (uint32_t)x) * (uint32_t)a.Ca; };
#pragma unroll
    for (int i = 0; i < NLB; ++i) {
        const int col = colbase + RPL * (wave + NW * i) + lrow;
        const bool cv = col < ncols;
        const int cc = cv ? col : 0;
        const int n = image_of(cc), rem = cc - n * OHW;
        const int oh = row_of(rem), ow = rem - oh * OWc;
        boh[i] = cv ? oh : kFar;
        bow[i] = ow;
        bh[i] = cv ? (CLS ? oh + dc.bh : DGRAD ? oh + a.pad_h : oh * a.stride_h - a.pad_h) : kFar;
        bw[i] = CLS ? (ow + dc.bw) : DGRAD ? (ow + a.pad_w) : (ow * a.stride_w - a.pad_w);
        bimg[i] = (uint32_t)n * (uint32_t)(a.IH * a.IW * a.Ca);
        bbase[i] = bimg[i] + pixel(bh[i], bw[i]);
    }
    // a direction split into classes is a stride-1 pass; otherwise only the taps that divide reach a pixel
    const int dsh = CLS ? a.stride_h / a.cls_h : a.stride_h, dsw = CLS ? a.stride_w / a.cls_w : a.stride_w;
    const bool unit = !DGRAD || (dsh == 1 && dsw == 1);
    // Where the channels are whole stages, all lanes of a stage are at one filter tap: the position in the reduction is then the same for
    // all of them and kept in scalar registers, the loads add it to offsets that stay (A) or change with the tap (B).
    // (Not with ALLC: four copies of the loop, each run once or twice per block, wait for their instructions.)
    const bool uni = !ALLC && Cg16 % KG == 0;
    // Offsets of the next stage's loads, worked out a stage ahead: their arithmetic runs beside the matrix instructions, and no lane branches.
    uint32_t na[NLA], nb[NLB];
    uint32_t soff_a = 0, soff_b = 0;
    auto tap_b = [&](int r, int s, uint32_t tapoff, int cg, uint32_t past) {       // nb: granule cg of this lane's pixels under tap (r,s)
#pragma unroll
        for (int i = 0; i < NLB; ++i) {
            bool ok;
            uint32_t off;
            if (unit) {
                const int ih = DGRAD ? bh[i] - r : bh[i] + r, iw = DGRAD ? bw[i] - s : bw[i] + s;
                ok = ((unsigned)ih < (unsigned)a.IH) & ((unsigned)iw < (unsigned)a.IW);
                off = bbase[i] + tapoff;
            } else {
                const int th = bh[i] - r, tw = bw[i] - s;
                const int ih = th / dsh, iw = tw / dsw;
                ok = (th >= 0) & (tw >= 0) & (ih * dsh == th) & (iw * dsw == tw) & ((unsigned)ih < (unsigned)a.IH) & ((unsigned)iw < (unsigned)a.IW);
                ok = ok & (bh[i] < kFar);
                off = bimg[i] + pixel(ih, iw) + (uint32_t)(cg * 16);
            }
            nb[i] = (ok ? off : IGD_OOB) | past;
        }
    };
    // granule of the filter row: the taps of a class are a sub-grid of the R x S filter
    auto filter_granule = [&](int r, int s, int cg, int q) { return CLS ? ((dc.r0 + a.cls_h * r) * a.S + dc.s0 + a.cls_w * s) * Cg16 + cg : q; };
    // position of the next stage: filter tap (r,s), channel granule cg, granule index q in the reduction, byte offset from tap (0,0)'s pixel
    int r, s, cg, q;                                         // of this lane
    int ur = 0, us = 0, ucg = 0, uq = 0;                     // uni: of the stage's first granule
    uint32_t tapoff, utap = 0;
    auto lane_offsets = [&]() {
        const uint32_t past = q < gtot ? 0u : IGD_OOB;       // beyond the reduction: nothing is read
        const uint32_t wq = (uint32_t)filter_granule(r, s, cg, q) * 16u;
#pragma unroll
        for (int i = 0; i < NLA; ++i) na[i] = (aoff[i] + wq) | past;      // (a row beyond the last: from 2^31 on)
        tap_b(r, s, tapoff, cg, past);
    };
    auto first_stage = [&]() {
        if (uni) {
            ur = us = ucg = uq = 0;
            utap = 0;
            soff_b = 0;
            soff_a = (uint32_t)filter_granule(0, 0, 0, 0) * 16u;
#pragma unroll
            for (int i = 0; i < NLA; ++i) na[i] = aoff[i] + (uint32_t)(gsw * 16);
            tap_b(0, 0, (uint32_t)(gsw * 16), gsw, 0u);
        } else {
            const int tap = gsw / Cg16;
            cg = gsw - tap * Cg16;
            r = tap / (ns > 0 ? ns : 1);
            s = tap - r * ns;
            q = gsw;
            tapoff = (DGRAD ? 0u - pixel(r, s) : pixel(r, s)) + (uint32_t)(cg * 16);
            lane_offsets();
        }
    };
    auto next_stage = [&]() {
        // (forward: a tap's first granule follows the last one of the tap before it)
        const uint32_t over_row = (uint32_t)((DGRAD ? ns - a.IW : a.IW - ns) * a.Ca);
        if (uni) {
            uq += KG;
            ucg += KG;
            soff_b += KG * 16;
            if (ucg == Cg16) {
                ucg = 0;
                soff_b = 0;
                utap += DGRAD ? 0u - (uint32_t)a.Ca : (uint32_t)a.Ca;
                if (++us == ns) {
                    us = 0;
                    ++ur;
                    utap += over_row;
                }
                tap_b(ur, us, utap + (uint32_t)(gsw * 16), gsw, 0u);
            }
            soff_a = (uint32_t)filter_granule(ur, us, ucg, uq) * 16u;
        } else {
            q += KG;
            cg += KG;
            tapoff += KG * 16;
            auto next_tap = [&](bool wrap) {
                cg -= wrap ? Cg16 : 0;
                s += wrap ? 1 : 0;
                const bool row = s == ns;
                s = row ? 0 : s;
                r += row ? 1 : 0;
                if (DGRAD) tapoff -= wrap ? 2u * (uint32_t)a.Ca : 0u;
                tapoff += row ? over_row : 0u;
            };
            if (Cg16 >= KG) {
                next_tap(cg >= Cg16);
            } else {
#pragma unroll 1
                for (int left = KG; left > 0; left -= Cg16) next_tap(cg >= Cg16);       // (at most KG / Cg16 + 1 taps further)
            }
            lane_offsets();
        }
    };
    auto load = [&](int buf, int u) {                        // the u-th of this wave's NL loads of a stage
        const uint32_t boff = (uint32_t)buf * (STAGE_SLOTS * 16u);
        if (u < NLA) igd_load_lds(wr, lds_a0 + boff + (uint32_t)u * (NW * 64 * 16), na[u < NLA ? u : 0], (uint32_t)__builtin_amdgcn_readfirstlane((int)soff_a));
        else igd_load_lds(xr, lds_b0 + boff + (uint32_t)(u - NLA) * (NW * 64 * 16), nb[u < NLA ? 0 : u - NLA], (uint32_t)__builtin_amdgcn_readfirstlane((int)soff_b));
    };
    auto issue = [&](int buf, bool next) {                   // a stage's loads at once; next: another one follows
#pragma unroll
        for (int u = 0; u < NL; ++u) load(buf, u);
        if (next) next_stage();
    };

    v16i acc[NC][MI][NJ];
#pragma unroll
    for (int c = 0; c < NC; ++c)
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
            for (int j = 0; j < NJ; ++j)
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[c][i][j][v] = 0;

#pragma unroll
    for (int c = 0; c < NC; ++c) {
    if (ALLC && c > 0) {
        // the next class: its taps and offsets; the ring is free once every wave has read the last stage
        dc = dgrad_class<2>(a, c);
        nr = dc.nr;
        ns = dc.ns;
        gtot = nr * ns * Cg16;
        nsteps = (gtot + KG - 1) / KG;
#pragma unroll
        for (int i = 0; i < NLB; ++i) {
            bh[i] = boh[i] == kFar ? kFar : boh[i] + dc.bh;
            bw[i] = bow[i] + dc.bw;
            bbase[i] = bimg[i] + pixel(bh[i], bw[i]);
        }
        __syncthreads();
    }
    // prologue: the first NSTAGE-1 stages on their way
    first_stage();
    if (nsteps > 0) issue(0, nsteps > 1);     // (a class without taps has nothing to load: its pixels get zeros)
#pragma unroll
    for (int p = 1; p < NSTAGE - 1; ++p) {
        if (nsteps > p) issue(p, nsteps > p + 1);
    }
    for (int step = 0; step < nsteps; ++step) {
        const int buf = step % NSTAGE;
        // this stage's loads are the oldest outstanding ones; the loads of the up to NSTAGE - 2 stages
        // behind it may still be in flight
        if (NSTAGE == 4 && step + 2 < nsteps) igd_wait_vmcnt<NSTAGE == 4 ? 2 * NL : 0>();
        else if (NSTAGE >= 3 && step + 1 < nsteps) igd_wait_vmcnt<NSTAGE >= 3 ? NL : 0>();
        else igd_wait_vmcnt<0>();
        __syncthreads();   // every wave's part of this stage is in LDS; stage step-1 has been read by all
        // the next loads go into the buffer read in stage step-1
        const bool more = step + NSTAGE - 1 < nsteps, after = step + NSTAGE < nsteps;
        const int nbuf = (step + NSTAGE - 1) % NSTAGE;
        const uint4* __restrict__ sA = ring + buf * STAGE_SLOTS;
        const uint4* __restrict__ sB = sA + BM * KG;
        // Operands of PRE steps of 32 reduction bytes are requested ahead of the products, in turn with the loads of the next stage: either
        // keeps its pipe busy for hundreds of cycles (a wave's operands 16 reads of 1 KB at 128 bytes per cycle and compute unit, its loads
        // 8 of 1 KB at 64), so neither should queue behind the other.
        constexpr int KK = KG / 2, PRE = NJ * MI > 4 ? 2 : KK, RD = PRE * (MI + NJ);
        v4i fa[PRE][MI], fb[PRE][NJ];
        auto read = [&](int kk, int o) {                     // operand o of a step: MI filter fragments, then NJ pixel fragments
            const int g = kk * 2 + (lane >> 5);
            const uint4 t = o < MI ? sA[igd_slot<KG>(wm * 64 + o * 32 + (lane & 31), g)] : sB[igd_slot<KG>(wn * CW + (o - MI) * 32 + (lane & 31), g)];
            const v4i v = v4i{(int)t.x, (int)t.y, (int)t.z, (int)t.w};
            if (o < MI) fa[kk % PRE][o < MI ? o : 0] = v;
            else fb[kk % PRE][o < MI ? 0 : o - MI] = v;
        };
        if (more && !ALLC) {
#pragma unroll
            for (int u = 0; u < NL; ++u) {
                load(nbuf, u);
#pragma unroll
                for (int v = u * RD / NL; v < (u + 1) * RD / NL; ++v) read(v / (MI + NJ), v % (MI + NJ));
            }
            if (after) next_stage();
        } else {
            if (more) issue(nbuf, after);
#pragma unroll
            for (int v = 0; v < RD; ++v) read(v / (MI + NJ), v % (MI + NJ));
        }
#pragma unroll
        for (int kk = 0; kk < KK; ++kk) {
#pragma unroll
            for (int i = 0; i < MI; ++i)
#pragma unroll
                for (int j = 0; j < NJ; ++j)
                    acc[c][i][j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(fa[kk % PRE][i], fb[kk % PRE][j], acc[c][i][j], 0, 0, 0);
            if (kk + PRE < KK) {
#pragma unroll
                for (int o = 0; o < MI + NJ; ++o) read(kk + PRE, o);
            }
        }
    }
    }   // classes

    // ---- epilogue: Eq.2, straight into N,C,H,W ----------------------------------------------
    const float scale = __fmul_rn(a.sa[0], a.sb[0]);
    if constexpr (STG) {
        // Image planes of whole 16-byte groups: the tile goes through LDS, 64 rows at a time, so that a store instruction writes
        // the tile's columns of two to four channels as contiguous 16-byte pieces (512 bytes per channel and 128 columns) and
        // not 128 bytes each of two channels, which on planes that are no whole cache lines share a line at either end.
        // 24 -> 144 1x1 at 56 x 56, batch 64: 33.6 -> 26.7 us; 128 -> 512 at 28 x 28: 23.6 -> 20.5 (floor 19.9); 96 -> 576 at
        // 14 x 14: 12.1 -> 9.6.  Other planes (17 x 17, 7 x 7) keep the stores below: with 4-byte aligned 16-byte stores
        // and groups split at image borders they lose 3 us.
        constexpr int PITCH = BN + 8;         // 4 * PITCH mod 64 = 32: the half-waves of a store, 4 rows apart, use different banks
        static_assert(32 * WM * PITCH * 4 <= NSTAGE * STAGE_SLOTS * 16, "the staged rows fit the ring");
        int* const stg = reinterpret_cast<int*>(ring);
        constexpr int QPR = BN / 4, RPI = 64 * NW / QPR;     // 16-byte groups per row, rows per pass of the block
        const int q = tid % QPR, r0 = tid / QPR;
        const int col = colbase + 4 * q;
        const int n = image_of(col), opix = col - n * OHW;
#pragma unroll
        for (int i = 0; i < MI; ++i) {
            __syncthreads();
#pragma unroll
            for (int j = 0; j < NJ; ++j)
#pragma unroll
                for (int v = 0; v < 16; ++v)
                    stg[(wm * 32 + 8 * (v >> 2) + 4 * (lane >> 5) + (v & 3)) * PITCH + wn * CW + j * 32 + (lane & 31)] = acc[0][i][j][v];
            __syncthreads();
            if (col >= ncols) continue;
            // all of a lane's pieces are read before the first is written, and one 64-bit address serves them
            constexpr int PM = 32 / RPI;                      // pieces per 32 rows
            static_assert(32 % RPI == 0, "whole passes");
            int4 t[WM * PM];
#pragma unroll
            for (int u = 0; u < WM * PM; ++u) t[u] = *reinterpret_cast<const int4*>(stg + (u / PM * 32 + u % PM * RPI + r0) * PITCH + 4 * q);
            const int row0 = rowbase + i * 32 + r0;
            const size_t o0 = ((size_t)n * a.rows + row0) * OHWfull + opix;
            const bool full = rowbase + BM <= a.rows;         // (uniform)
#pragma unroll
            for (int u = 0; u < WM * PM; ++u) {
                const int dr = u / PM * 64 + u % PM * RPI;    // rows further on
                if (full || row0 + dr < a.rows) {
                    const size_t o = o0 + (size_t)dr * OHWfull;
                    *reinterpret_cast<float4*>(a.out + o) = make_float4(__fmul_rn((float)t[u].x, scale), __fmul_rn((float)t[u].y, scale),
                                                                        __fmul_rn((float)t[u].z, scale), __fmul_rn((float)t[u].w, scale));
                    if (a.acc) { a.acc[o] = t[u].x; a.acc[o + 1] = t[u].y; a.acc[o + 2] = t[u].z; a.acc[o + 3] = t[u].w; }
                }
            }
        }
        return;
    }
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
        const int col = colbase + wn * CW + j * 32 + (lane & 31);
        if (col >= ncols) continue;
        const int n = image_of(col);
        int opix = col - n * OHW;
        int ci = 0, cj = 0;
        if (CLS) {
            ci = row_of(opix);
            cj = opix - ci * OWc;
            opix = (dc.ch + a.cls_h * ci) * a.OW + dc.cw + a.cls_w * cj;
        }
#pragma unroll
        for (int i = 0; i < MI; ++i) {
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int row = rowbase + wm * 64 + i * 32 + 8 * (v >> 2) + 4 * (lane >> 5) + (v & 3);
                if (row < a.rows) {
                    const size_t idx = ((size_t)n * a.rows + row) * OHWfull + opix;
                    const int val = acc[0][i][j][v];
                    if (ALLC) {
                        // the cell's four pixels, classes (row parity, column parity) = 0 .. 3; the last cell row / column
                        // of an odd image holds one row / column only
                        const size_t o = ((size_t)n * a.rows + row) * OHWfull + (size_t)(2 * ci) * a.OW + 2 * cj;
                        const bool two = 2 * ci + 1 < a.OH, right = 2 * cj + 1 < a.OW;
                        const int v00 = val, v01 = acc[NC > 1 ? 1 : 0][i][j][v], v10 = acc[NC > 2 ? 2 : 0][i][j][v],
                                  v11 = acc[NC > 3 ? 3 : 0][i][j][v];
                        if (!(a.OW & 1)) {          // every cell starts on an 8-byte boundary
                            *reinterpret_cast<float2*>(a.out + o) = make_float2(__fmul_rn((float)v00, scale), __fmul_rn((float)v01, scale));
                            if (two) *reinterpret_cast<float2*>(a.out + o + a.OW) = make_float2(__fmul_rn((float)v10, scale), __fmul_rn((float)v11, scale));
                            if (a.acc) {
                                *reinterpret_cast<int2*>(a.acc + o) = make_int2(v00, v01);
                                if (two) *reinterpret_cast<int2*>(a.acc + o + a.OW) = make_int2(v10, v11);
                            }
                        } else {
                            a.out[o] = __fmul_rn((float)v00, scale);
                            if (right) a.out[o + 1] = __fmul_rn((float)v01, scale);
                            if (two) {
                                a.out[o + a.OW] = __fmul_rn((float)v10, scale);
                                if (right) a.out[o + a.OW + 1] = __fmul_rn((float)v11, scale);
                            }
                            if (a.acc) {
                                a.acc[o] = v00;
                                if (right) a.acc[o + 1] = v01;
                                if (two) {
                                    a.acc[o + a.OW] = v10;
                                    if (right) a.acc[o + a.OW + 1] = v11;
                                }
                            }
                        }
                    } else if (CELL) {
                        const size_t o = ((size_t)n * a.rows + row) * OHWfull + (size_t)(2 * ci) * a.OW + 2 * cj;
                        const bool two = 2 * ci + 1 < a.OH;
                        store_cell<float, float2>(a.out, o, a.OW, two, dc.ch, dc.cw, __fmul_rn((float)val, scale));
                        if (a.acc) store_cell<int32_t, int2>(a.acc, o, a.OW, two, dc.ch, dc.cw, val);
                    } else {
                        a.out[idx] = __fmul_rn((float)val, scale);
                        if (a.acc) a.acc[idx] = val;
                    }
                }
            }
        }
    }
}

}  // namespace int8t
