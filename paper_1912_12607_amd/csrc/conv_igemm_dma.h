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
__device__ __forceinline__ DgradClass dgrad_class(const IgemmArgs& a, int cls) {
    DgradClass c;
    const int csh = a.cls_h, csw = a.cls_w;     // the stride, or 1 where that direction is not split
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
    const int wg_i = block >> 3;
    int cgroup = wg_i / rtiles;
    DgradClass dc;
    if (CLS) {
        if (CELL) {
            dc = dgrad_class(a, ALLC ? 0 : a.cell - 1);
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
    int nr = CLS ? dc.nr : a.R, ns = CLS ? dc.ns : a.S;  // (ALLC: of the class being run)
    int gtot = nr * ns * Cg16;
    int nsteps = (gtot + KG - 1) / KG;
    // colrun (igemm_colrun): an XCD takes a run of column tiles instead of every eighth.
    const int ctile = a.colrun ? (int)(block & 7) * a.colrun + cgroup : (cgroup << 3) + (int)(block & 7);
    if (ctile * BN >= ncols) return;
    const int rowbase = (wg_i % rtiles) * BM;
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
    int bh[NLB], bw[NLB];
    int boh[NLB], bow[NLB];                                  // (ALLC) the column's cell, to which each class adds its offset
    uint32_t bimg[NLB];                                      // byte offset of the column's image or OOB
#pragma unroll
    for (int i = 0; i < NLB; ++i) {
        const int col = colbase + RPL * (wave + NW * i) + lrow;
        const bool cv = col < ncols;
        const int cc = cv ? col : 0;
        const int n = cc / OHW, rem = cc - n * OHW;
        const int oh = rem / OWc, ow = rem - oh * OWc;
        boh[i] = oh;
        bow[i] = ow;
        bh[i] = CLS ? (oh + dc.bh) : DGRAD ? (oh + a.pad_h) : (oh * a.stride_h - a.pad_h);
        bw[i] = CLS ? (ow + dc.bw) : DGRAD ? (ow + a.pad_w) : (ow * a.stride_w - a.pad_w);
        bimg[i] = cv ? (uint32_t)n * (uint32_t)(a.IH * a.IW * a.Ca) : IGD_OOB;
    }
    // reduction position of this lane's granule: filter tap (r,s) and channel granule cg
    int r, s, cg;
    int qnext;                                               // granule index of the next stage to issue
    auto first_granule = [&]() {
        const int tap = gsw / Cg16;
        cg = gsw - tap * Cg16;
        r = tap / (ns > 0 ? ns : 1);
        s = tap - r * ns;
        qnext = gsw;
    };
    first_granule();

    auto issue_a = [&](int buf) {
        const uint32_t boff = (uint32_t)buf * (STAGE_SLOTS * 16u);
        const bool qv = qnext < gtot;
        // granule of the filter row: the taps of a class are a sub-grid of the R x S filter
        const int wq = CLS ? ((dc.r0 + a.cls_h * r) * a.S + dc.s0 + a.cls_w * s) * Cg16 + cg : qnext;
#pragma unroll
        for (int i = 0; i < NLA; ++i) {
            const uint32_t off = (qv && aoff[i] != IGD_OOB) ? aoff[i] + (uint32_t)wq * 16u : IGD_OOB;
            igd_load_lds(wr, lds_a0 + boff + (uint32_t)i * (NW * 64 * 16), off);
        }
    };
    auto issue_b = [&](int buf) {
        const uint32_t boff = (uint32_t)buf * (STAGE_SLOTS * 16u);
        const bool qv = qnext < gtot;
#pragma unroll
        for (int i = 0; i < NLB; ++i) {
            int ih, iw;
            bool ok = qv && bimg[i] != IGD_OOB;
            if (DGRAD) {
                const int th = bh[i] - r, tw = bw[i] - s;
                // a direction split into classes is a stride-1 pass; otherwise only the taps that divide reach a pixel
                const int dsh = CLS ? a.stride_h / a.cls_h : a.stride_h, dsw = CLS ? a.stride_w / a.cls_w : a.stride_w;
                if (dsh == 1 && dsw == 1) {
                    ih = th;
                    iw = tw;
                } else {
                    ih = th / dsh;
                    iw = tw / dsw;
                    ok = ok && th >= 0 && tw >= 0 && (ih * dsh == th) && (iw * dsw == tw);
                }
            } else {
                ih = bh[i] + r;
                iw = bw[i] + s;
            }
            ok = ok && (unsigned)ih < (unsigned)a.IH && (unsigned)iw < (unsigned)a.IW;
            const uint32_t off = ok ? bimg[i] + (uint32_t)((ih * a.IW + iw) * a.Ca + cg * 16) : IGD_OOB;
            igd_load_lds(xr, lds_b0 + boff + (uint32_t)i * (NW * 64 * 16), off);
        }
        // advance this lane's reduction position by one stage (KG granules)
        qnext += KG;
        cg += KG;
        while (cg >= Cg16) {
            cg -= Cg16;
            if (++s == ns) {
                s = 0;
                ++r;
            }
        }
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
        dc = dgrad_class(a, c);
        nr = dc.nr;
        ns = dc.ns;
        gtot = nr * ns * Cg16;
        nsteps = (gtot + KG - 1) / KG;
#pragma unroll
        for (int i = 0; i < NLB; ++i) {
            bh[i] = boh[i] + dc.bh;
            bw[i] = bow[i] + dc.bw;
        }
        first_granule();
        __syncthreads();
    }
    // prologue: the first NSTAGE-1 stages on their way
    if (nsteps > 0) {     // (a class without taps has nothing to load: its pixels get zeros)
        issue_a(0);
        issue_b(0);
    }
#pragma unroll
    for (int p = 1; p < NSTAGE - 1; ++p) {
        if (nsteps > p) {
            issue_a(p);
            issue_b(p);
        }
    }
    for (int step = 0; step < nsteps; ++step) {
        const int buf = step % NSTAGE;
        // this stage's loads are the oldest outstanding ones; the loads of the up to NSTAGE - 2 stages
        // behind it may still be in flight
        if (NSTAGE == 4 && step + 2 < nsteps) igd_wait_vmcnt<NSTAGE == 4 ? 2 * NL : 0>();
        else if (NSTAGE >= 3 && step + 1 < nsteps) igd_wait_vmcnt<NSTAGE >= 3 ? NL : 0>();
        else igd_wait_vmcnt<0>();
        __syncthreads();   // every wave's part of this stage is in LDS; stage step-1 has been read by all
        // the next loads go into the buffer read in stage step-1; the weight half is requested now,
        // the pixel half in the middle of this stage's MFMAs, so the memory pipeline sees a steady
        // stream instead of one burst per stage
        const bool more = step + NSTAGE - 1 < nsteps;
        const int nbuf = (step + NSTAGE - 1) % NSTAGE;
        if (more) issue_a(nbuf);
        const uint4* __restrict__ sA = ring + buf * STAGE_SLOTS;
        const uint4* __restrict__ sB = sA + BM * KG;
#pragma unroll
        for (int kk = 0; kk < KG / 2; ++kk) {
            const int g = kk * 2 + (lane >> 5);
            v4i fa[MI], fb[NJ];
#pragma unroll
            for (int i = 0; i < MI; ++i) {
                const uint4 t = sA[igd_slot<KG>(wm * 64 + i * 32 + (lane & 31), g)];
                fa[i] = v4i{(int)t.x, (int)t.y, (int)t.z, (int)t.w};
            }
#pragma unroll
            for (int j = 0; j < NJ; ++j) {
                const uint4 t = sB[igd_slot<KG>(wn * CW + j * 32 + (lane & 31), g)];
                fb[j] = v4i{(int)t.x, (int)t.y, (int)t.z, (int)t.w};
            }
#pragma unroll
            for (int i = 0; i < MI; ++i)
#pragma unroll
                for (int j = 0; j < NJ; ++j)
                    acc[c][i][j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(fa[i], fb[j], acc[c][i][j], 0, 0, 0);
            if (kk == (KG >= 8 ? KG / 4 - 1 : 0) && more) issue_b(nbuf);
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
        const int n = col / OHW, opix = col - n * OHW;
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
#pragma unroll 4
            for (int r = r0; r < 32 * WM; r += RPI) {
                const int row = rowbase + (r >> 5) * 64 + i * 32 + (r & 31);
                if (row >= a.rows) continue;
                const int4 t = *reinterpret_cast<const int4*>(stg + r * PITCH + 4 * q);
                const size_t o = ((size_t)n * a.rows + row) * OHWfull + opix;
                *reinterpret_cast<float4*>(a.out + o) = make_float4(__fmul_rn((float)t.x, scale), __fmul_rn((float)t.y, scale),
                                                                    __fmul_rn((float)t.z, scale), __fmul_rn((float)t.w, scale));
                if (a.acc) { a.acc[o] = t.x; a.acc[o + 1] = t.y; a.acc[o + 2] = t.z; a.acc[o + 3] = t.w; }
            }
        }
        return;
    }
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
        const int col = colbase + wn * CW + j * 32 + (lane & 31);
        if (col >= ncols) continue;
        const int n = col / OHW;
        int opix = col - n * OHW;
        int ci = 0, cj = 0;
        if (CLS) {
            ci = opix / OWc;
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
