// Host side of the dense passes with the filter bank on chip (conv_band.h), their launch alone, and the one that they share with
// backward-weight.
#include <algorithm>

#include "conv_band.h"

namespace int8t {

// A pass in a launch of its own.
template <bool DGRAD, int MT, int NTW, bool UNI, int STG>
__global__ __launch_bounds__(256) void band_kernel(const IgemmArgs a, int BP, int nbands_h, int nbands) {
    band_walk<DGRAD, MT, NTW, UNI, STG>(a, BP, nbands_h, nbands, (int)blockIdx.x, (int)gridDim.x);
}
template <bool DGRAD, int NKS>
__global__ __launch_bounds__(256, 2) void band_reg_kernel(const IgemmArgs a, int BP, int nbands_h, int nbands, const BandRegTab tab) {
    band_reg_walk<DGRAD, NKS>(a, BP, nbands_h, nbands, tab, (int)blockIdx.x, (int)gridDim.x);
}

bool band_plan(const IgemmArgs& a, BandPlan* p) {
    if (a.stride_h != 1 || a.stride_w != 1 || a.rows > 64 || a.OW > BAND_MAXPIX) return false;
    const int Cg16 = a.Ca >> 4;
    const int G = a.R * a.S * Cg16;
    if (G > BAND_MAXG) return false;
    if ((size_t)a.N * a.rows * a.OH * a.OW > 0x7FFFFFFFull) return false;
    // band height: as many output rows as fit 128 pixels (one 32-pixel tile per wave; smaller bands
    // balance better over the persistent blocks than 256-pixel ones); one row of up to 256 pixels
    // (two tiles per wave) when a single row is wider than 128
    int ntw = 1;
    int BP = 128 / a.OW;
    if (BP < 1) { ntw = 2; BP = 1; }
    if (BP > a.OH) BP = a.OH;
    const int WW = a.OW + a.S - 1;
    const int kw = (WW * Cg16 + 255) / 256;
    while (BP > 1 && (BP + a.R - 1) * kw > BAND_STAGE) --BP;
    const int WH = BP + a.R - 1;
    if (WH * kw > BAND_STAGE) return false;
    p->BP = BP;
    p->ntw = ntw;
    p->mt = a.rows > 32 ? 2 : 1;
    p->uni = a.rows % 8 == 0;
    p->few = WH * kw <= BAND_STAGE_FEW;
    p->lds = ((size_t)64 * odd_pitch(G) + (size_t)WH * WW * odd_pitch(Cg16) + 1) * 16 + (size_t)(G + 4) * sizeof(int2);
    if (p->lds > BAND_LDS_MAX) return false;
    p->nbands_h = (a.OH + BP - 1) / BP;
    p->nbands = a.N * p->nbands_h;
    // register-resident weights when the reduction length is one of the instantiated ones
    p->nks = 0;
    if (ntw == 1 && (Cg16 & 1) == 0 && WH <= BAND_REG_ROWS && WW * Cg16 <= 256 && (size_t)a.rows * a.OH * a.OW <= ((size_t)1 << 29) &&
        (G == 4 || G == 8 || G == 18 || G == 36)) {
        p->nks = G / 2;
        p->lds = std::max((size_t)WH * WW * odd_pitch(Cg16) * 16, (size_t)64 * odd_pitch(G) * 16);    // the weight matrix passes through LDS first
        p->tab = BandRegTab{};
        const int PG = odd_pitch(Cg16);
        const int drmin = a.dgrad ? (a.pad_h - (a.R - 1)) : -a.pad_h;
        const int dsmin = a.dgrad ? (a.pad_w - (a.S - 1)) : -a.pad_w;
        for (int ks = 0; 2 * ks < G; ++ks) {
            const int g = 2 * ks, tap = g / Cg16, cg = g - tap * Cg16;
            const int r = tap / a.S, sx = tap - r * a.S;
            const int dr = a.dgrad ? (a.pad_h - r) : (r - a.pad_h);
            const int ds = a.dgrad ? (a.pad_w - sx) : (sx - a.pad_w);
            p->tab.koff[ks] = ((dr - drmin) * WW + (ds - dsmin)) * PG + cg;
        }
    }
    return true;
}

// Returns true (and launches) when the layer fits this kernel; false: use the implicit GEMM.
bool launch_band(const IgemmArgs& a, hipStream_t st, hipError_t* err, bool dry_run) {
    BandPlan p;
    if (!band_plan(a, &p)) return false;
    if (dry_run) return true;
    const dim3 grid(p.nbands < 512 ? p.nbands : 512);
    if (p.nks) {
        typedef void (*kern_t)(const IgemmArgs, int, int, int, const BandRegTab);
        const int slot = 2 * (p.nks == 2 ? 0 : p.nks == 4 ? 1 : p.nks == 9 ? 2 : 3) + (a.dgrad ? 1 : 0);
        static const kern_t kerns[8] = {band_reg_kernel<false, 2>, band_reg_kernel<true, 2>, band_reg_kernel<false, 4>, band_reg_kernel<true, 4>,
                                        band_reg_kernel<false, 9>, band_reg_kernel<true, 9>, band_reg_kernel<false, 18>, band_reg_kernel<true, 18>};
        static std::atomic<unsigned long long> attr_done[8];
        const hipError_t e = raise_dynamic_lds(reinterpret_cast<const void*>(kerns[slot]), (int)BAND_LDS_MAX, attr_done[slot]);
        if (e != hipSuccess) { *err = e; return true; }
        KernelTimer kt(KID_BAND_REG, st);
        launch_timed(kt, kerns[slot], grid, dim3(256), p.lds, st, a, p.BP, p.nbands_h, p.nbands, p.tab);
        *err = hipGetLastError();
        return true;
    }
    const int variant = (a.dgrad ? 16 : 0) + (p.mt - 1) * 8 + (p.ntw - 1) * 4 + (p.few ? 0 : 2) + (p.uni ? 1 : 0);
    typedef void (*kern_t)(const IgemmArgs, int, int, int);
#define BK(D, M, N) band_kernel<D, M, N, false, BAND_STAGE_FEW>, band_kernel<D, M, N, true, BAND_STAGE_FEW>, band_kernel<D, M, N, false, BAND_STAGE>, band_kernel<D, M, N, true, BAND_STAGE>
    static const kern_t kerns[32] = {BK(false, 1, 1), BK(false, 1, 2), BK(false, 2, 1), BK(false, 2, 2),
                                     BK(true, 1, 1),  BK(true, 1, 2),  BK(true, 2, 1),  BK(true, 2, 2)};
#undef BK
    static std::atomic<unsigned long long> attr_done[32];
    {
        hipError_t e = raise_dynamic_lds(reinterpret_cast<const void*>(kerns[variant]), (int)BAND_LDS_MAX, attr_done[variant]);
        if (e != hipSuccess) { *err = e; return true; }
    }
    {
        KernelTimer kt(KID_BAND, st);
        launch_timed(kt, kerns[variant], grid, dim3(256), p.lds, st, a, p.BP, p.nbands_h, p.nbands);
    }
    *err = hipGetLastError();
    return true;
}

}  // namespace int8t
