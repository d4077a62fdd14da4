// Host side of backward-weight on image lines (conv_wgrad_lines.h): where it applies, its plan, its launch.
#include "conv_wgrad_lines.h"

namespace int8t {

// The pass in a launch of its own (wgrad_lines_tile).
template <int ST, int WM, int WN, int GP, bool S2 = false>
__global__ __launch_bounds__(256, 2) void wgrad_lines_kernel(const WgradArgs a) {
    wgrad_lines_tile<ST, WM, WN, GP, S2>(a, blockIdx.x);
}

bool wgrad_lines_s2(const WgradArgs& a) {
    return a.R == 3 && a.S == 3 && a.stride_h == 2 && a.stride_w == 2 && a.pad_h <= 2 && a.pad_w <= 2;
}

bool wgrad_lines_applies(const WgradArgs& a) {
    const bool one = a.R == 1 && a.S == 1;
    if (a.s2d) return false;
    // strides: 1x1 filters without padding (the pass then runs on every stride-th row and pixel), and 3x3 filters
    // under stride 2 x 2
    if ((a.stride_h != 1 || a.stride_w != 1) && !(one && a.pad_h == 0 && a.pad_w == 0) && !wgrad_lines_s2(a)) return false;
    const bool along_w = a.S == 3 || a.S == 5 || a.S == 7;
    const bool along_h = a.S == 1 && (a.R == 3 || a.R == 5 || a.R == 7);
    if (!one && !along_w && !along_h) return false;
    // byte offsets into either tensor stay below the value that stands for "nothing to load"
    if ((unsigned long long)a.N * a.H * a.W * a.Cp >= IGD_OOB || (unsigned long long)a.N * a.P * a.Q * a.Kp >= IGD_OOB) return false;
    return true;
}

void wgrad_plan_lines(WgradArgs* a) {
    const bool along_w = wgrad_lines_along_w(a->R, a->S);
    const int ST = along_w ? a->S : a->R;
    const int WT = ST == 1 ? 2 : 1;              // MFMA tiles per wave and tap in each direction
    const bool s2 = wgrad_lines_s2(*a);
    const int GP = ST == 1 ? 4 : s2 ? 3 : ST == 5 ? 6 : 8;      // a multiple of the window's ST + 1 slots (of 3 under stride 2)
    a->lines = 1;
    a->TB = ST;
    a->CS = WT;
    a->BP = a->BQ = a->ntp = a->ntq = a->ngrp = 0;
    a->xt_slots = 0;
    a->tapgroups = along_w ? a->R : 1;
    a->ktiles = (a->K + 64 * WT - 1) / (64 * WT);
    a->ctiles = (a->Cp + 64 * WT - 1) / (64 * WT);
    const int NLI = along_w ? a->P : a->Q;
    const int QL = along_w ? a->Q : a->P;
    const int WLn = (a->stride_h != 1 || a->stride_w != 1) ? QL : along_w ? a->W : a->H;
    const int pl = s2 ? 1 : along_w ? a->pad_w : a->pad_h;      // (stride 2: QL + 1 steps per chunk)
    a->chunks = (a->N * NLI + WL_LINES - 1) / WL_LINES;
    a->lds_bytes = (size_t)WL_NSTAGE * wl_stage_bytes(WT, WT, GP, s2 ? 2 : 1);
    // Split count by the same estimate as wgrad_plan(): rounds of resident blocks (two per compute unit),
    // a block pays a prologue plus its stages, every split one write and one read of the partial tiles.
    const int out_tiles = a->ktiles * a->ctiles * a->tapgroups;
    const int slots = 512;
    const double stages_per_chunk = (double)(WLn + pl) / GP;
    const double mfma_per_chunk = (double)QL * ST * WT * WT;   // per wave, a little less at the image border
    const double t_chunk = stages_per_chunk * 0.45 + 0.014 * 2.0 * mfma_per_chunk;
    const double t_partial = (double)a->K * a->R * a->S * a->Cp * 8.0 / 4.0e6;
    a->t_chunk = (float)t_chunk;
    a->t_partial = (float)t_partial;
    int splits = 1;
    double best = 1e30;
    for (int sp = 1; sp <= a->chunks && sp <= 4096; ++sp) {
        const long long blocks = (long long)out_tiles * sp;
        const double rounds = (double)((blocks + slots - 1) / slots);
        const double t = rounds * (3.0 + ((a->chunks + sp - 1) / sp) * t_chunk) + sp * t_partial;
        if (t < best) { best = t; splits = sp; }
        if (blocks > 8LL * slots || (long long)a->chunks * (sp + 2) >= (1LL << 31)) break;
    }
    if (a->variant == VAR_WGRAD_FEWER) splits = splits > 1 ? splits / 2 : 1;
    if (a->variant == VAR_WGRAD_MORE && 2 * splits <= a->chunks && 2 * splits <= 4096 && (long long)a->chunks * (2 * splits) < (1LL << 31)) splits *= 2;
    a->splits = splits;
    // XCD patches (see the kernel): the split of 8 into xgk x xgc whose patches read the fewest slices
    a->xgk = a->xgc = 0;
    if (a->ktiles * a->ctiles >= 16) {
        int best = 1 << 30;
        for (int gk = 1; gk <= 8; gk *= 2) {
            const int gc = 8 / gk;
            if (gk > a->ktiles || gc > a->ctiles) continue;
            const int cost = (a->ktiles + gk - 1) / gk + (a->ctiles + gc - 1) / gc;
            if (cost < best) { best = cost; a->xgk = gk; a->xgc = gc; }
        }
    }
    const int pk = a->xgk ? (a->ktiles + a->xgk - 1) / a->xgk : a->ktiles, pc = a->xgk ? (a->ctiles + a->xgc - 1) / a->xgc : a->ctiles;
    a->by_tiles = fast_div((unsigned)(pk * pc * a->tapgroups));
    a->by_taps = fast_div((unsigned)a->tapgroups);
    a->by_ctiles = fast_div((unsigned)pc);
    a->by_splits = fast_div((unsigned)a->splits);
    a->by_lines = fast_div((unsigned)NLI);
}

unsigned wgrad_lines_grid(const WgradArgs& a) {
    const unsigned out_tiles = (unsigned)(a.ktiles * a.ctiles * a.tapgroups);
    if (a.xgk > 0) {
        const unsigned pk = (unsigned)((a.ktiles + a.xgk - 1) / a.xgk), pc = (unsigned)((a.ctiles + a.xgc - 1) / a.xgc);
        return 8u * pk * pc * (unsigned)a.tapgroups * (unsigned)a.splits;
    }
    return wgrad_xcd_mapping(a.splits) ? out_tiles * 8u * (unsigned)((a.splits + 7) / 8) : out_tiles * (unsigned)a.splits;
}

hipError_t launch_wgrad_lines(const WgradArgs& a, hipStream_t st) {
    const dim3 grid(wgrad_lines_grid(a));
    KernelTimer kt(KID_WGRAD_LINES, st);
#define LAUNCH(STv, WTv, GPv, S2v)                                                                       \
    do {                                                                                                 \
        static std::atomic<unsigned long long> attr_done;                                                \
        hipError_t ea = raise_dynamic_lds(reinterpret_cast<const void*>(wgrad_lines_kernel<STv, WTv, WTv, GPv, S2v>), \
                                          WL_NSTAGE * wl_stage_bytes(WTv, WTv, GPv, S2v ? 2 : 1), attr_done); \
        if (ea != hipSuccess) return ea;                                                                 \
        launch_timed(kt, (wgrad_lines_kernel<STv, WTv, WTv, GPv, S2v>), grid, dim3(256), a.lds_bytes, st, a); \
    } while (0)
    if (a.TB == 3 && wgrad_lines_s2(a)) LAUNCH(3, 1, 3, true);
    else if (a.TB == 3) LAUNCH(3, 1, 8, false);
    else if (a.TB == 5) LAUNCH(5, 1, 6, false);     // (35 x 35, 5x5, 48 -> 64 channels, batch 32: 23.2 us on wgrad_kernel, 15.9 here)
    else if (a.TB == 7) LAUNCH(7, 1, 8, false);
    else if (a.TB == 1) LAUNCH(1, 2, 4, false);
    else return hipErrorInvalidValue;
#undef LAUNCH
    return hipGetLastError();
}

}  // namespace int8t
