// Dense backward-weight convolution: plan, launches and the reduction of the shares' partial tiles (the kernel that works on image
// granules: conv_wgrad_tile.h; on image lines: conv_wgrad_lines.h).
#include "conv_wgrad_tile.h"

namespace int8t {

// The pass in a launch of its own (wgrad_tile).
template <int TB, int CS, bool PK = false>
__global__ __launch_bounds__(256, 2) void wgrad_kernel(const WgradArgs a) {
    wgrad_tile<TB, CS, PK>(a, blockIdx.x);
}

// Where a sum of filter k, tap rs, channel c of the pass's own geometry goes.
__device__ __forceinline__ void wgrad_result(const WgradArgs& a, int k, int rs, int c, int sum, float scale) {
    if (c >= a.C) return;
    size_t o = ((size_t)k * a.C + c) * (a.R * a.S) + rs;
    if (a.s2d) {
        // back from the space-to-depth form: channel (2 dy + dx) * oC + c0 of tap (r', s') is channel c0
        // of tap (2 r' + dy - eh, 2 s' + dx - ew); taps outside the layer's own filter are dropped
        const int blk = c / a.oC, c0 = c - blk * a.oC;
        const int rr = rs / a.S;
        const int r = 2 * rr + (blk >> 1) - a.eh, s = 2 * (rs - rr * a.S) + (blk & 1) - a.ew;
        if (r < 0 || r >= a.oR || s < 0 || s >= a.oS) return;
        o = (((size_t)k * a.oC + c0) * a.oR + r) * a.oS + s;
    }
    a.dw[o] = __fmul_rn((float)sum, scale);
    if (a.acc) a.acc[o] = sum;
}

// Few weights under many shares (a share's partial tile set is a few hundred KB at most): a block owns Q quads of four
// filters, side by side in the partial's own order whatever taps and channels they belong to, its threads are (quads) x (split
// lanes); every thread has up to 8 shares' 16 bytes in flight at once, the lanes of a wave are combined by lane
// exchanges, the four waves through LDS.
// Bound: one round trip to memory and the launch.  Before, 4 or 16 quads x one tap with the shares one after the other and the lanes summed
// in LDS, and now, us: 3x3, 64 channels at 56 x 56, batch 64 (112 shares) 7.2, 4.7; 1x1, 64 -> 256 at 56 x 56, batch 256 (224) 7.2, 4.6;
// 1x1, 1024 -> 256 at 14 x 14, batch 128 (19) 6.8, 5.5; 5x5, 48 -> 64 at 35 x 35, batch 32 (35) 5.4, 4.5.
// Few shares of many weights are bandwidth: 1x1, 1024 -> 2048 at 4 x 4, batch 256 (3 shares, 34 MB), all 8 loads of a lane / the one it needs:
// 10.4, 9.4; 2048 -> 512 at 7 x 7, batch 64 (3) 6.3, 5.7.
template <int Q>
__global__ __launch_bounds__(256) void wgrad_reduce_flat_kernel(const WgradArgs a) {
    constexpr int ZL = 256 / Q, ZU = 8;
    __shared__ int4 part[4][Q];
    const unsigned ncolsp = (unsigned)(a.R * a.S) * (unsigned)a.Cp, quads = (unsigned)((a.K + 3) >> 2) * ncolsp;
    const unsigned q0 = blockIdx.x * Q;
    const int zl = threadIdx.x / Q;
    const unsigned qi = q0 + threadIdx.x % Q;
    const int4* __restrict__ p = reinterpret_cast<const int4*>(a.partial) + (qi < quads ? qi : 0u);
    int4 sum = make_int4(0, 0, 0, 0);
    for (int z0 = 0; z0 < a.splits; z0 += ZU * ZL) {       // (the block's lanes together: no load that none of them needs)
        int4 v[ZU];
#pragma unroll
        for (int u = 0; u < ZU; ++u) {           // (a lane past the end takes the last share again, not added)
            v[u] = make_int4(0, 0, 0, 0);
            const int z = z0 + u * ZL + zl;
            if (z0 + u * ZL < a.splits) v[u] = p[(size_t)(z < a.splits ? z : a.splits - 1) * quads];
        }
#pragma unroll
        for (int u = 0; u < ZU; ++u) {
            const int keep = z0 + u * ZL + zl < a.splits ? -1 : 0;
            sum.x += v[u].x & keep; sum.y += v[u].y & keep; sum.z += v[u].z & keep; sum.w += v[u].w & keep;
        }
    }
#pragma unroll
    for (int o = Q; o < kWave; o <<= 1) {
        sum.x += __shfl_xor(sum.x, o, kWave); sum.y += __shfl_xor(sum.y, o, kWave);
        sum.z += __shfl_xor(sum.z, o, kWave); sum.w += __shfl_xor(sum.w, o, kWave);
    }
    if ((int)(threadIdx.x & (kWave - 1)) < Q) part[threadIdx.x / kWave][threadIdx.x % Q] = sum;
    __syncthreads();
    if (threadIdx.x >= 4 * Q) return;
    // (the filters of the quads one after the other: neighbouring threads then write neighbouring channels)
    const unsigned f = threadIdx.x / Q, u = threadIdx.x % Q;
    if (q0 + u >= quads) return;
    const int* const t = reinterpret_cast<const int*>(&part[0][0]) + 4 * u + f;
    const int v = (t[0] + t[4 * Q]) + (t[8 * Q] + t[12 * Q]);
    const unsigned k4 = (q0 + u) / ncolsp, col = q0 + u - k4 * ncolsp;
    const int k = (int)(4 * k4 + f), rs = (int)(col / (unsigned)a.Cp), c = (int)(col - (unsigned)rs * (unsigned)a.Cp);
    if (k < a.K) wgrad_result(a, k, rs, c, v, __fmul_rn(a.sa[0], a.sb[0]));
}

// The same with all taps of a filter in a block, or rows of them: the sums then leave as contiguous runs of the result.  A block owns
// four filters, QN channels x RSC taps; its 256 threads are 256/QN split lanes x QN channels.  Every thread adds up the
// splits z = lane, lane + 256/QN, ... of its channel at each tap (independent 16-byte loads, RSC of them in flight
// per split), the lanes are combined through LDS, and the sums leave in the order of the result tensor -- with
// all taps of a filter in the block (RSC = R*S) that is one contiguous run of QN*RSC floats per filter.  LDS holds
// [split lane][filter][channel][tap]; an odd number of taps per channel puts the stores of a wave in different banks.
template <int QN, int RSC>
__global__ __launch_bounds__(256) void wgrad_reduce_kernel(const WgradArgs a) {
    constexpr int ZL = 256 / QN, RUN = QN * RSC, PITCH = 4 * RUN;
    __shared__ int sred[ZL * PITCH];
    const int RS = a.R * a.S;
    const int ncolsp = RS * a.Cp;
    const size_t total = wgrad_partial_elems(a) >> 2;
    const int nrg = RS / RSC, nct = a.Cp / QN;
    int b = blockIdx.x;
    const int rg = b % nrg;
    b /= nrg;
    const int ct = b % nct, k4 = b / nct;
    const int qc = threadIdx.x % QN, zl = threadIdx.x / QN;
    const int4* __restrict__ p = reinterpret_cast<const int4*>(a.partial) + (size_t)k4 * ncolsp + (size_t)(rg * RSC) * a.Cp + ct * QN + qc;
    int4 s4[RSC];
#pragma unroll
    for (int j = 0; j < RSC; ++j) s4[j] = make_int4(0, 0, 0, 0);
    // ZU splits at a time, so that a thread has ZU * RSC (at least 4) loads in flight
    constexpr int ZU = RSC >= 4 ? 1 : RSC == 3 ? 2 : 4;
    int z = zl;
    for (; z + (ZU - 1) * ZL < a.splits; z += ZU * ZL) {
        int4 v[ZU][RSC];
#pragma unroll
        for (int u = 0; u < ZU; ++u)
#pragma unroll
            for (int j = 0; j < RSC; ++j) v[u][j] = p[(size_t)(z + u * ZL) * total + (size_t)j * a.Cp];
#pragma unroll
        for (int u = 0; u < ZU; ++u)
#pragma unroll
            for (int j = 0; j < RSC; ++j) { s4[j].x += v[u][j].x; s4[j].y += v[u][j].y; s4[j].z += v[u][j].z; s4[j].w += v[u][j].w; }
    }
    for (; z < a.splits; z += ZL) {
#pragma unroll
        for (int j = 0; j < RSC; ++j) {
            const int4 v = p[(size_t)z * total + (size_t)j * a.Cp];
            s4[j].x += v.x; s4[j].y += v.y; s4[j].z += v.z; s4[j].w += v.w;
        }
    }
    int* __restrict__ mine = sred + zl * PITCH + qc * RSC;
#pragma unroll
    for (int j = 0; j < RSC; ++j) {
        mine[j] = s4[j].x;
        mine[RUN + j] = s4[j].y;
        mine[2 * RUN + j] = s4[j].z;
        mine[3 * RUN + j] = s4[j].w;
    }
    __syncthreads();
    const int nz = a.splits < ZL ? a.splits : ZL;
    const float scale = __fmul_rn(a.sa[0], a.sb[0]);
    for (int t = threadIdx.x; t < PITCH; t += 256) {
        const int f = t / RUN, cl = (t - f * RUN) / RSC;
        int sum = 0;
        for (int z = 0; z < nz; ++z) sum += sred[z * PITCH + t];
        if (4 * k4 + f < a.K) wgrad_result(a, 4 * k4 + f, rg * RSC + (t - f * RUN - cl * RSC), ct * QN + cl, sum, scale);
    }
}

// The kernel VAR_AUTO runs: wgrad_lines_kernel wherever it applies (measured on the benchmark's 1x7, 7x1
// and 3x3 layers it needs 0.6 - 0.85 of wgrad_kernel's time), for 1x1 filters with fewer than 128 channels on one side where
//  - there are 256 input channels (the other kernel's 256-channel tile reads the gradient 16 images at a time and is slower at
//    every size: 21 random layers, 0.79 of its time alone and 0.56 in the shared launch of the three passes), or
//  - the 32-line chunks are at least as many as the positions of a line (a batch of 32, on square images).  A chunk is walked position
//    by position: with fewer, long ones most compute units have nothing to do (16 -> 24, 73 x 73, batch 16: 9.3 against 16.9 us).
//    Over 100 random layers 0.95 alone, 0.92 in the shared launch (40 -> 700, 20 x 20, batch 256: 36.6 and 23.5; 96 -> 512 at
//    28 x 28, batch 64: 21.2, 18.1; 64 -> 256 at 56 x 56, batch 256: 56.2, 52.9) -- but not for less than a hundred channels in all on
//    large images, where its 128 x 128 tile is mostly padding (24 -> 16, 70 x 70, batch 256: 29.1 against 37.5; 16 -> 40, 62 x 62,
//    batch 40: 11.2, 15.8).
bool wgrad_auto_lines(const WgradArgs& a) {
    if (!wgrad_lines_applies(a)) return false;
    if (!(a.R == 1 && a.S == 1) || (a.Cp >= 128 && a.Kp >= 128) || a.Cp >= 256) return true;
    return (long long)a.N * a.P >= 32ll * a.Q && !(a.Cp + a.Kp <= 96 && a.P * a.Q >= 1024);
}

size_t wgrad_s2d(WgradArgs* a) {
    a->s2d = 0;
    if (!s2d_applies(a->C, a->stride_h, a->stride_w)) return 0;
    const S2dGeo g = s2d_geometry(a->R, a->S, a->pad_h, a->pad_w);
    a->s2d = 1;
    a->oC = a->C; a->oR = a->R; a->oS = a->S; a->oH = a->H; a->oW = a->W;
    a->eh = g.eh;
    a->ew = g.ew;
    a->C = 4 * a->oC;
    a->Cp = 16;
    a->H = (a->H + 1) / 2;
    a->W = (a->W + 1) / 2;
    a->R = g.R2;
    a->S = g.S2;
    a->pad_h = g.ph;
    a->pad_w = g.pw;
    a->stride_h = a->stride_w = 1;        // P and Q stay: the rewritten layer has the same output pixels
    return (size_t)a->N * a->H * a->W * 16;
}

// ---------------------------------------------------------------------------------------------
// Host-side plan: tile shapes, tap grouping, split count.  Shared by the workspace query and the
// launch so that both see the same numbers.
// ---------------------------------------------------------------------------------------------
namespace {
// The plan of the most recent geometry, per host thread: a layer is planned once, not per call.
constexpr int kPlanKey = 17;
struct PlanCache {
    int key[kPlanKey];
    WgradArgs plan;
    bool valid;
};
thread_local PlanCache g_plan_cache = {};

// (s2d: a stem in its space-to-depth form may have the geometry of a plain layer, and takes another kernel)
void plan_key(const WgradArgs* a, int key[kPlanKey]) {
    const int k[kPlanKey] = {a->N, a->C, a->Cp, a->H, a->W, a->K, a->Kp, a->P, a->Q, a->R, a->S,
                             a->stride_h, a->stride_w, a->pad_h, a->pad_w, a->variant, a->s2d};
    for (int i = 0; i < kPlanKey; ++i) key[i] = k[i];
}
void wgrad_plan_uncached(WgradArgs* a);
}  // namespace

void wgrad_plan(WgradArgs* a) {
    int key[kPlanKey];
    plan_key(a, key);
    PlanCache& c = g_plan_cache;
    bool hit = c.valid;
    for (int i = 0; hit && i < kPlanKey; ++i) hit = c.key[i] == key[i];
    if (!hit) {
        wgrad_plan_uncached(a);
        for (int i = 0; i < kPlanKey; ++i) c.key[i] = key[i];
        c.plan = *a;
        c.valid = true;
        return;
    }
    const WgradArgs& p = c.plan;
    a->TB = p.TB; a->CS = p.CS; a->BP = p.BP; a->BQ = p.BQ; a->ntp = p.ntp; a->ntq = p.ntq;
    a->ngrp = p.ngrp; a->chunks = p.chunks; a->splits = p.splits;
    a->ktiles = p.ktiles; a->ctiles = p.ctiles; a->tapgroups = p.tapgroups;
    a->xt_slots = p.xt_slots; a->lds_bytes = p.lds_bytes; a->lines = p.lines; a->xgk = p.xgk; a->xgc = p.xgc; a->pk = p.pk;
    a->by_tiles = p.by_tiles; a->by_taps = p.by_taps; a->by_ctiles = p.by_ctiles; a->by_splits = p.by_splits; a->by_lines = p.by_lines;
    a->t_chunk = p.t_chunk; a->t_partial = p.t_partial;
}

namespace {
void wgrad_plan_uncached(WgradArgs* a) {
    a->lines = 0;
    a->xgk = a->xgc = 0;
    if (a->variant == VAR_WGRAD_LINES || (a->variant != VAR_WGRAD_IMAGES && wgrad_auto_lines(*a))) {
        wgrad_plan_lines(a);
        return;
    }
    const int RS = a->R * a->S;
    // taps per block / channel slabs per wave: one filter row of a 3-wide filter, a whole 1x7 or
    // 7x1 filter, a wide channel tile for 1x1, one tap at a time otherwise
    a->pk = 0;
    if (a->Cp == 16 && RS % 4 == 0) { a->TB = 4; a->CS = 1; a->pk = 1; }      // four taps side by side in the 64 columns
    else if (RS == 1) { a->TB = 1; a->CS = (a->Cp >= 256) ? 4 : 1; }
    else if (RS % 3 == 0 && a->S == 3) { a->TB = 3; a->CS = 1; }
    else if (RS == 7) { a->TB = 7; a->CS = 1; }
    else { a->TB = 1; a->CS = 1; }
    // TB divides R*S in every case, so a tap group is never ragged
    const int CT = a->pk ? 16 : 64 * a->CS;          // channels staged per window pixel
    a->tapgroups = (RS + a->TB - 1) / a->TB;
    a->ktiles = (a->K + W2_BM - 1) / W2_BM;
    a->ctiles = (a->Cp + CT - 1) / CT;
    // Output-pixel tile BP x BQ: the one that covers the most useful pixels per chunk among those
    // whose staged window fits LDS, whose loader tasks fit one per thread and whose pixel count fits
    // the unrolled MFMA steps.  (More pixels per chunk = more MFMAs per barrier pair and per
    // transposed byte; tiles that divide P and Q waste nothing at the edges.)
    int BP = 1, BQ = 1;
    double best_score = -1.0;
    for (int bp = 1; bp <= a->P && bp <= 2 * W2_MAXSTEPS; ++bp) {
        for (int bq = 1; bq <= a->Q && bp * bq <= 2 * W2_MAXSTEPS; ++bq) {
            int maxwin = 0;
            for (int g = 0; g < a->tapgroups; ++g) {
                const int t0 = g * a->TB, nt = (RS - t0 < a->TB) ? (RS - t0) : a->TB;
                int rmin, rmax, smin, smax;
                tap_extent(t0, nt, a->S, &rmin, &rmax, &smin, &smax);
                const int WH = (bp - 1) * a->stride_h + (rmax - rmin) + 1;
                const int WW = (bq - 1) * a->stride_w + (smax - smin) + 1;
                if (WH * WW > maxwin) maxwin = WH * WW;
            }
            const size_t lds = (size_t)(maxwin * (CT + W2_PAD) + (bp * bq + 1) * (W2_BM + W2_PAD)) * 16 +
                               2 * W2_MAXSTEPS * sizeof(int2);
            const int ntask = maxwin * (CT / 16) + bp * bq * 4;   // one loader task per thread
            const bool fits = lds <= (size_t)W2_LDS_BUDGET && ntask <= 256;
            if (!fits && !(bp == 1 && bq == 1)) continue;
            const int ntp = (a->P + bp - 1) / bp, ntq = (a->Q + bq - 1) / bq;
            const double cover = (double)a->P * a->Q / ((double)ntp * bp * ntq * bq);
            // useful pixels per chunk, discounted by the fixed cost of a chunk (about 6 pixels' worth)
            const double score = cover * (bp * bq) / (bp * bq + 6.0);
            if (score > best_score) {
                best_score = score;
                BP = bp;
                BQ = bq;
                a->xt_slots = maxwin * (CT + W2_PAD);
                a->lds_bytes = lds;
            }
        }
    }
    const int np = (a->P + BP - 1) / BP;
    const int nq = (a->Q + BQ - 1) / BQ;
    a->BP = BP;
    a->BQ = BQ;
    a->ntp = np;
    a->ntq = nq;
    a->ngrp = (a->N + 15) / 16;
    a->chunks = a->ngrp * np * nq;
    const int out_tiles = a->ktiles * a->ctiles * a->tapgroups;
    // Split count: the one with the smallest estimated time.  Blocks run in rounds of `slots`
    // (blocks resident on the chip: registers allow two per compute unit for the narrow tiles, one
    // for the wide ones); a block pays a prologue plus its chunks; every split adds one write and
    // one read of the int32 partial tile set.  The constants are rough measurements in microseconds.
    const int acc_tiles = a->pk ? 1 : a->TB * a->CS;
    const int per_cu_regs = acc_tiles == 1 ? 3 : 2;   // by register count of the variants
    int per_cu_lds = (int)((160 * 1024) / a->lds_bytes);
    if (per_cu_lds < 1) per_cu_lds = 1;
    const int slots = 256 * (per_cu_regs < per_cu_lds ? per_cu_regs : per_cu_lds);
    const double t_chunk = 1.2 * per_cu_regs + 0.014 * (BP * BQ + 1) / 2 * acc_tiles;
    const double t_partial = (double)a->K * RS * a->Cp * 8.0 / 4.0e6;
    int splits = 1;
    double best = 1e30;
    for (int sp = 1; sp <= a->chunks && sp <= 4096; ++sp) {
        const long long blocks = (long long)out_tiles * sp;
        const double rounds = (double)((blocks + slots - 1) / slots);
        const double t = rounds * (3.0 + ((a->chunks + sp - 1) / sp) * t_chunk) + sp * t_partial;
        if (t < best) { best = t; splits = sp; }
        if (blocks > 8LL * slots || (long long)a->chunks * (sp + 2) >= (1LL << 31)) break;
    }
    // a caller may ask for half or twice the shares of this choice (per-layer tuning by measurement)
    if (a->variant == VAR_WGRAD_FEWER) splits = splits > 1 ? splits / 2 : 1;
    if (a->variant == VAR_WGRAD_MORE && 2 * splits <= a->chunks && 2 * splits <= 4096 && (long long)a->chunks * (2 * splits) < (1LL << 31)) splits *= 2;
    a->splits = splits;
}
}  // namespace

unsigned wgrad_grid(const WgradArgs& a) {
    const unsigned out_tiles = (unsigned)(a.ktiles * a.ctiles * a.tapgroups);
    return wgrad_xcd_mapping(a.splits) ? out_tiles * 8u * (unsigned)((a.splits + 7) / 8) : out_tiles * (unsigned)a.splits;
}

hipError_t launch_wgrad(const WgradArgs& a_in, hipStream_t st) {
    WgradArgs a = a_in;
    if (a.s2d) {
        if (!a.xs_ready) {
            const hipError_t e = launch_s2d_repack(a.x, a.xs, a.N, a.oH, a.oW, a.oC, nullptr, nullptr, 0, 0, 0, S2dGeo{}, st);
            if (e != hipSuccess) return e;
        }
        a.x = a.xs;
    }
    const dim3 grid(wgrad_grid(a));
    // the staged tiles may exceed the default 64 KB of dynamic LDS: raise the limit once per variant
#define LAUNCH(TBv, CSv, PKv)                                                                                  \
    do {                                                                                                  \
        static std::atomic<unsigned long long> attr_done;                                                 \
        hipError_t ea = raise_dynamic_lds(reinterpret_cast<const void*>(wgrad_kernel<TBv, CSv, PKv>), W2_LDS_BUDGET, \
                                          attr_done);                                                     \
        if (ea != hipSuccess) return ea;                                                                  \
        launch_timed(kt, (wgrad_kernel<TBv, CSv, PKv>), grid, dim3(256), a.lds_bytes, st, a);                \
    } while (0)
    if (a.lines) {
        hipError_t el = launch_wgrad_lines(a, st);
        if (el != hipSuccess) return el;
    } else {
        KernelTimer kt(KID_WGRAD, st);
        if (a.pk) LAUNCH(4, 1, true);
        else if (a.TB == 1 && a.CS == 1) LAUNCH(1, 1, false);
        else if (a.TB == 1 && a.CS == 4) LAUNCH(1, 4, false);
        else if (a.TB == 3) LAUNCH(3, 1, false);
        else if (a.TB == 7) LAUNCH(7, 1, false);
        else return hipErrorInvalidValue;
    }
#undef LAUNCH
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    return launch_wgrad_reduce(a, st);
}

// A block's quads in the flat reduction.  Longer runs read better, but a thread should have all its shares in flight at once (8 loads,
// 256 / Q lanes) and the chip two blocks per compute unit.
static int wgrad_flat_quads(unsigned quads, int splits) {
    int q = 64;
    while (q > 8 && (quads / q < 512 || (long long)splits * q > 8 * 256)) q /= 2;
    return q;
}

hipError_t launch_wgrad_reduce(const WgradArgs& a, hipStream_t st) {
    if (a.direct && a.lines) return hipSuccess;       // (wgrad_lines_tile wrote the result)
    // Shape of the reducing blocks: taps (9, 7 or 3 where they divide R*S; they leave as runs) x channels (64 or 16), the flat kernel, which
    // stores single floats R*S apart, if nothing fits.  A block's threads are channels x (split lanes): 64 channels leave 4 lanes, which
    // is what few shares can keep busy, and their longer runs want the chip just filled; of 16 channels few blocks do, but many
    // shares are many loads for each, and flat blocks are more.  us, 64 channels / 16 / flat:
    //   1x7, 192 -> 768, 4 shares   6.3  6.6  10.2     3x3, 512 -> 160, 3 shares   4.9  6.0   5.1     7x7, 160 -> 192, 3 shares     -   9.1  15.2
    //   3x3, 768 -> 320, 2 shares   7.6 11.7  12.3     3x3, 1024 -> 64, 8 shares   7.1  5.4   5.0     7x1, 512 -> 192, 13 shares  8.8  8.0   7.1
    // Over 260 layers of 3, 7, 9 and 49 taps and 2 to 24 shares this takes 1.010 of the time of the best shape of each (1.13 at most); channels
    // before taps and 1024 blocks for any shape, as it was, 1.074 (2.0 at most).
    const int RS = a.R * a.S;
    int rsc = 1, qn = 0;
    for (const int taps : {9, 7, 3}) {
        if (RS % taps != 0 || rsc > 1) continue;
        auto blocks = [&](int channels) { return a.Cp % channels == 0 ? (long long)((a.K + 3) / 4) * (a.Cp / channels) * (RS / taps) : 0ll; };
        if (a.splits <= 6 && blocks(64) >= 320) qn = 64;
        else if (blocks(16) >= (a.splits <= 12 ? 128 : 1024)) qn = 16;
        if (qn) rsc = taps;
    }
    KernelTimer kt(KID_WGRAD_REDUCE, st);
    if (rsc == 1) {
        const unsigned quads = (unsigned)(wgrad_partial_elems(a) >> 2);       // (fewer than 2^31 weights with their padding: api.hip)
        const int q = wgrad_flat_quads(quads, a.splits);
        const dim3 blocks((quads + q - 1) / q);
        if (q == 64) launch_timed(kt, (wgrad_reduce_flat_kernel<64>), blocks, dim3(256), 0, st, a);
        else if (q == 32) launch_timed(kt, (wgrad_reduce_flat_kernel<32>), blocks, dim3(256), 0, st, a);
        else if (q == 16) launch_timed(kt, (wgrad_reduce_flat_kernel<16>), blocks, dim3(256), 0, st, a);
        else launch_timed(kt, (wgrad_reduce_flat_kernel<8>), blocks, dim3(256), 0, st, a);
        return hipGetLastError();
    }
    const dim3 blocks((unsigned)((a.K + 3) / 4 * (a.Cp / qn) * (RS / rsc)));
#define REDUCE(RSCv)                                                                                         \
    do {                                                                                                     \
        if (qn == 64) launch_timed(kt, (wgrad_reduce_kernel<64, RSCv>), blocks, dim3(256), 0, st, a);      \
        else launch_timed(kt, (wgrad_reduce_kernel<16, RSCv>), blocks, dim3(256), 0, st, a);               \
    } while (0)
    if (rsc == 9) REDUCE(9);
    else if (rsc == 7) REDUCE(7);
    else REDUCE(3);
#undef REDUCE
    return hipGetLastError();
}

}  // namespace int8t
