// The three convolutions of a training step (forward, backward-data, backward-weight), or the two backward ones, in one
// launch.  They depend on the codes of a, W and g_z only, not on one another.
//
// Bound: a small layer's passes are bound by the latency of their tiles' load-multiply stages and by launches, not by a rate:
// 3x3 on 256 channels at 14 x 14, batch 64, has 400 tiles of 128 x 64 per pass for 256 compute units, each about 36 stages
// of 0.5 us.  Side by side the passes fill the compute units that each of them leaves idle.  The tiles are those of the
// kernels that run the passes alone (igemm_dma_tile, wgrad_lines_tile); block ranges deal them: backward-weight first, whose
// blocks live longest.  All forms take 72 KB of LDS at most, so two blocks fit a compute unit.
#include <algorithm>

#include "conv_igemm_dma.h"
#include "conv_wgrad_lines.h"
#include "conv_wgrad_tile.h"

namespace int8t {

namespace {
struct TrioBlocks {
    unsigned wgrad, wgrad8, fwd;     // backward-weight's blocks, and rounded up to the 8 XCDs; the forward pass's
    bool fwd64, bwd64;               // 64 x 128 tiles (conv_trio_tile)
};
template <bool DGRAD, int BN, bool STG>
__device__ __forceinline__ void trio_pass(const IgemmArgs& a, bool rows64, unsigned block) {
    if (rows64) igemm_dma_tile<DGRAD, 1, 8, 2, false, false, 128, false, STG, 4>(a, block);
    else igemm_dma_tile<DGRAD, 2, 8, 2, false, false, BN, false, STG>(a, block);
}
// ST = 0: backward-weight on image granules, one tap and 64 channels per block (narrow 1x1 layers)
constexpr int trio_wt(int ST) { return ST == 1 ? 2 : 1; }
constexpr int trio_gp(int ST) { return ST == 1 ? 4 : ST == 5 ? 6 : 8; }
template <int BN, int ST>
constexpr size_t trio_lds() {
    if (ST == 0) return W2_LDS_BUDGET;
    return std::max((size_t)2 * (128 + BN) * 8 * 16, (size_t)WL_NSTAGE * wl_stage_bytes(trio_wt(ST), trio_wt(ST), trio_gp(ST)));
}
}  // namespace

// ST taps along backward-weight's lines; STG: results of whole 16-byte groups staged through LDS (igemm_dma_tile).
template <int BN, int ST, bool STG>
__global__ __launch_bounds__(256, 2) void conv_trio_kernel(const IgemmArgs f, const IgemmArgs b, const WgradArgs w, const TrioBlocks n) {
    const unsigned block = blockIdx.x;
    if (block < n.wgrad8) {
        if (block >= n.wgrad) return;
        if constexpr (ST == 0) wgrad_tile<1, 1>(w, block);
        else wgrad_lines_tile<ST, trio_wt(ST), trio_wt(ST), trio_gp(ST)>(w, block);
    } else if (block < n.wgrad8 + n.fwd) {
        trio_pass<false, BN, STG>(f, n.fwd64, block - n.wgrad8);
    } else {
        trio_pass<true, BN, STG>(b, n.bwd64, block - n.wgrad8 - n.fwd);
    }
}

// Which layers, and with which tile.  Over 200 random stride-1 layers of 1 to 350 MB, us for the three passes one by one, on
// 128 x 64 tiles together and on 128 x 128 tiles together:
//   3x3, 256 channels, 14 x 14, batch 64            57.6   50.4   45.7      7 x 7, 512 channels, 3x3, batch 64   78.9  51.3  58.3
//   5x5, 48 -> 64 channels, 35 x 35, batch 32       52.2   37.5   42.8      1x1, 960 -> 160, 7 x 7, batch 64     29.4  17.2  19.4
//   1x1, 1024 -> 256, 14 x 14, batch 128            67.9   61.2   53.9      3x3, 16 -> 32, 16 x 16, batch 2      20.6   8.9   9.7
//   3x3, 64 channels, 56 x 56, batch 64             57.2   92.1   75.6      1x7, 768 channels, 17 x 17, batch 64  267   328   277
// One by one stay (the last row): passes that the filter-bank-resident kernels run with many tiles (more than 4000 of 64
// columns over both; the 128-row tiles are half empty there and fetch every pixel once per tap), and passes that fill the chip
// with 256 x 256 tiles.  The wider tile where the work per block slot (512 of them) exceeds 1.2 times the longest reduction: below,
// the time is one tile's chain of stages, and the narrow tile's is shorter.  Against the best of the three per layer this
// rule loses 1.3 % on average, 19 % at most.  The two backward passes alone (a forward pass ran earlier; 104 random layers:
// 7x1, 76 -> 216 channels, 65 x 65, batch 3: 33.0, 21.7, 22.6): up to 3000 such tiles, the wider tile from twice the longest
// reduction on; loses 1.9 % on average, 13 % at most.  Layers whose backward-weight works on image granules (narrow 1x1 layers,
// 2x2 and the like; 100 random ones: 1x1, 64 channels, 56 x 56, batch 2, 18.7, 10.1, 9.9; 96 -> 576 at 14 x 14, batch 64,
// 32.9, 25.0, 25.5; 24 -> 144 at 56 x 56, 53.9, 71.0, 57.9): up to 3000 tiles as well.
//
// Passes that alone run as a split reduction (few tiles, long reductions; with the caller's scratch) have one tile's whole chain of
// stages in here, about 1 us each beside backward-weight's blocks, against 15 - 25 us for the split.  Of 200 random ones, us
// for the three passes one by one and all in one launch:
//   5x5, 1024 channels, 10 x 10, batch 1             260    354      3x3, 120 -> 816, 5 x 5, batch 1               32.0   40.5
//   5x5, 128 -> 1016, 15 x 15, batch 1              85.6    158      5x5, 384 -> 512, 15 x 15, batch 14             164    135
//   5x5, 1024 -> 96, 8 x 8, batch 4                 67.0    128      5x5, 328 -> 272, 15 x 15, batch 5              159    128
// The forward pass alone splits: it runs ahead and the two backward ones share the launch (conv_trio_fwd_apart; 59.2 on the third
// layer of the left column), unless backward-data's chain, which stays whole, is nearly as long (the last layer: 146 that way).
// Backward-data splits: one by one, unless its chain is fewer than 45 stages longer than that of a forward pass that stays whole;
// without the forward pass one by one always (0.81 of the shared launch's time on average, 7 % slower at most).  Over the 200 the
// three passes take 0.93 of the time one by one on average and 1.07 at most, 0.89 and 1.10 of the time all in one launch.
static long long trio_stages(const IgemmArgs& a) { return ((long long)a.R * a.S * (a.Ca >> 4) + 7) / 8; }
bool conv_trio_fwd_apart(const IgemmArgs& fwd, const IgemmArgs& bwd) {
    return igemm_splits(fwd) && !igemm_splits(bwd) && 5 * trio_stages(fwd) >= 8 * trio_stages(bwd);
}
// Passes of at most 64 rows leave half of every 128-row tile empty: they take 64 x 128 tiles (four waves of 64 x 32) instead, where the
// work per block slot, counted with these, makes up for the chain of stages of one tile, which is 5 - 10 % longer than that
// of a 128 x 64 tile: from 0.4 times the longest reduction on where all passes are that narrow, on the launch whose blocks fit
// a compute unit three times; from 0.55 times on beside a wider pass, with the wider tile for that one; the two backward passes
// alone from 0.45 on.  Over 290 random such layers, the three passes, us before and now:
//   5x5, 48 -> 64, 35 x 35, batch 32    41.7   35.6      3x3, 64 channels, 28 x 28, batch 64     26.6   23.1
//   5x5, 32 -> 64, 28 x 28, batch 32    27.0   21.5      3x3, 32 -> 29, 21 x 21, batch 256       42.1   33.5
//   3x3, 40 -> 186, 28 x 28, batch 256  144.7  128.8     3x3, 408 -> 8, 9 x 9, batch 256         42.6   36.5
// all narrow 0.86 of the time before on average, mixed 0.97, the two backward ones 0.95, none slower.  64 x 256 tiles gained
// nothing (5x5, 48 -> 64: 40.5).
TrioTile conv_trio_tile(const IgemmArgs* fwd, const IgemmArgs& bwd, const WgradArgs& w) {
    const TrioTile apart{0, false};
    if (w.variant != VAR_AUTO || w.s2d || !(w.lines || (w.TB == 1 && w.CS == 1 && !w.pk))) return apart;
    if (igemm_splits(bwd)) {
        if (!fwd) return apart;
        const bool both = igemm_splits(*fwd);
        const long long f = trio_stages(*fwd), b = trio_stages(bwd);
        if (both ? std::max(f, b) >= 45 : b >= 45 + f) return apart;
    }
    long long band_tiles = 0, work = 0, longest = 0;
    long long work64 = 0;                 // in half units: a pass of at most 64 rows on 64 x 128 tiles
    int narrow = 0, passes = 0;
    for (const IgemmArgs* a : {fwd, &bwd}) {
        if (!a) continue;
        if (a->variant != VAR_AUTO || a->stride_h != 1 || a->stride_w != 1) return apart;
        const int v = igemm_auto_variant(*a);
        if (v == VAR_WIDE256) return apart;
        const long long tiles = (((long long)a->N * a->OH * a->OW + 63) / 64) * ((a->rows + 127) / 128);
        const long long gran = (long long)a->R * a->S * (a->Ca >> 4);
        if (v == VAR_BAND) band_tiles += tiles;
        work += tiles * gran;
        work64 += (a->rows <= 64 ? 1 : 2) * tiles * gran;
        narrow += a->rows <= 64;
        ++passes;
        longest = std::max(longest, gran);
    }
    // in hundredths of (512 block slots x the longest reduction), against twice the work64 units
    const long long least = !fwd ? 45 : narrow == passes ? 40 : 55;
    const bool rows64 = narrow > 0 && 100 * work64 >= 2 * least * 512 * longest;
    // (narrow 1x1 layers also where backward-weight works on lines: 24 -> 144 at 56 x 56, batch 64, 3136 tiles: 54 either way)
    const bool narrow1 = w.R * w.S == 1 && !(w.Cp >= 128 && w.Kp >= 128) && !(w.Cp >= 256 && w.Kp >= 64);
    if (band_tiles > (fwd && w.lines && !narrow1 ? 4000 : 3000)) return apart;
    if (rows64) return TrioTile{narrow == passes ? 64 : 128, true};
    return TrioTile{5 * work >= (fwd ? 6 : 10) * 512 * longest ? 128 : 64, false};
}

// When `count` blocks of one length after another have been dealt to the slots that are free first; returns the end of the last.
namespace {
struct SlotClock {
    double at[4];        // the slots by the time they are free from: one more time per deal, three passes at most
    int n[4], size = 1;
    explicit SlotClock(int slots) { at[0] = 0.0; n[0] = slots; }
    double deal(long long count, double length) {
        double end = 0.0;
        while (count > 0) {
            int i = 0;
            for (int k = 1; k < size; ++k)
                if (at[k] < at[i]) i = k;
            if (count >= n[i]) {
                count -= n[i];
                at[i] += length;
            } else {
                at[size] = at[i] + length;
                n[size++] = (int)count;
                n[i] -= (int)count;
                end = std::max(end, at[size - 1]);
                break;
            }
            end = std::max(end, at[i]);
        }
        return end;
    }
};
}  // namespace

// Backward-weight's shares in a shared launch: what it takes by itself, or fewer where the tiles of the other passes fill the chip anyway.
// By itself the pass has to fill 512 block slots; in here every share costs a block's setup and a partial tile to write and to read, and the last
// turn of the slots may hold a few blocks only.  One share leaves the reduction's launch out.  The estimate deals the blocks to the slots in
// the order of the launch; its constants are fitted to the two and the three passes of 50 layers of 1 to 60 GOP with 1, 0.7, 0.5, 0.35 and 0.25 of the
// shares (units of their own: only the order of the estimates counts).  Fewer where the estimate falls by a tenth, not below a half but for one: over
// these layers 0.97 of the time with all the shares on average and 1.015 at most (from a fiftieth on 0.95, but 1.09 at most).  us with all and as chosen:
//   3x3, 512 channels, 7 x 7, batch 64, two             40.5   28.6      3x3, 215 -> 197, 15 x 15, batch 6, three                   19.1   13.3
//   7x1, 130 -> 959, 34 x 34, batch 7, two              53.5   44.8      3x3 under stride 2, 677 -> 365, 19 x 19, batch 10, three   54.8   39.6
static int trio_shares(const IgemmArgs* fwd, const IgemmArgs& bwd, const WgradArgs& w, TrioTile tile) {
    if (!w.lines || w.splits <= 1) return w.splits;
    auto estimate = [&](int shares) {
        SlotClock clock(512);
        const double length = 2.38 + (double)((w.chunks + shares - 1) / shares) * w.t_chunk * 2.37;
        double end = clock.deal((long long)w.ktiles * w.ctiles * w.tapgroups * shares, length);
        for (const IgemmArgs* a : {fwd, &bwd}) {
            if (!a) continue;
            const bool half = tile.rows64 && a->rows <= 64;       // 64 x 128 tiles
            const int cols = half ? 128 : tile.bn;
            const long long tiles = (((long long)a->N * a->OH * a->OW + cols - 1) / cols) * ((a->rows + (half ? 63 : 127)) / (half ? 64 : 128));
            const int taps = a->dgrad ? a->stride_h * a->stride_w : 1;      // (a pixel of a strided backward-data pass meets one class of taps)
            const int stages = (a->R * a->S * (a->Ca >> 4) + 8 * taps - 1) / (8 * taps);
            end = std::max(end, clock.deal(tiles, 1.46 + stages * 1.51 * (0.35 + 0.65 * (half ? 0.5 : tile.bn / 128.0))));
        }
        WgradArgs t = w;
        t.splits = shares;
        return end + shares * (double)w.t_partial * 1.11 + (wgrad_single_share(t) ? 0.0 : 10.39);
    };
    int best = w.splits;
    double least = estimate(w.splits);
    const double all = least;
    for (const int part : {70, 50, 35, 25}) {
        const int shares = std::max(1, (w.splits * part + 50) / 100);
        if (part < 50 && shares > 1) continue;
        const double t = estimate(shares);
        if (t * 1.1 < all && t < least) {
            least = t;
            best = shares;
        }
    }
    return best;
}

// (the estimate takes 0.2 us of the host for layers of a few hundred tiles, 1.4 us for tens of thousands)
static void set_trio_shares(WgradArgs* w, const IgemmArgs* fwd, const IgemmArgs& bwd, TrioTile tile) {
    const int shares = trio_shares(fwd, bwd, *w, tile);
    if (shares == w->splits) return;
    w->splits = shares;
    w->by_splits = fast_div((unsigned)shares);
    w->direct = wgrad_single_share(*w);         // (passes that share a launch overlap nothing)
}

hipError_t launch_conv_trio(const IgemmArgs* fwd, const IgemmArgs& bwd, const WgradArgs& w_all, TrioTile tile, hipStream_t st) {
    WgradArgs w = w_all;
    set_trio_shares(&w, fwd, bwd, tile);
    const int bn = tile.bn;
    IgemmArgs f = fwd ? *fwd : bwd, b = bwd;
    TrioBlocks n;
    n.wgrad = w.lines ? wgrad_lines_grid(w) : wgrad_grid(w);
    n.wgrad8 = (n.wgrad + 7) & ~7u;
    n.fwd64 = tile.rows64 && f.rows <= 64;
    n.bwd64 = tile.rows64 && b.rows <= 64;
    n.fwd = fwd ? igemm_plain_blocks(&f, n.fwd64 ? 64 : 128, n.fwd64 ? 128 : bn) : 0;
    const unsigned nb = igemm_plain_blocks(&b, n.bwd64 ? 64 : 128, n.bwd64 ? 128 : bn);
    if ((fwd && !n.fwd) || !nb) return hipErrorInvalidValue;
    const dim3 grid(n.wgrad8 + n.fwd + nb);
    const bool stg = ((f.OH * f.OW) & 3) == 0 && ((b.OH * b.OW) & 3) == 0;
    KernelTimer kt(KID_CONV_TRIO, st);
#define LAUNCH(BNv, STv, STGv)                                                                                                     \
    do {                                                                                                                           \
        static std::atomic<unsigned long long> attr_done;                                                                         \
        const hipError_t e = raise_dynamic_lds(reinterpret_cast<const void*>(conv_trio_kernel<BNv, STv, STGv>), (int)trio_lds<BNv, STv>(), attr_done); \
        if (e != hipSuccess) return e;                                                                                             \
        launch_timed(kt, (conv_trio_kernel<BNv, STv, STGv>), grid, dim3(256), trio_lds<BNv, STv>(), st, f, b, w, n);               \
    } while (0)
#define LAUNCH_ST(BNv, STv) do { if (stg) LAUNCH(BNv, STv, true); else LAUNCH(BNv, STv, false); } while (0)
#define LAUNCH_BN(STv) do { if (bn == 64) LAUNCH_ST(64, STv); else LAUNCH_ST(128, STv); } while (0)
    if (!w.lines) LAUNCH_BN(0);
    else if (w.TB == 1) LAUNCH_BN(1);
    else if (w.TB == 3) LAUNCH_BN(3);
    else if (w.TB == 5) LAUNCH_BN(5);
    else if (w.TB == 7) LAUNCH_BN(7);
    else return hipErrorInvalidValue;
#undef LAUNCH_BN
#undef LAUNCH_ST
#undef LAUNCH
    const hipError_t e = hipGetLastError();
    return e != hipSuccess ? e : launch_wgrad_reduce(w, st);
}

// ---------------------------------------------------------------------------------------------
// The same for strided layers whose backward-weight works on image lines (3x3 under stride 2 x 2, 1x1 without padding).  The tiles are
// the 128 x 64 ones; backward-data in the form it takes by itself: the pixel classes of a cell one after the other in a
// block, cells with one class of taps, a class per tile, or plain.
// Over 100 random such layers, us for the three passes one by one and in one launch (0.70 on average), and for the two backward ones (0.77):
//   3x3, 128 channels, 56 x 56, batch 64       79.0   73.0     60.6   53.8     1x1, 1024 -> 2048, 14 x 14, batch 64   70.5  60.4  50.6  49.7
//   3x3, 256 channels, 28 x 28, batch 64       72.3   62.0     53.4   48.5     1x1, 544 -> 164, 9 x 9, batch 30       25.1  14.1  19.1  13.3
//   3x3, 192 -> 320, 17 x 17, pad 0, batch 64  51.2   34.7     39.0   30.2     3x3, 16 -> 32, 16 x 16, batch 2        16.8   8.8  12.9   8.8
// Apart stay 1x1 layers of many tiles, which are bound by writing results that the wider tiles alone write through LDS
// (8 -> 360, 31 x 31, batch 216, 5800 tiles: 53.6 against 62.9), passes on 256 x 256 tiles and split reductions.
// ---------------------------------------------------------------------------------------------
template <int FORM, bool S2>
__global__ __launch_bounds__(256, 2) void conv_trio_strided_kernel(const IgemmArgs f, const IgemmArgs b, const WgradArgs w, const TrioBlocks n) {
    const unsigned block = blockIdx.x;
    if (block < n.wgrad8) {
        if (block >= n.wgrad) return;
        if constexpr (S2) wgrad_lines_tile<3, 1, 1, 3, true>(w, block);
        else wgrad_lines_tile<1, 2, 2, 4>(w, block);
    } else if (block < n.wgrad8 + n.fwd) {
        igemm_dma_tile<false, 2, 8, 2, false, false, 64>(f, block - n.wgrad8);
    } else {
        constexpr bool CLS = FORM != STRIDED_PLAIN, CELL = FORM == STRIDED_CELL || FORM == STRIDED_CELLS;
        igemm_dma_tile<true, 2, 8, 2, CLS, CELL, 64, FORM == STRIDED_CELLS>(b, block - n.wgrad8 - n.fwd);
    }
}

bool conv_trio_strided(const IgemmArgs* fwd, const IgemmArgs& bwd, const WgradArgs& w) {
    if (w.variant != VAR_AUTO || w.s2d || !w.lines || !(w.TB == 1 || wgrad_lines_s2(w))) return false;
    long long tiles = 0;
    for (const IgemmArgs* a : {fwd, &bwd}) {
        if (!a) continue;
        if (a->variant != VAR_AUTO || igemm_splits(*a) || igemm_auto_variant(*a) == VAR_WIDE256) return false;
        const long long pixels = (long long)a->N * a->OH * a->OW;
        tiles += (pixels + 63) / 64 * ((a->rows + 127) / 128);
    }
    return w.TB == 3 || tiles <= 4500;
}

hipError_t launch_conv_trio_strided(const IgemmArgs* fwd, const IgemmArgs& bwd, const WgradArgs& w_all, hipStream_t st) {
    WgradArgs w = w_all;
    set_trio_shares(&w, fwd, bwd, TrioTile{64, false});
    IgemmArgs f = fwd ? *fwd : bwd, b = bwd;
    TrioBlocks n{};
    n.wgrad = wgrad_lines_grid(w);
    n.wgrad8 = (n.wgrad + 7) & ~7u;
    n.fwd = fwd ? igemm_plain_blocks(&f, 128, 64) : 0;
    int form = STRIDED_PLAIN;
    const unsigned nb = igemm_strided_blocks(&b, &form);
    if ((fwd && !n.fwd) || !nb) return hipErrorInvalidValue;
    const bool s2 = w.TB == 3;
    const dim3 grid(n.wgrad8 + n.fwd + nb);
    const size_t lds = std::max((size_t)2 * (128 + 64) * 8 * 16, w.lds_bytes);
    KernelTimer kt(KID_CONV_TRIO, st);
#define LAUNCH(Fv, S2v)                                                                                                            \
    do {                                                                                                                           \
        static std::atomic<unsigned long long> attr_done;                                                                         \
        const hipError_t e = raise_dynamic_lds(reinterpret_cast<const void*>(conv_trio_strided_kernel<Fv, S2v>), 72 * 1024, attr_done); \
        if (e != hipSuccess) return e;                                                                                             \
        launch_timed(kt, (conv_trio_strided_kernel<Fv, S2v>), grid, dim3(256), lds, st, f, b, w, n);                               \
    } while (0)
    // (3x3 filters have four classes of taps, 1x1 filters one)
    if (s2 && form == STRIDED_CELLS) LAUNCH(STRIDED_CELLS, true);
    else if (s2 && form == STRIDED_CLASSES) LAUNCH(STRIDED_CLASSES, true);
    else if (s2 && form == STRIDED_PLAIN) LAUNCH(STRIDED_PLAIN, true);
    else if (!s2 && form == STRIDED_CELL) LAUNCH(STRIDED_CELL, false);
    else if (!s2 && form == STRIDED_PLAIN) LAUNCH(STRIDED_PLAIN, false);
    else return hipErrorInvalidValue;
#undef LAUNCH
    const hipError_t e = hipGetLastError();
    return e != hipSuccess ? e : launch_wgrad_reduce(w, st);
}

}  // namespace int8t
