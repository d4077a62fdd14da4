// Forward pass of a 1x1 layer whose codes nobody wants afterwards (a network in use, no gradients): Eq.1 of activations and weights
// inside the convolution, from the fp32 tensors.
//
// Bound: HBM, the fp32 activations and results.  Quantizing first writes a code per activation and reads it back -- 115 MB in, 29
// out, 29 in and 19 out for 144 -> 24 channels at 56 x 56, batch 64 -- and is a launch of its own; a filter bank that fits LDS
// reads every activation once anyway, so nothing speaks for codes in memory.
//
// A block keeps the filter bank's codes in LDS (quantized there, from the partial maxima) and walks tiles of 128 pixels, 64 channels at
// a time: a thread loads 2 x 4 channels x 4 pixels, quantizes, turns them round in registers as the quantizer does, and leaves
// four channels per pixel in an LDS tile ([pixel][80 bytes]: an odd number of 16-byte granules, conflict-free operand
// reads); the next 64 channels are on their way meanwhile, two tiles alternate, one barrier per 64 channels.
#include "device_common.h"
#include "kernels.h"

namespace int8t {

typedef int infer_v4i __attribute__((ext_vector_type(4)));
typedef int infer_v16i __attribute__((ext_vector_type(16)));

constexpr int INF_PIX = 128, INF_CH = 64, INF_PITCH = INF_CH + 16;
constexpr int INF_TILE = INF_PIX * INF_PITCH;            // bytes of one LDS tile of codes
constexpr int INF_BANK = 64 * (4 * INF_CH + 16);         // ... of the largest filter bank's codes

// Blocks per compute unit (by registers)
constexpr int inf_blocks(int RT) { return RT == 1 ? 4 : 3; }

// RT: 32-row tiles of filters; VEC: planes of whole 16-byte groups
template <int RT, bool VEC>
__global__ __launch_bounds__(256, inf_blocks(RT)) void infer_1x1_kernel(const InferArgs a) {
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
    __shared__ float s_max[2];
    raise_wave_priority();
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int pq = tid & 15, cgp = tid >> 4;             // this thread's pixel quad (of either half of a tile) and channels 4 * cgp ..
    const int nch = (a.C + INF_CH - 1) / INF_CH;
    const int wpitch = nch * INF_CH + 16;                // an odd number of granules
    unsigned char* const xt = lds;                       // two tiles of codes
    unsigned char* const wt = lds + 2 * INF_TILE;        // [RT * 32][wpitch]

    float4 f[2][4];                                      // [half][channel]: four pixels
    auto fetch = [&](int tile, int cc) {
        const int n = tile / a.tiles_img, p0 = (tile - n * a.tiles_img) * INF_PIX;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int p = p0 + 64 * h + 4 * pq;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int c = cc * INF_CH + 4 * cgp + j;
                const size_t at = ((size_t)n * a.C + c) * a.HW + p;
                // (unconditional loads: what is not there re-reads the first floats and is zeroed)
                if (VEC) {
                    const bool ok = c < a.C && p < a.HW;
                    f[h][j] = *reinterpret_cast<const float4*>(a.x + (ok ? at : (size_t)0));
                    if (!ok) f[h][j] = make_float4(0.f, 0.f, 0.f, 0.f);
                } else {
                    float v[4];
#pragma unroll
                    for (int k = 0; k < 4; ++k) {
                        const bool ok = c < a.C && p + k < a.HW;
                        v[k] = a.x[ok ? at + k : (size_t)0];
                        if (!ok) v[k] = 0.0f;
                    }
                    f[h][j] = make_float4(v[0], v[1], v[2], v[3]);
                }
            }
        }
    };
    int tile = blockIdx.x, cc = 0;
    if (tid < 2 * kWave) {
        const float m = absmax_partials_wave(wave ? a.part_w : a.part_x, wave ? a.np_w : a.np_x, lane);
        if (lane == 0) s_max[wave] = m;
    }
    if (tile < a.tiles) fetch(tile, 0);
    __syncthreads();
    const float inv_x = inv_scale_of(s_max[0]), inv_w = inv_scale_of(s_max[1]);
    const float scale = __fmul_rn(scale_of(s_max[0]), scale_of(s_max[1]));
    {
        // the filter bank's codes, four channels at a time, zeros beyond it
        const int per_row = nch * (INF_CH / 4);
        for (int i = tid; i < RT * 32 * per_row; i += 256) {
            const int k = i / per_row, c = 4 * (i - k * per_row);
            float v[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const bool ok = k < a.K && c + j < a.C;
                v[j] = a.w[ok ? (size_t)k * a.C + c + j : (size_t)0];
                if (!ok) v[j] = 0.0f;
            }
            *reinterpret_cast<uint32_t*>(wt + k * wpitch + c) =
                pack4(quantize_one<false>(v[0], inv_w, 0u, 0u, 0u), quantize_one<false>(v[1], inv_w, 0u, 0u, 0u),
                      quantize_one<false>(v[2], inv_w, 0u, 0u, 0u), quantize_one<false>(v[3], inv_w, 0u, 0u, 0u));
        }
    }
    infer_v16i acc[RT];
#pragma unroll
    for (int r = 0; r < RT; ++r)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[r][v] = 0;
    const unsigned char* const rx = xt + (wave * 32 + (lane & 31)) * INF_PITCH + 16 * (lane >> 5);
    const unsigned char* const rw = wt + (lane & 31) * wpitch + 16 * (lane >> 5);
    int buf = 0;
    while (tile < a.tiles) {                             // (uniform over the block)
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            uint32_t d[4], o[4];
#pragma unroll
            for (int j = 0; j < 4; ++j)
                d[j] = pack4(quantize_one<false>(f[h][j].x, inv_x, 0u, 0u, 0u), quantize_one<false>(f[h][j].y, inv_x, 0u, 0u, 0u),
                             quantize_one<false>(f[h][j].z, inv_x, 0u, 0u, 0u), quantize_one<false>(f[h][j].w, inv_x, 0u, 0u, 0u));
            transpose4x4_bytes(d, o);                    // d[channel] = 4 pixels -> o[pixel] = 4 channels
#pragma unroll
            for (int k = 0; k < 4; ++k)
                *reinterpret_cast<uint32_t*>(xt + buf * INF_TILE + (64 * h + 4 * pq + k) * INF_PITCH + 4 * cgp) = o[k];
        }
        const int now = tile, cnow = cc;
        if (++cc == nch) {
            cc = 0;
            tile += (int)gridDim.x;
        }
        if (tile < a.tiles) fetch(tile, cc);
        __syncthreads();      // this tile's codes are there (the first time: the filters' too), the other tile has been read
#pragma unroll
        for (int kk = 0; kk < INF_CH / 32; ++kk) {
            const infer_v4i fb = *reinterpret_cast<const infer_v4i*>(rx + buf * INF_TILE + 32 * kk);
#pragma unroll
            for (int r = 0; r < RT; ++r) {
                const infer_v4i fa = *reinterpret_cast<const infer_v4i*>(rw + r * 32 * wpitch + cnow * INF_CH + 32 * kk);
                acc[r] = __builtin_amdgcn_mfma_i32_32x32x32_i8(fa, fb, acc[r], 0, 0, 0);
            }
        }
        buf ^= 1;
        if (cnow + 1 < nch) continue;
        const int n = now / a.tiles_img, p = (now - n * a.tiles_img) * INF_PIX + wave * 32 + (lane & 31);
#pragma unroll
        for (int r = 0; r < RT; ++r)
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int k = 32 * r + 8 * (v >> 2) + 4 * (lane >> 5) + (v & 3);
                if (k < a.K && p < a.HW) a.y[((size_t)n * a.K + k) * a.HW + p] = __fmul_rn((float)acc[r][v], scale);
                acc[r][v] = 0;
            }
    }
}

// Which layers (70 random ones with at most 64 filters, us for max|.|, codes and convolution / here): up to 256 channels, where a
// tile is at most four rounds of loads (400 channels, 8 x 8, batch 32: 15.0, 24.8), on planes of whole 16-byte groups; a filter bank of
// more than 8 K elements, which every block quantizes, only where a block has tiles enough to pay for it (256 -> 64 at 14 x 14, batch 64,
// 128 tiles: 17.9, 19.8; at 56 x 56: 95.3, 87.4).  144 -> 24 at 56 x 56, batch 64: 60.1, 50.7; 32 -> 16 at 112 x 112: 70.6, 53.2;
// 64 -> 32 at 14 x 14, batch 135: 15.5, 9.5.  Other planes load float by float and gain what the launch saves, up to one round of tiles
// of 64 channels (40 -> 8 at 19 x 19, batch 55: 12.7, 8.5; 8 -> 8 at 47 x 47, batch 256, 4608 tiles: 35.1, 47.2).
bool infer_1x1_applies(const InferArgs& a) {
    if (a.K > 64 || a.C > 4 * INF_CH || a.HW < 64) return false;
    const long long tiles = (long long)a.N * ((a.HW + INF_PIX - 1) / INF_PIX);
    if ((a.HW & 3) == 0) return (long long)a.K * a.C <= 8192 || tiles >= 512;
    return a.C <= INF_CH && a.K <= 32 && tiles <= 1024;
}

hipError_t launch_infer_1x1(const InferArgs& in, hipStream_t st) {
    InferArgs a = in;
    a.tiles_img = (a.HW + INF_PIX - 1) / INF_PIX;
    a.tiles = a.tiles_img * a.N;
    const int nch = (a.C + INF_CH - 1) / INF_CH, rt = a.K <= 32 ? 1 : 2;
    const size_t lds = 2 * (size_t)INF_TILE + (size_t)rt * 32 * (nch * INF_CH + 16);
    // whole rounds of resident blocks
    const int slots = 256 * inf_blocks(rt), rounds = (a.tiles + slots - 1) / slots, blocks = (a.tiles + rounds - 1) / rounds;
    KernelTimer kt(KID_INFER, st);
#define LAUNCH(RTv, VECv)                                                                                               \
    do {                                                                                                                \
        static std::atomic<unsigned long long> attr_done;                                                               \
        const hipError_t e = raise_dynamic_lds(reinterpret_cast<const void*>(infer_1x1_kernel<RTv, VECv>), 2 * INF_TILE + INF_BANK, attr_done); \
        if (e != hipSuccess) return e;                                                                                  \
        launch_timed(kt, (infer_1x1_kernel<RTv, VECv>), dim3(blocks), dim3(256), lds, st, a);                           \
    } while (0)
    const bool vec = (a.HW & 3) == 0;
    if (rt == 1) { if (vec) LAUNCH(1, true); else LAUNCH(1, false); }
    else { if (vec) LAUNCH(2, true); else LAUNCH(2, false); }
#undef LAUNCH
    return hipGetLastError();
}

}  // namespace int8t
