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
// reads); the next two rounds of 64 channels are on their way meanwhile, two tiles alternate, one barrier per 64 channels.  (With one round
// ahead, zeroed where it was loaded -- which waited for it on the spot -- and addresses of 64 bits, us per call: 144 -> 24 at 56 x 56, batch 64:
// 53.3, now 49.8; 32 -> 16 at 112 x 112: 55.8, 48.1; 16 -> 34 at 96 x 96, batch 43: 33.6, 26.8.  Five blocks per compute unit: no gain.)
// Planes of no whole 16-byte groups: blocks with one round each (infer_1x1_applies(), the grid), whose 32 loads of a float are what they
// wait for; one round ahead, and only if there is one.  150 layers with two empty rounds of loads / so: 1.12 and 0.92 of the time with 64-bit addresses
// (16 -> 8 at 61 x 61, batch 32: 13.3, 9.6 us; 40 -> 24 at 81 x 81, batch 16: 16.0, 12.3; 8 -> 8 at 73 x 73, batch 8: 7.9, 6.2).
#include <algorithm>

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

    float4 f0[2][4], f1[2][4];                           // [half][channel]: four pixels, of this round of 64 channels and the next
    // Loads and stores go through a descriptor that spans one image: channels and filters beyond it, and lanes given an offset beyond
    // it, read zeros and write nothing.  No branches, past the last tile neither (an empty descriptor): the compiler then knows what is
    // outstanding and waits for one round only.
    constexpr uint32_t kOut = 0x80000000u;
    const uint32_t plane = 4u * (uint32_t)a.HW, x_bytes = (uint32_t)a.C * plane, y_bytes = (uint32_t)a.K * plane;
    auto fetch = [&](float4 (&f)[2][4], int tile, int cc) {
        const int n = tile / a.tiles_img, p0 = (tile - n * a.tiles_img) * INF_PIX;
        const __amdgpu_buffer_rsrc_t img = __builtin_amdgcn_make_buffer_rsrc(
            const_cast<float*>(a.x) + (tile < a.tiles ? (size_t)n * a.C * a.HW : (size_t)0), 0, tile < a.tiles ? x_bytes : 0u, 0x00020000);
        const uint32_t row = (uint32_t)(cc * INF_CH + 4 * cgp) * plane;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int p = p0 + 64 * h + 4 * pq;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const uint32_t at = row + (uint32_t)j * plane + 4u * (uint32_t)p;
                if (VEC) {
                    const auto v = __builtin_amdgcn_raw_buffer_load_b128(img, p < a.HW ? at : kOut, 0, 0);
                    f[h][j] = make_float4(__uint_as_float(v[0]), __uint_as_float(v[1]), __uint_as_float(v[2]), __uint_as_float(v[3]));
                } else {
                    float v[4];
#pragma unroll
                    for (int k = 0; k < 4; ++k) v[k] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(img, p + k < a.HW ? at + 4u * k : kOut, 0, 0));
                    f[h][j] = make_float4(v[0], v[1], v[2], v[3]);
                }
            }
        }
    };
    if (tid < 2 * kWave) {
        const float m = absmax_partials_wave(wave ? a.part_w : a.part_x, wave ? a.np_w : a.np_x, lane);
        if (lane == 0) s_max[wave] = m;
    }
    // the rounds of a block, 64 channels of a tile each: the one at work, the next one and the one after it
    int tile = blockIdx.x, cc = 0;
    auto after = [&](int& t, int& c) {
        if (++c == nch) {
            c = 0;
            t += (int)gridDim.x;
        }
    };
    int tile1 = tile, cc1 = 0;
    after(tile1, cc1);
    int tile2 = tile1, cc2 = cc1;
    fetch(f0, tile, 0);
    if (VEC) fetch(f1, tile1, cc1);
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
    auto round = [&](float4 (&f)[2][4], unsigned char* const xb, const unsigned char* const rb) {
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
                *reinterpret_cast<uint32_t*>(xb + (64 * h + 4 * pq + k) * INF_PITCH + 4 * cgp) = o[k];
        }
        if (!VEC && tile1 < a.tiles) fetch(f, tile1, cc1);      // (uniform)
        __syncthreads();      // this tile's codes are there (the first time: the filters' too), the other tile has been read
#pragma unroll
        for (int kk = 0; kk < INF_CH / 32; ++kk) {
            const infer_v4i fb = *reinterpret_cast<const infer_v4i*>(rb + 32 * kk);
#pragma unroll
            for (int r = 0; r < RT; ++r) {
                const infer_v4i fa = *reinterpret_cast<const infer_v4i*>(rw + r * 32 * wpitch + cc * INF_CH + 32 * kk);
                acc[r] = __builtin_amdgcn_mfma_i32_32x32x32_i8(fa, fb, acc[r], 0, 0, 0);
            }
        }
        if (cc + 1 == nch) {
            const int n = tile / a.tiles_img, p = (tile - n * a.tiles_img) * INF_PIX + wave * 32 + (lane & 31);
            const __amdgpu_buffer_rsrc_t img = __builtin_amdgcn_make_buffer_rsrc(a.y + (size_t)n * a.K * a.HW, 0, y_bytes, 0x00020000);
            const uint32_t at = p < a.HW ? (uint32_t)(4 * (lane >> 5)) * plane + 4u * (uint32_t)p : kOut;
#pragma unroll
            for (int r = 0; r < RT; ++r)
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(__fmul_rn((float)acc[r][v], scale)), img,
                                                          at + (uint32_t)(32 * r + 8 * (v >> 2) + (v & 3)) * plane, 0, 0);
                    acc[r][v] = 0;
                }
        }
        // (behind the results: a wait for the next round then does not wait for these loads)
        after(tile2, cc2);
        if (VEC) fetch(f, tile2, cc2);
        tile = tile1;
        cc = cc1;
        tile1 = tile2;
        cc1 = cc2;
    };
    while (tile < a.tiles) {                             // (uniform over the block)
        round(f0, xt, rx);
        if (tile >= a.tiles) break;
        round(VEC ? f1 : f0, xt + INF_TILE, rx + INF_TILE);
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
    if (4ll * a.HW * std::max(a.C, a.K) >= 1ll << 31) return false;       // (one image's descriptor)
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
