// Space-to-depth form of the codes of a stride-2 layer with at most 4 input channels (kernels.h has
// the index algebra).  Channels-last codes keep 16 bytes per pixel however few channels are in use:
// the 7x7 stride-2 stem of an image network on 3 channels would spend 13 of every 16 reduction bytes
// on padding.  The rewritten layer has 4 C channels in the granule and a quarter of the taps; the
// dense kernels then run on it unchanged.  Forward and backward-weight need the same form of the input codes: a step makes it once
// where the forward pass's scratch is known to hold it (int8t_conv_bwd_weight_fwd): 7x7 on 3 channels, 224 x 224, batch 64, the
// whole step 345 -> 331 us; the copy reads 51 MB for 10 MB of codes, 10 us alone and 14 beside other kernels.  A step that forms the
// codes as well writes both forms at once (quantize_s2d_pixels()): only the filters are left to rewrite then.
#include "device_common.h"
#include "kernels.h"

namespace int8t {

// Input codes: byte (2 dy + dx) * C + c of pixel (h', w') is channel c of pixel (2 h' + dy, 2 w' + dx),
// zero where that pixel lies beyond an odd image.
// One thread per output pixel; it reads the first four bytes of four input pixels.
__device__ __forceinline__ void s2d_pixels(const int8_t* __restrict__ x, int8_t* __restrict__ xs, int N, int H, int W, int C,
                                           const unsigned block) {
    const int H2 = (H + 1) >> 1, W2 = (W + 1) >> 1;
    const size_t t = (size_t)block * 256 + threadIdx.x;
    if (t >= (size_t)N * H2 * W2) return;
    const int w2 = (int)(t % W2);
    const size_t nh = t / W2;
    const int h2 = (int)(nh % H2);
    const size_t n = nh / H2;
    const uint32_t* __restrict__ row0 = reinterpret_cast<const uint32_t*>(x) + ((n * H + 2 * h2) * (size_t)W + 2 * w2) * 4;
    const uint32_t* __restrict__ row1 = row0 + (size_t)W * 4;
    const bool w1 = 2 * w2 + 1 < W, h1 = 2 * h2 + 1 < H;     // the block's second column / row exists
    const uint32_t px[4] = {row0[0], w1 ? row0[4] : 0u, h1 ? row1[0] : 0u, (h1 && w1) ? row1[4] : 0u};
    reinterpret_cast<uint4*>(xs)[t] = s2d_pack(px, C);
}

// Filter codes: tap (r', s') of the rewritten filter gathers the taps (2 r' + dy - eh, 2 s' + dx - ew)
// of the layer's own filter in the same channel order; taps outside it are zero.
__device__ __forceinline__ void s2d_filters(const int8_t* __restrict__ w, int8_t* __restrict__ ws, int K, int R, int S, int C, const S2dGeo& g,
                                            const unsigned block) {
    const int t = (int)block * 256 + (int)threadIdx.x;
    if (t >= K * g.R2 * g.S2) return;
    const int s2 = t % g.S2, r2 = (t / g.S2) % g.R2, k = t / (g.S2 * g.R2);
    uint32_t px[4];
#pragma unroll
    for (int b = 0; b < 4; ++b) {
        const int r = 2 * r2 + (b >> 1) - g.eh, s = 2 * s2 + (b & 1) - g.ew;
        const bool ok = r >= 0 && r < R && s >= 0 && s < S;
        px[b] = ok ? reinterpret_cast<const uint32_t*>(w)[((size_t)(k * R + r) * S + s) * 4] : 0u;
    }
    reinterpret_cast<uint4*>(ws)[t] = s2d_pack(px, C);
}

// Both in one launch, the filters' few blocks first (a launch of their own took 4 us).
__global__ __launch_bounds__(256) void s2d_repack_kernel(const int8_t* __restrict__ x, int8_t* __restrict__ xs, int N, int H, int W, int C,
                                                         const int8_t* __restrict__ w, int8_t* __restrict__ ws, int K, int R, int S, S2dGeo g,
                                                         unsigned filter_blocks) {
    raise_wave_priority();
    if (blockIdx.x < filter_blocks) s2d_filters(w, ws, K, R, S, C, g, blockIdx.x);
    else s2d_pixels(x, xs, N, H, W, C, blockIdx.x - filter_blocks);
}

hipError_t launch_s2d_repack(const int8_t* x, int8_t* xs, int N, int H, int W, int C, const int8_t* w, int8_t* ws, int K, int R, int S,
                             const S2dGeo& g, hipStream_t st) {
    const size_t npix = x ? (size_t)N * ((H + 1) / 2) * ((W + 1) / 2) : 0;
    const unsigned filter_blocks = w ? (unsigned)((K * g.R2 * g.S2 + 255) / 256) : 0u;
    KernelTimer kt(KID_S2D_REPACK, st);
    launch_timed(kt, s2d_repack_kernel, dim3(filter_blocks + (unsigned)((npix + 255) / 256)), dim3(256), 0, st, x, xs, N, H, W, C, w, ws, K, R, S, g,
                 filter_blocks);
    return hipGetLastError();
}

}  // namespace int8t
