// Depthwise 3x3 layers under stride 1 and "same" padding: quantization and convolutions in one pass over the fp32 tensors.
//
// Bound: HBM.  The passes one after the other move, per element of a and of g_z together, 8 bytes into the quantizer and 2 out of
// it, those 2 bytes twice into the convolutions (forward and backward-data, then backward-weight) and 8 out of them.  A
// depthwise result depends on one plane only, so a block that holds the codes of a plane of a and of the same plane of g_z in
// LDS has everything the three passes need: the codes are written for whoever wants them and never read back (18 bytes
// per element instead of 22, and one launch instead of two), and a window of a cut out of LDS serves a forward output and a
// tap of backward-weight alike.
//
// A block takes one channel (or `cg` consecutive ones of small planes, one contiguous run per image) through a share of the
// batch: its nine backward-weight sums stay in registers, the next image's floats are on their way while this image's products
// run.  Half of the passes (XQ: codes of a and W, forward; GQ: codes of g_z, the two backward passes on codes of a and W
// that are there already) are instantiations of their own, for steps on two streams and for the autograd modules.
#include "device_common.h"
#include "kernels.h"

namespace int8t {

// Blocks per compute unit (by registers): what a grid is dealt for, so that no block waits for a second round.
constexpr int dwf_blocks(int U, bool XQ, bool GQ) { return !GQ ? 7 : U > 1 ? 4 : XQ ? 5 : 6; }

// U: chunks of four elements per thread, image and tensor (planes of up to 1024 * U elements); GROUP: cg channels of U = 1.
// With rows of whole dwords (always without GROUP) a thread's chunk is also its four results of a row.
template <int U, bool GROUP, bool XQ, bool GQ>
__global__ __launch_bounds__(256, dwf_blocks(U, XQ, GQ)) void dw_fused_kernel(const DwFused a) {
    constexpr int NT = 256;
    raise_wave_priority();
    extern __shared__ __attribute__((aligned(16))) int8_t lds[];
    __shared__ float s_max[2];
    __shared__ int red[GROUP ? 32 * 9 : (NT / kWave) * 9];
    const int tid = threadIdx.x;
    const int cg = GROUP ? a.cg : 1, groups = a.C / cg;
    const int share = blockIdx.x / groups, c0 = (blockIdx.x - share * groups) * cg;
    const int n0 = (int)(((long long)a.N * share) / a.shares), n1 = (int)(((long long)a.N * (share + 1)) / a.shares);
    const int W = a.W, H = a.H, HW = H * W, pitch = a.pitch, psize = (H + 2) * pitch;     // (multiples of 4)
    const int nch = (cg * HW) >> 2;                          // chunks of an image's run
    int8_t* const xs = lds;                                  // cg planes of (H + 2) rows, the element (h, w) at row h + 1, byte w + 4
    int8_t* const gs = lds + cg * psize;

    if (XQ && tid < 2 * kWave) {
        const bool second = tid >= kWave;
        const float m = absmax_partials_wave(second ? a.part_w : a.part_x, second ? a.np_w : a.np_x, tid & (kWave - 1));
        if ((tid & (kWave - 1)) == 0) s_max[second] = m;
    }
    // this thread's chunks: place in the run, and in LDS (`brk` bytes at off, the others at off2 behind the end of the row)
    const size_t img = (size_t)a.C * HW;
    const size_t run0 = (size_t)n0 * img + (size_t)c0 * HW;
    float4 fx[U], fg[U];
    uint32_t cx[U];
    int off[U], off2 = 0, brk = 4;
    bool ok[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int i = tid + u * NT;
        ok[u] = i < nch;
        const int e = ok[u] ? 4 * i : 0;
        const int pl = GROUP ? e / HW : 0, rem = e - pl * HW, row = rem / W, col = rem - row * W;
        off[u] = pl * psize + (row + 1) * pitch + col + 4;
        if (GROUP && col + 4 > W) {
            brk = W - col;
            off2 = (row + 1 < H ? pl * psize + (row + 2) * pitch : (pl + 1) * psize + pitch) + 4;
        }
    }
    auto fetch = [&](size_t run) {                           // (unconditional: the surplus repeats the run's first chunk)
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const size_t at = run + (ok[u] ? 4 * (tid + u * NT) : 0);
            if (XQ) fx[u] = *reinterpret_cast<const float4*>(a.x + at);
            else cx[u] = *reinterpret_cast<const uint32_t*>(a.xq + at);
            if (GQ) fg[u] = *reinterpret_cast<const float4*>(a.g + at);
        }
    };
    if (n0 < n1) fetch(run0);
    for (int i = tid; i < ((GQ ? 2 : 1) * cg * psize) >> 2; i += NT) reinterpret_cast<uint32_t*>(lds)[i] = 0u;

    // the task's channel and place: GROUP, `slot` lanes per channel; else every thread the block's channel
    const int QW = (W + 3) >> 2;
    int tpl = 0, trow = 0, tcol = 0;
    bool active = true;
    if (GROUP) {
        const int pr = tid / a.slot, tr = tid - pr * a.slot;
        active = pr < cg && tr < H * QW;
        tpl = active ? pr : 0;
        trow = active ? tr / QW : 0;
        tcol = active ? (tr - trow * QW) << 2 : 0;
    }
    __syncthreads();
    // scales, and this channel's weights: rows of three bytes, for backward-data turned around
    float inv_x = 0.0f, inv_g = 0.0f, scale_x, scale_w, scale_g = 0.0f;
    const int ct = c0 + tpl;
    int wt[9];
    if (XQ) {
        inv_x = inv_scale_of(s_max[0]);
        scale_x = scale_of(s_max[0]);
        const float inv_w = inv_scale_of(s_max[1]);
        scale_w = scale_of(s_max[1]);
#pragma unroll
        for (int i = 0; i < 9; ++i) wt[i] = quantize_one<false>(a.w[(size_t)ct * 9 + i], inv_w, 0u, 0u, 0u);
        if (share == 0 && (GROUP ? active && trow == 0 && tcol == 0 : tid == 0)) {
#pragma unroll
            for (int i = 0; i < 9; ++i) a.wq[(size_t)ct * 9 + i] = (int8_t)wt[i];
        }
        if (blockIdx.x == 0 && tid == 0) {
            *a.sx = scale_x;
            *a.sw = scale_w;
        }
    } else {
        scale_x = *a.sx;
        scale_w = *a.sw;
#pragma unroll
        for (int i = 0; i < 9; ++i) wt[i] = (int)a.wq[(size_t)ct * 9 + i];
    }
    if (GQ) {
        const float clip = *a.clip;
        inv_g = __fmul_rn(inv_scale_of(clip), kTwo24);       // the scaled value carries 24 fraction bits
        scale_g = scale_of(clip);
        if (blockIdx.x == 0 && tid == 0) *a.sg = scale_g;
    }
    uint32_t wf[3], wb[3];
#pragma unroll
    for (int r = 0; r < 3; ++r) {
        wf[r] = pack4(wt[3 * r], wt[3 * r + 1], wt[3 * r + 2], 0);
        wb[r] = pack4(wt[8 - 3 * r], wt[7 - 3 * r], wt[6 - 3 * r], 0);
    }
    float sf = __fmul_rn(scale_x, scale_w), sb = __fmul_rn(scale_g, scale_w);
    int acc[9];
#pragma unroll
    for (int i = 0; i < 9; ++i) acc[i] = 0;

    auto put = [&](int8_t* plane, int u, uint32_t d) {       // four codes into the staged plane
        if (!GROUP || brk == 4) {
            if (!GROUP || (W & 3) == 0) {
                *reinterpret_cast<uint32_t*>(plane + off[u]) = d;
                return;
            }
        }
#pragma unroll
        for (int b = 0; b < 4; ++b) plane[b < brk ? off[u] + b : off2 + b - brk] = (int8_t)(d >> (8 * b));
    };
    auto store4 = [&](float* out, int32_t* accp, const int (&sum)[4], float scale, int col) {
        if ((W & 3) == 0) {
            *reinterpret_cast<float4*>(out) = make_float4(__fmul_rn((float)sum[0], scale), __fmul_rn((float)sum[1], scale),
                                                          __fmul_rn((float)sum[2], scale), __fmul_rn((float)sum[3], scale));
        } else {
#pragma unroll
            for (int j = 0; j < 4; ++j)
                if (col + j < W) out[j] = __fmul_rn((float)sum[j], scale);
        }
        if (accp) {   // the accumulator output is only required to be 4-byte aligned
#pragma unroll
            for (int j = 0; j < 4; ++j)
                if (col + j < W) accp[j] = sum[j];
        }
    };
    // four results of a row, at LDS place `at` (the row above, the four bytes to the left) and element `o` of the tensors
    auto task = [&](int at, size_t o, int col) {
        const uint32_t* const xr = reinterpret_cast<const uint32_t*>(xs + at);
        const uint32_t* const gr = reinterpret_cast<const uint32_t*>(gs + at);
        const int g4 = GQ ? (int)gr[(pitch >> 2) + 1] : 0;
        int f[4] = {0, 0, 0, 0}, b[4] = {0, 0, 0, 0};
#pragma unroll
        for (int r = 0; r < 3; ++r) {
            uint32_t d[3], win[4];
#pragma unroll
            for (int k = 0; k < 3; ++k) d[k] = xr[r * (pitch >> 2) + k];
            win[0] = __builtin_amdgcn_alignbyte(d[1], d[0], 3);
            win[1] = d[1];
            win[2] = __builtin_amdgcn_alignbyte(d[2], d[1], 1);
            win[3] = __builtin_amdgcn_alignbyte(d[2], d[1], 2);
            if (XQ) {
#pragma unroll
                for (int j = 0; j < 4; ++j) f[j] = __builtin_amdgcn_sdot4((int)win[j], (int)wf[r], f[j], false);
            }
            if (GQ) {
#pragma unroll
                for (int s = 0; s < 3; ++s) acc[3 * r + s] = __builtin_amdgcn_sdot4((int)win[s], g4, acc[3 * r + s], false);
#pragma unroll
                for (int k = 0; k < 3; ++k) d[k] = gr[r * (pitch >> 2) + k];
                win[0] = __builtin_amdgcn_alignbyte(d[1], d[0], 3);
                win[1] = d[1];
                win[2] = __builtin_amdgcn_alignbyte(d[2], d[1], 1);
                win[3] = __builtin_amdgcn_alignbyte(d[2], d[1], 2);
#pragma unroll
                for (int j = 0; j < 4; ++j) b[j] = __builtin_amdgcn_sdot4((int)win[j], (int)wb[r], b[j], false);
            }
        }
        if (XQ) store4(a.y + o, a.y_acc ? a.y_acc + o : nullptr, f, sf, col);
        if (GQ) store4(a.dx + o, a.dx_acc ? a.dx_acc + o : nullptr, b, sb, col);
    };

    size_t run = run0;
    for (int n = n0; n < n1; ++n, run += img) {
        uint32_t qx[U], qg[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            qg[u] = 0u;
            if (XQ) {
                qx[u] = pack4(quantize_one<false>(fx[u].x, inv_x, 0u, 0u, 0u), quantize_one<false>(fx[u].y, inv_x, 0u, 0u, 0u),
                              quantize_one<false>(fx[u].z, inv_x, 0u, 0u, 0u), quantize_one<false>(fx[u].w, inv_x, 0u, 0u, 0u));
            } else {
                qx[u] = cx[u];
            }
        }
        if (GQ) {
            // round down for these elements only.  The codes of a pass through the first switch, so that they are formed
            // ahead of it; the multiply-adds between the switches are volatile, as the switches are; what is multiplied
            // after them is read from LDS behind the barrier.
            float t0 = inv_g, t1 = 0.0f;
#pragma unroll
            for (int u = 0; u < U; ++u) asm volatile("" : "+v"(qx[u]));
            fp32_round_down_mode(t0, t1);
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const uint32_t at = (uint32_t)(run + 4 * (size_t)(tid + u * NT));
                qg[u] = pack4(quantize_one<true>(fg[u].x, t0, a.key_x, a.key_a, at), quantize_one<true>(fg[u].y, t0, a.key_x, a.key_a, at + 1),
                              quantize_one<true>(fg[u].z, t0, a.key_x, a.key_a, at + 2), quantize_one<true>(fg[u].w, t0, a.key_x, a.key_a, at + 3));
            }
            fp32_round_nearest_mode(t1);
        }
        __syncthreads();                                     // the previous image has been read (and the borders are zero)
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (!ok[u]) continue;
            const size_t at = run + 4 * (tid + u * NT);
            if (XQ) *reinterpret_cast<uint32_t*>(a.xq + at) = qx[u];
            if (GQ) *reinterpret_cast<uint32_t*>(a.gq + at) = qg[u];
            put(xs, u, qx[u]);
            if (GQ) put(gs, u, qg[u]);
        }
        __syncthreads();
        if (n + 1 < n1) fetch(run + img);
        if (GROUP) {
            if (active) task(tpl * psize + trow * pitch + tcol, run + (size_t)tpl * HW + trow * W + tcol, tcol);
        } else {
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (ok[u]) task(off[u] - pitch - 4, run + 4 * (tid + u * NT), 0);
        }
    }
    if (!GQ) return;
    // backward-weight's sums of the share: over a channel's lanes (GROUP) or over the block
    int32_t* const part = a.partial + ((size_t)share * a.C + c0) * 9;
    const int lanes = GROUP ? a.slot : kWave;
    for (int o = lanes >> 1; o > 0; o >>= 1) {
#pragma unroll
        for (int i = 0; i < 9; ++i) acc[i] += __shfl_xor(acc[i], o, kWave);
    }
    const int pr = tid / lanes;
    if (tid - pr * lanes == 0 && pr < (GROUP ? cg : NT / kWave)) {
#pragma unroll
        for (int i = 0; i < 9; ++i) red[pr * 9 + i] = acc[i];
    }
    __syncthreads();
    if (GROUP) {
        for (int i = tid; i < cg * 9; i += NT) part[i] = red[i];
    } else if (tid < 9) {
        part[tid] = (red[tid] + red[9 + tid]) + (red[18 + tid] + red[27 + tid]);
    }
}

// Which layers: those of dw_trio_kernel with rows of at least four elements; every one of 17 measured gains.  Batch 64, us for a
// step that keeps the clip value (max|.|, codes and passes; in two launches and the reduction's / here): 144 channels at 56 x 56
// 154 / 127 (the launch itself 102 us for 520 MB, 5.1 TB/s), 192 at 28 x 28 56 / 41, 576 at 14 x 14 63 / 38, 960 at 7 x 7 40 / 23;
// 32 channels at 16 x 16, batch 2, 14.2 / 11.1; the halves at 144 channels, 56 x 56: 70 / 61 with the forward pass, 73 / 61 with
// the backward ones.  Fills the launch shape.
static bool dw_fused_plan(DwFused* a, const DwArgs& wgrad) {
    const int HW = a->H * a->W, QW = (a->W + 3) / 4;
    if (a->W < 4 || wgrad.threads != 256) return false;
    if (wgrad.cg > 1) {
        a->cg = wgrad.cg;
        a->slot = 4;
        while (a->slot < a->H * QW) a->slot *= 2;
        if ((a->cg * HW & 15) != 0 || a->cg * HW > 1024 || a->slot > kWave || a->cg * a->slot > 256 || a->cg > 32) return false;
    } else {
        a->cg = 1;
        if ((a->W & 3) != 0 || (HW & 15) != 0 || HW > 4096) return false;
    }
    a->pitch = ((a->W + 3) & ~3) + 8;                        // four bytes on either side: windows end inside the last dword
    return true;
}
bool dw_fused_applies(int H, int W, const DwArgs& wgrad) {
    DwFused a{};
    a.H = H; a.W = W;
    return dw_fused_plan(&a, wgrad);
}

// `shares` of the batch: one round of resident blocks, at most as many as backward-weight's scratch holds.
bool launch_dw_fused(const DwFused& in, const DwArgs& wgrad, hipStream_t st, hipError_t* err) {
    DwFused a = in;
    if (!dw_fused_plan(&a, wgrad)) return false;
    const bool xq = a.x != nullptr, gq = a.g != nullptr, group = wgrad.cg > 1;
    const int HW = a.H * a.W;
    const size_t lds = (size_t)(gq ? 2 : 1) * a.cg * (a.H + 2) * a.pitch;
    const int groups = a.C / a.cg;
    const int u = group || HW <= 1024 ? 1 : HW <= 2048 ? 2 : 4;
    int shares = 256 * dwf_blocks(u, xq, gq) / groups;
    if (shares > wgrad.chunks) shares = wgrad.chunks;
    if (shares > a.N) shares = a.N;
    if (shares < 1) shares = 1;
    const int per = (a.N + shares - 1) / shares;             // images per share, evenly
    a.shares = (a.N + per - 1) / per;
    const dim3 grid((unsigned)groups * (unsigned)a.shares);
    {
        KernelTimer kt(KID_DW_TRIO, st);
#define LAUNCH(Uv, Gv)                                                                                             \
    do {                                                                                                           \
        if (xq && gq) launch_timed(kt, (dw_fused_kernel<Uv, Gv, true, true>), grid, dim3(256), lds, st, a);        \
        else if (xq) launch_timed(kt, (dw_fused_kernel<Uv, Gv, true, false>), grid, dim3(256), lds, st, a);        \
        else launch_timed(kt, (dw_fused_kernel<Uv, Gv, false, true>), grid, dim3(256), lds, st, a);                \
    } while (0)
        if (group) LAUNCH(1, true);
        else if (u == 1) LAUNCH(1, false);
        else if (u == 2) LAUNCH(2, false);
        else LAUNCH(4, false);
#undef LAUNCH
    }
    *err = hipGetLastError();
    if (*err == hipSuccess && gq) {
        DwArgs w = wgrad;
        w.chunks = a.shares;
        *err = launch_dw_wgrad_reduce(w, st);
    }
    return true;
}

}  // namespace int8t
