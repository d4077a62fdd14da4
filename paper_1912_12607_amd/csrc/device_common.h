// Shared device helpers of the gfx950 INT8 training-convolution kernels.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "kernels.h"

namespace int8t {

constexpr int kWave = 64;            // CDNA wavefront width

// Raises the wave's issue priority.  For the kernels that may run on a second stream beside the clip search: they wait for
// memory most of the time and issue little, the search's waves issue all the time, and at equal priority the older waves
// -- the search's -- go first (64 -> 256 1x1 layer at 56 x 56, batch 256: step 1233 -> 1124 us; 7x7 stem, batch 64: 365 ->
// 336).  Alone on the chip all waves of such a kernel have the same priority and nothing changes.  In the shared launches of the
// convolution passes forward and backward-data raise theirs and backward-weight does not; with none or all three raised
// the three passes take between 4 % less and 4 % more, now one and now the other (3x3, 256 channels, 14 x 14, batch 64: 48.6 us as
// it is, 46.8 none, 49.7 all; 5x5, 48 -> 64, 35 x 35, batch 32: 41.2, 42.7, 42.6; depthwise, 576 channels, 14 x 14: 43.2, 44.1, 43.9).
__device__ __forceinline__ void raise_wave_priority() { __builtin_amdgcn_s_setprio(3); }

// ---------------------------------------------------------------------------
// Wavefront / block reductions (64-wide shuffles, then one LDS hop per wave).
// ---------------------------------------------------------------------------
// Over the four rows of 16 lanes with DPP operands -- exchanges of neighbours, of pairs, of quads -- and over the rows through scalar
// registers: a lane exchange through LDS costs a round trip per step, six of them in a row, which a pass over a small tensor
// has nothing to hide behind (with the batched launches' block ranges in one load, toy layer, whole step: 25.1 -> 24.5 us).  All 64
// lanes have to be active.
template <int CTRL>
__device__ __forceinline__ int dpp_word(int v) { return __builtin_amdgcn_update_dpp(v, v, CTRL, 0xf, 0xf, false); }
template <int CTRL>
__device__ __forceinline__ float dpp_of(float v) { return __int_as_float(dpp_word<CTRL>(__float_as_int(v))); }
template <int CTRL>
__device__ __forceinline__ double dpp_of(double v) { return __hiloint2double(dpp_word<CTRL>(__double2hiint(v)), dpp_word<CTRL>(__double2loint(v))); }
__device__ __forceinline__ float lane_of(float v, int lane) { return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), lane)); }
__device__ __forceinline__ double lane_of(double v, int lane) {
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), lane), __builtin_amdgcn_readlane(__double2loint(v), lane));
}
constexpr int kDppSwap1 = 0xB1, kDppSwap2 = 0x4E, kDppRor4 = 0x124, kDppRor8 = 0x128;      // quad_perm 1,0,3,2 and 2,3,0,1; row_ror
__device__ __forceinline__ float wave_max(float v) {
    v = fmaxf(v, dpp_of<kDppSwap1>(v));
    v = fmaxf(v, dpp_of<kDppSwap2>(v));
    v = fmaxf(v, dpp_of<kDppRor4>(v));
    v = fmaxf(v, dpp_of<kDppRor8>(v));
    return fmaxf(fmaxf(lane_of(v, 0), lane_of(v, 16)), fmaxf(lane_of(v, 32), lane_of(v, 48)));
}
__device__ __forceinline__ double wave_sum(double v) {
    v += dpp_of<kDppSwap1>(v);
    v += dpp_of<kDppSwap2>(v);
    v += dpp_of<kDppRor4>(v);
    v += dpp_of<kDppRor8>(v);
    return (lane_of(v, 0) + lane_of(v, 16)) + (lane_of(v, 32) + lane_of(v, 48));
}
__device__ __forceinline__ unsigned long long wave_sum(unsigned long long v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, kWave);
    return v;
}

// Block-wide max over 256 threads; result valid in every thread.
__device__ __forceinline__ float block_max_256(float v, float* lds4) {
    v = wave_max(v);
    const int w = threadIdx.x >> 6;
    __syncthreads();
    if ((threadIdx.x & 63) == 0) lds4[w] = v;
    __syncthreads();
    return fmaxf(fmaxf(lds4[0], lds4[1]), fmaxf(lds4[2], lds4[3]));
}

// max|x| from the per-block partials an absmax pass left behind, in two halves so that a kernel can deal
// with the partials FIRST and ask for its own data after: loads return in order, and a block that fetches
// its tile and then the partials can start on nothing until both are there (a quantize pass of 3840 blocks:
// 21 us that way, 15.5 us with the clip value handed in).  The first wave fetches and reduces the partials
// and leaves the result in LDS -- all blocks of the consuming pass read the same few cache lines, one wave
// each is enough -- while the other waves go straight on to their loads; everybody picks the value up after
// a barrier.
__device__ __forceinline__ float absmax_partials_wave(const float* __restrict__ part, int nparts, int lane) {
    // (straight-line loads: after a load inside a loop the compiler waits for ALL outstanding loads at
    // the next register it cannot account for, which serialised the tile loads that follow)
    float v[kAbsmaxPartials / kWave];
#pragma unroll
    for (int u = 0; u < kAbsmaxPartials / kWave; ++u) {
        const int i = lane + kWave * u;
        v[u] = part[i < nparts ? i : 0];      // (unconditional: a repeated partial does not change the max)
    }
    float m = 0.0f;
#pragma unroll
    for (int u = 0; u < kAbsmaxPartials / kWave; ++u) m = fmaxf(m, v[u]);
    return wave_max(m);
}
__device__ __forceinline__ void absmax_partials_begin(const float* __restrict__ part, int nparts, float* lds4) {
    if (threadIdx.x < kWave) {
        const float m = absmax_partials_wave(part, nparts, (int)threadIdx.x);
        if (threadIdx.x == 0) lds4[0] = m;
    }
}
// (all threads get the result; a barrier inside)
__device__ __forceinline__ float absmax_partials_end(const float* lds4) {
    __syncthreads();
    return lds4[0];
}
__device__ __forceinline__ float reduce_absmax_partials(const float* __restrict__ part, int nparts,
                                                        float* lds4) {
    absmax_partials_begin(part, nparts, lds4);
    return absmax_partials_end(lds4);
}

// ---------------------------------------------------------------------------
// Uniform draw for the stochastic rounding of Eq.3: 24 bits, a stateless function of
// (seed, logical element index).  The paper's in-kernel generator (Suppl. "Stochastic
// Rounding", Eq.8) is keyed by thread index; keying by element index instead makes the
// codes independent of launch geometry.  The 64-bit seed is first hashed into two 32-bit
// keys (on the host, once per call); the draw is one avalanche finaliser (multiply /
// xor-shift) over (index ^ key_x) + key_a.  Hashing the seed first matters: with the raw
// seed words as keys, two seeds that differ by d in their low word gave the same table at
// indices xor-ed with d, so layers and iterations seeded 1, 2, 3, ... shared their noise.
// ---------------------------------------------------------------------------
__host__ __device__ __forceinline__ uint32_t rng_mix32(uint32_t x) {
    x ^= x >> 16;
    x *= 0x85EBCA6Bu;
    x ^= x >> 13;
    x *= 0xC2B2AE35u;
    x ^= x >> 16;
    return x;
}
__device__ __forceinline__ uint32_t rng24(uint32_t key_x, uint32_t key_a, uint32_t index) {
    return rng_mix32((index ^ key_x) + key_a) >> 8;
}
// the two keys of a seed: key_x = mix(low word ^ mix(high word + golden ratio)), key_a = mix(key_x + golden ratio)
__host__ __device__ __forceinline__ uint32_t seed_key_x(uint64_t seed) {
    return rng_mix32((uint32_t)seed ^ rng_mix32((uint32_t)(seed >> 32) + 0x9E3779B9u));
}
__host__ __device__ __forceinline__ uint32_t seed_key_a(uint64_t seed) { return rng_mix32(seed_key_x(seed) + 0x9E3779B9u); }

// 127 / c as one correctly rounded fp32 division; 0 for an all-zero tensor.
__device__ __forceinline__ float inv_scale_of(float c) { return (c > 0.0f) ? __fdiv_rn(127.0f, c) : 0.0f; }
__device__ __forceinline__ float scale_of(float c) { return (c > 0.0f) ? __fdiv_rn(c, 127.0f) : 0.0f; }

constexpr float kTwo24 = 16777216.0f;

// Eq.1 on the scaled value, nearest rounding: t = clip(x * inv, 127), |t| <= 127 exactly.
__device__ __forceinline__ int round_nearest_code(float x, float inv) {
    const float t = fminf(fmaxf(__fmul_rn(x, inv), -127.0f), 127.0f);
    return (int)rintf(t);
}

// ---------------------------------------------------------------------------
// Stochastic rounding (Eq.3) on the magnitude:  m = min(127, floor((|x| * inv24 + u) / 2^24)),
// inv24 = inv * 2^24, u a 24-bit draw; the code is sign(x) * m.  floor((P + u)/2^24) of the EXACT
// product P is obtained from one fp32 fused multiply-add evaluated with rounding toward minus
// infinity: every multiple of 2^24 below 2^31 is representable, so rounding the sum down never
// moves it across one, and the saturating float->int32 conversion caps the result at 2^31 - 1,
// whose top byte is 127.  Two instructions per code, no clamp.
// The wave's fp32 rounding mode is switched once; values that must have been computed in the
// default mode are passed through the switch so that the compiler cannot move their
// computation behind it.  fp64 arithmetic has its own mode bits and is not affected.
// ---------------------------------------------------------------------------
__device__ __forceinline__ void fp32_round_down_mode(float& keep0, float& keep1) {
    asm volatile("s_setreg_imm32_b32 hwreg(HW_REG_MODE, 0, 2), 2\n\ts_nop 3" : "+v"(keep0), "+v"(keep1));
}
// back to round-to-nearest-even (the default) for the fp32 operations that follow
__device__ __forceinline__ void fp32_round_nearest_mode(float& keep0) {
    asm volatile("s_setreg_imm32_b32 hwreg(HW_REG_MODE, 0, 2), 0\n\ts_nop 3" : "+v"(keep0));
}
// floor(|x| * inv24 + uf) as int32, saturated at 2^31 - 1 (needs the round-down mode).
__device__ __forceinline__ int stoch_fixed(float x, float inv24, float uf) {
    float t;
    int X;
    asm volatile("v_fma_f32 %0, |%1|, %2, %3" : "=v"(t) : "v"(x), "v"(inv24), "v"(uf));
    asm("v_cvt_i32_f32 %0, %1" : "=v"(X) : "v"(t));
    return X;
}
// One code, with NaN -> 0.  STOCH needs fp32_round_down_mode() and inv = inv24.
template <bool STOCH>
__device__ __forceinline__ int quantize_one(float x, float inv, uint32_t seed_lo, uint32_t seed_hi_mul,
                                            uint32_t index) {
    if (STOCH) {
        const float uf = (float)rng24(seed_lo, seed_hi_mul, index);   // exact: 24 bits
        const int m = stoch_fixed(x, inv, uf) >> 24;                  // NaN converts to 0
        return (x < 0.0f) ? -m : m;
    } else {
        float t = __fmul_rn(x, inv);
        t = (t != t) ? 0.0f : t;
        t = fminf(fmaxf(t, -127.0f), 127.0f);
        return (int)rintf(t);
    }
}

// 4x4 byte transpose with v_perm_b32 (the gfx950 byte permute; the paper's Suppl. "INT8 Convolution"
// does the same "4x4 8-bit integer block transpose" with prmt): in d[i] = bytes (i,0..3), out
// o[j] = bytes (0..3, j).  Two rounds of four permutes: pairs of rows interleaved, then the halves
// joined.  Used by the activation quantizer (channel-major dwords -> pixel-major) and by
// backward-weight's loader (image-major -> channel-major).
__device__ __forceinline__ void transpose4x4_bytes(const uint32_t d[4], uint32_t o[4]) {
    // v_perm_b32 picks 4 bytes out of the 8 bytes {hi, lo}; selector byte 0-3 = lo, 4-7 = hi
    const uint32_t t0 = __builtin_amdgcn_perm(d[1], d[0], 0x05010400u);  // d0.b0 d1.b0 d0.b1 d1.b1
    const uint32_t t1 = __builtin_amdgcn_perm(d[1], d[0], 0x07030602u);  // d0.b2 d1.b2 d0.b3 d1.b3
    const uint32_t t2 = __builtin_amdgcn_perm(d[3], d[2], 0x05010400u);
    const uint32_t t3 = __builtin_amdgcn_perm(d[3], d[2], 0x07030602u);
    o[0] = __builtin_amdgcn_perm(t2, t0, 0x05040100u);  // t0.b0 t0.b1 t2.b0 t2.b1
    o[1] = __builtin_amdgcn_perm(t2, t0, 0x07060302u);  // t0.b2 t0.b3 t2.b2 t2.b3
    o[2] = __builtin_amdgcn_perm(t3, t1, 0x05040100u);
    o[3] = __builtin_amdgcn_perm(t3, t1, 0x07060302u);
}

__device__ __forceinline__ uint32_t pack4(int q0, int q1, int q2, int q3) {
    return (uint32_t)(q0 & 0xff) | ((uint32_t)(q1 & 0xff) << 8) | ((uint32_t)(q2 & 0xff) << 16) |
           ((uint32_t)q3 << 24);
}

// The first C bytes of four 32-bit words, packed back to back into 16 bytes (the rest zero).
__device__ __forceinline__ uint4 s2d_pack(const uint32_t px[4], int C) {
    const uint32_t keep = C >= 4 ? 0xffffffffu : ((1u << (8 * C)) - 1u);
    unsigned long long lo = 0, hi = 0;        // a 128-bit shift register
#pragma unroll
    for (int b = 0; b < 4; ++b) {
        const unsigned long long v = px[b] & keep;
        const int sh = 8 * C * b;             // 0 .. 96
        if (sh < 64) {
            lo |= v << sh;
            if (sh > 32) hi |= v >> (64 - sh);
        } else {
            hi |= v << (sh - 64);
        }
    }
    return make_uint4((uint32_t)lo, (uint32_t)(lo >> 32), (uint32_t)hi, (uint32_t)(hi >> 32));
}

}  // namespace int8t
