// Direction Sensitive Gradient Clipping (Sec.3.4 of the paper) as a candidate search.
//
// One sweep over the gradient evaluates the candidate clip values side by side.  Per candidate j
// it needs A_j = sum g*q_j and B_j = sum q_j^2 (and G = sum g^2 once); the deviation of Eq.6 is
// then d_j = 1 - A_j / sqrt(G * B_j): the scale s_j cancels between the numerator and |ghat|, so no
// dequantized tensor is ever formed.  The uniform draw of the stochastic rounding (Eq.3) is taken
// once per element and shared by all candidates -- the same draw the later quantize call uses,
// so the search scores exactly the codes that will be produced.
//
// The sweep is bound by the vector ALUs, not by HBM (4 bytes per element against several
// operations per element AND candidate), so the arithmetic is arranged to need few instructions:
//   * codes are sign(g) * m with m the rounded magnitude, so g*q = |g|*m and q^2 = m^2: the whole
//     search runs on magnitudes and never looks at a sign;
//   * m = floor(|g| * inv + u): one round-down fused multiply-add and one convert that floors,
//     saturates at 255 and drops its byte into the dword of four elements.  The clip at 127 costs a shift and a
//     mask per dword more (floor(2t) >> 1 = floor(t), 255 >> 1 = 127) and is left out for the eights of candidates
//     none of which clips any of the wave's 256 elements: with the heavy tails of a gradient that is three
//     of the four eights of the default grid nearly always (205 M elements: 22 us of 478);
//   * |g| is turned, once per element, into a 44-bit fixed-point integer relative to max|g|
//     (H * 2^22 + L, H, L <= 2^22), and both halves into three byte digits.  In the round-down mode adding
//     2^23 leaves floor(.) in the low mantissa bits, so the halves cost adds instead of floor / round / convert;
//   * the sums A_j = sum |g| m_j (six digit sums) and B_j = sum m_j^2 are int8 x int8 products
//     with int32 accumulation, i.e. matrix products [digits x elements] * [elements x candidates]
//     and [candidates x elements] * [elements x candidates] (diagonal): they go to the matrix
//     cores.  A lane computes the codes of ITS four elements for all candidates, but an MFMA
//     operand wants one candidate's codes of 16 elements: the code dwords pass through a wave-private
//     LDS tile (no barriers needed: a wave reads only what it wrote), sixteen candidates at a time.
//
// What an instruction costs here (one SIMD, many waves, cycles per wave instruction): 2 - 2.5 for fp32 add / multiply /
// fused multiply-add, integer add, right shift and the bitwise operations on vector registers, 4 - 4.5 for
// everything else (conversions, byte permutes, min / max, 24-bit and full integer multiplies, left shifts, and any of the first
// group with a scalar operand) -- two pipes, of which one does everything.  A wave's 256 elements take 380 vector instructions
// where one of the four eights of candidates clips: 64 per eight (a multiply-add with its scalar scale and a convert per
// element and candidate), 16 cheap ones more where it clips, 108 for the draw, the digits and the loop; with 16 MFMAs and
// their operand reads (a fifth of the time) they are what the loop consists of.
//
// One block of 16 waves per compute unit: a compute unit issues from its oldest waves first, so of three equal
// blocks that share one the first was done in half the time of the last, and the last ran alone (205 M elements: blocks
// between 237 and 448 us).  The waves of a block therefore take their wave-iterations from a counter in LDS as
// they come.  616 -> 466 us at 205 M elements, 161 -> 118 at 51 M, 47.6 -> 38.6 at 12.8 M, 21.4 -> 18.3 at 3.2 M.
// The block leaves half the wave slots, 66 KB of LDS and 3/8 of the registers (192 of a lane's 512: a block of four waves that takes
// more waits until this one is done) to kernels of another stream; those raise their
// waves' priority (they are bound by HBM and issue little), which is what lets them run beside this kernel.
//
// The integer sums are exact and order independent; the only error against an fp64 evaluation is
// the fixed-point rounding of |g|, |delta| <= max|g| * 2^-44 per element, i.e. at most
// 2^-44 * sqrt(n) in d_j (Cauchy-Schwarz), far below the resolution the search needs.
//
// Blocks add their 64-bit integer totals (sum H*m, sum L*m, sum m^2 per candidate) into one of
// DSGC_GROUPS accumulator sets with device-scope atomics -- integer addition, so the result does
// not depend on the order -- and take a ticket; the block that draws the last ticket sums the
// sets, evaluates Eq.6 for every candidate and picks the clip value.  The accumulators and the
// ticket are cleared by the absmax pass that always precedes the sweep.
#include "device_common.h"
#include "kernels.h"

namespace int8t {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v16i __attribute__((ext_vector_type(16)));

constexpr int DSGC_JC = 32;        // candidates per block: the 32 columns of one MFMA tile
constexpr int DSGC_JPAD = 64;      // row pitch of the partial arrays (= INT8T_MAX_CANDIDATES)
constexpr int DSGC_MAX_BLOCKS = 256;         // one per compute unit
constexpr int DSGC_MAX_THREADS = 1024;
constexpr int DSGC_GROUPS = 32;     // accumulator sets the blocks spread their atomics over
constexpr int DSGC_JH = 16;                 // candidates per pass through the LDS tile: the columns of one MFMA
constexpr int DSGC_ROWS = DSGC_JH + 6;      // 16 code rows, then the 6 digit rows
// A wave's LDS tile holds 256 elements x DSGC_ROWS byte rows, stored by 16-element granule:
// [granule 0..15][row][16 bytes], with the granule pitch padded to 23 rows.  An MFMA operand read
// (16 lanes = 16 consecutive rows of one granule) is then 256 contiguous bytes, and the 16 granules
// a store instruction touches (4 lanes each) start 92 banks apart, i.e. in 16 different groups of
// 4 banks -- both free of bank conflicts.
constexpr int DSGC_GPITCH = (DSGC_ROWS + 1) * 16;   // 368 bytes
constexpr int DSGC_TILE = 16 * DSGC_GPITCH;         // 5888 bytes per wave
// int32 accumulators: |digit * code| <= 128 * 127 per element and lane sum; flushed well before 2^31
// (64 iterations: 64 x 256 elements x 16256 < 2^28.1)
constexpr int DSGC_FLUSH_ITERS = 64;

// bytes [a.b0, b.b0, c.b0, d.b0]
__device__ __forceinline__ uint32_t low_bytes(int a, int b, int c, int d) {
    const uint32_t lo = __builtin_amdgcn_perm((uint32_t)b, (uint32_t)a, 0x0c0c0400u);
    const uint32_t hi = __builtin_amdgcn_perm((uint32_t)d, (uint32_t)c, 0x04000c0cu);
    return lo | hi;
}

// Byte digits of four integers 0 <= v <= 2^22, handed in as y = v + 0x8080 in the low 24 bits (the top byte is
// ignored): v = d0 + 256 d1 + 65536 d2 with -128 <= d0, d1 < 128 (bytes 0 and 1 of y, each minus 128) and
// 0 <= d2 <= 64.  plane[b] packs digit b of the four values as signed bytes.
__device__ __forceinline__ void digit_planes(const uint32_t y[4], uint32_t plane[3]) {
    const uint32_t t0 = __builtin_amdgcn_perm(y[1], y[0], 0x05010400u);  // y0.b0 y1.b0 y0.b1 y1.b1
    const uint32_t t1 = __builtin_amdgcn_perm(y[1], y[0], 0x0c0c0602u);  // y0.b2 y1.b2 0 0
    const uint32_t t2 = __builtin_amdgcn_perm(y[3], y[2], 0x05010400u);
    const uint32_t t3 = __builtin_amdgcn_perm(y[3], y[2], 0x06020c0cu);  // 0 0 y2.b2 y3.b2
    plane[0] = __builtin_amdgcn_perm(t2, t0, 0x05040100u) ^ 0x80808080u;
    plane[1] = __builtin_amdgcn_perm(t2, t0, 0x07060302u) ^ 0x80808080u;
    plane[2] = t1 | t3;
}

// 2 v of a scale, on the scalar unit: the exponent plus one, an infinity (the reciprocal of a very small clip value) stays
// one, and 0 stays 0 -- the scale of an infinite clip value, which has to turn an infinite element into no number and so into
// code 0, and of candidates that do not exist.
// Volatile, so that the doubled scales of all candidates are not kept, and spilled, across the loop.
__device__ __forceinline__ float twice(float v) {
    int b;
    asm volatile("s_min_u32 %0, %1, 0x800000\n\ts_add_u32 %0, %0, %1\n\ts_min_u32 %0, %0, 0x7f800000" : "=&s"(b) : "s"(v) : "scc");
    return __int_as_float(b);
}

// Two candidates against four elements: the magnitudes floor(|x_e| * inv + u_e) of both as bytes (saturated at 255).
// The two chains are interleaved: a convert-and-pack depends on the one before it.
__device__ __forceinline__ void stoch_codes4x2(const float x[4], float ia, float ib, const float uf[4], uint32_t& a, uint32_t& b) {
    float t0, t1, t2, t3, s0, s1, s2, s3;
    asm volatile(
        "v_fma_f32 %2, |%10|, %14, %16\n\t"
        "v_fma_f32 %6, |%10|, %15, %16\n\t"
        "v_fma_f32 %3, |%11|, %14, %17\n\t"
        "v_cvt_pk_u8_f32 %0, %2, 0, 0\n\t"
        "v_fma_f32 %7, |%11|, %15, %17\n\t"
        "v_cvt_pk_u8_f32 %1, %6, 0, 0\n\t"
        "v_fma_f32 %4, |%12|, %14, %18\n\t"
        "v_cvt_pk_u8_f32 %0, %3, 1, %0\n\t"
        "v_fma_f32 %8, |%12|, %15, %18\n\t"
        "v_cvt_pk_u8_f32 %1, %7, 1, %1\n\t"
        "v_fma_f32 %5, |%13|, %14, %19\n\t"
        "v_cvt_pk_u8_f32 %0, %4, 2, %0\n\t"
        "v_fma_f32 %9, |%13|, %15, %19\n\t"
        "v_cvt_pk_u8_f32 %1, %8, 2, %1\n\t"
        "v_cvt_pk_u8_f32 %0, %5, 3, %0\n\t"
        "v_cvt_pk_u8_f32 %1, %9, 3, %1"
        : "=&v"(a), "=&v"(b), "=&v"(t0), "=&v"(t1), "=&v"(t2), "=&v"(t3), "=&v"(s0), "=&v"(s1), "=&v"(s2), "=&v"(s3)
        : "v"(x[0]), "v"(x[1]), "v"(x[2]), "v"(x[3]), "s"(ia), "s"(ib), "v"(uf[0]), "v"(uf[1]), "v"(uf[2]), "v"(uf[3]));
}

template <bool STOCH>
__global__ __launch_bounds__(DSGC_MAX_THREADS) void dsgc_sweep_kernel(
    const float* __restrict__ g, size_t n, const float* __restrict__ ratios, int n_cand,
    const float* __restrict__ absmax_part, int nparts, uint32_t seed_lo, uint32_t seed_hi_mul,
    unsigned long long* __restrict__ acc, unsigned int* __restrict__ ticket, const double* __restrict__ partG,
    float* __restrict__ clip_out, double* __restrict__ dev_out, double* __restrict__ dev_all_out) {
    constexpr int JC = DSGC_JC, JH = DSGC_JH;
    __shared__ float lds4[4];
    __shared__ unsigned int s_last;
    __shared__ unsigned long long s_tot[JC * 3];
    __shared__ int s_next;
    extern __shared__ __attribute__((aligned(16))) unsigned char s_tile[];     // one tile per wave
    const int nwaves = (int)blockDim.x >> 6;

    const int j0 = blockIdx.y * JC;
    const int jn = (n_cand - j0 < JC) ? (n_cand - j0) : JC;
    // Everything the prologue fetches is requested before the first wait: the absmax partials, the ratios and
    // the wave's first 16 bytes per lane of g (one memory round trip instead of three in a row, about 1 us
    // of a sweep that takes 10 us on a small tensor).
    absmax_partials_begin(absmax_part, nparts, lds4);
    const size_t n4 = n >> 2;
    const float4* __restrict__ g4 = reinterpret_cast<const float4*>(g);
    // the wave-iterations (64 float4 each) of a block: blockIdx.x + k * gridDim.x, k = 0, 1, ..; its waves take them as they come
    const int w = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), lane = threadIdx.x & 63;
    const size_t i_first = ((size_t)w * gridDim.x + blockIdx.x) * 64 + lane;
    const float4 f_first = (i_first < n4) ? g4[i_first] : make_float4(0.f, 0.f, 0.f, 0.f);
    const float ratio_j = ratios[j0 + (lane < jn ? lane : 0)];
    if (threadIdx.x < 3 * JC) s_tot[threadIdx.x] = 0ull;
    if (threadIdx.x == 0) s_next = nwaves;
    const float M = absmax_partials_end(lds4);
    // fixed point: max|g| < 2^e, |g| * 2^(22-e) <= 2^22
    int e2 = 0;
    float mant = frexpf(M, &e2);
    // lane j < 32 of every wave: candidate j's clip value, scale and -- a little below the clip value -- the largest |g|
    // it surely does not clip; of the latter the smallest of every eight candidates.  A candidate that does not exist has
    // scale 0; one whose scale overflows sends its eight to the clipping form.
    const float clip_j = lane < jn ? __fmul_rn(M, ratio_j) : 0.0f;
    const float inv_j = inv_scale_of(clip_j);
    float thr_j = inv_j == 0.0f ? __builtin_huge_valf() : inv_j < __builtin_huge_valf() ? 0.99f * clip_j : 0.0f;
#pragma unroll
    for (int o = 1; o < 8; o <<= 1) thr_j = fminf(thr_j, __shfl_xor(thr_j, o, kWave));
    float inv[JC], thr[JC / 8];
#pragma unroll
    for (int j = 0; j < JC; ++j) inv[j] = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(inv_j), j));
#pragma unroll
    for (int q = 0; q < JC / 8; ++q) thr[q] = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(thr_j), 8 * q));
    float e2f = (float)e2;
    // From here on every fp32 operation of the stochastic sweep is either exact or meant to round down; the candidates'
    // scales above are in scalar registers by now, computed in the default mode.
#pragma unroll
    for (int j = 0; j < JC; ++j) asm volatile("" : "+s"(inv[j]));
    if (STOCH) fp32_round_down_mode(mant, e2f);
    const int shift = 22 - (int)e2f;

    const int l16 = lane & 15, kg = lane >> 4;
    unsigned char* __restrict__ const tile = s_tile + (size_t)w * DSGC_TILE;
    // this lane's four elements live in granule lane / 4, bytes 4 * (lane % 4) ..; + 16 * row
    uint32_t* __restrict__ const wr = reinterpret_cast<uint32_t*>(tile + (lane >> 2) * DSGC_GPITCH + 4 * (lane & 3));
    // MFMA operands of this lane (16 x 16 x 64 tiles: a lane supplies 16 reduction bytes of one row):
    // codes of candidate l16 of the half in the tile / digit row min(l16, 5), granule 4 * step + kg
    const unsigned char* __restrict__ const rd_code = tile + kg * DSGC_GPITCH + l16 * 16;
    const unsigned char* __restrict__ const rd_dig = tile + kg * DSGC_GPITCH + (JH + (l16 < 5 ? l16 : 5)) * 16;

    // per candidate half h: [digit row][candidate] (rows 0..5 used) and [candidate][candidate] (diagonal used)
    v4i accA[2], accB[2];
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int v = 0; v < 4; ++v) accA[h][v] = accB[h][v] = 0;

    // int32 tiles -> the block's 64-bit per-candidate totals, accumulators cleared
    auto flush = [&]() {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            // accA[h]: lane (column l16, kg), register v holds digit row 4*kg + v: rows 0..3 (the H digits
            // and L digit 0) sit in the lanes kg = 0, rows 4..5 (L digits 1, 2) in registers 0..1 of kg = 1
            long long ph = 0, pl = 0;
            if (kg == 0) {
                ph = (long long)accA[h][0] + 256LL * accA[h][1] + 65536LL * accA[h][2];
                pl = (long long)accA[h][3];
            } else if (kg == 1) {
                pl = 256LL * accA[h][0] + 65536LL * accA[h][1];
            }
            unsigned long long* const t = s_tot + (16 * h + l16) * 3;
            if (kg == 0) __hip_atomic_fetch_add(t + 0, (unsigned long long)ph, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            if (kg < 2) __hip_atomic_fetch_add(t + 1, (unsigned long long)pl, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            // accB[h]: the diagonal element of column l16 is row l16 = 4*kg + v
            int diag = 0;
#pragma unroll
            for (int v = 0; v < 4; ++v) diag = (v == (l16 & 3)) ? accB[h][v] : diag;
            if ((l16 >> 2) == kg) __hip_atomic_fetch_add(t + 2, (unsigned long long)(long long)diag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
#pragma unroll
            for (int v = 0; v < 4; ++v) accA[h][v] = accB[h][v] = 0;
        }
    };
    // constants of the loop in vector registers: with a literal or scalar operand the adds take twice as long
    float cmag = 8388608.0f + 32896.0f, c22 = 4194304.0f, cm24 = 0x1p-24f;
    uint32_t mask7 = 0x7f7f7f7fu;
    asm volatile("" : "+v"(cmag), "+v"(c22), "+v"(cm24), "+v"(mask7));

    // one wave iteration: 256 consecutive elements, four per lane
    auto group = [&](const float x[4], uint32_t index0) {
        float uf[4] = {0.f, 0.f, 0.f, 0.f};
        uint32_t H[4], L[4];
        const uint32_t ix = index0 ^ seed_lo;            // index0 is a multiple of 4: (index0 + e) ^ key = ix ^ e
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const float xs = ldexpf(fabsf(x[e]), shift);     // exact, 0 .. 2^22
            if (STOCH) {
                uf[e] = (float)(rng_mix32((ix ^ (uint32_t)e) + seed_hi_mul) >> 8) * cm24;
                // round-down mode: 2^23 + 0x8080 + floor(xs), i.e. floor(xs) + 0x8080 in the low mantissa bits; then the
                // remainder times 2^22, rounded to nearest (floor of it plus a half; every step but the last exact)
                const float hs = xs + cmag;
                const float ls = __builtin_fmaf(xs - (hs - cmag), c22, 0.5f) + cmag;
                H[e] = __float_as_uint(hs);
                L[e] = __float_as_uint(ls);
            } else {
                const float h = floorf(xs);
                H[e] = (uint32_t)h + 0x8080u;          // (digit_planes' offset)
                L[e] = (uint32_t)rintf((xs - h) * 4194304.0f) + 0x8080u;
            }
        }
        uint32_t pH[3], pL[3];
        digit_planes(H, pH);
        digit_planes(L, pL);
#pragma unroll
        for (int b = 0; b < 3; ++b) {
            wr[(JH + b) * 4] = pH[b];
            wr[(JH + 3 + b) * 4] = pL[b];
        }
        const float xm = STOCH ? fmaxf(fmaxf(fmaxf(fabsf(x[0]), fabsf(x[1])), fabsf(x[2])), fabsf(x[3])) : 0.0f;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
#pragma unroll
            for (int q = 2 * h; q < 2 * h + 2; ++q) {
                uint32_t* const wq = wr + (8 * q - JH * h) * 4;
                if (!STOCH) {
#pragma unroll
                    for (int j = 0; j < 8; ++j)
                        wq[4 * j] = low_bytes(round_nearest_code(fabsf(x[0]), inv[8 * q + j]), round_nearest_code(fabsf(x[1]), inv[8 * q + j]),
                                              round_nearest_code(fabsf(x[2]), inv[8 * q + j]), round_nearest_code(fabsf(x[3]), inv[8 * q + j]));
                } else if (!__any(xm >= thr[q])) {
#pragma unroll
                    for (int j = 0; j < 8; j += 2) {
                        uint32_t a, b;
                        stoch_codes4x2(x, inv[8 * q + j], inv[8 * q + j + 1], uf, a, b);
                        wq[4 * j] = a;
                        wq[4 * j + 4] = b;
                    }
                } else {
                    float u2[4];
#pragma unroll
                    for (int e = 0; e < 4; ++e) u2[e] = uf[e] + uf[e];
#pragma unroll
                    for (int j = 0; j < 8; j += 2) {
                        uint32_t a, b;
                        stoch_codes4x2(x, twice(inv[8 * q + j]), twice(inv[8 * q + j + 1]), u2, a, b);
                        wq[4 * j] = (a >> 1) & mask7;
                        wq[4 * j + 4] = (b >> 1) & mask7;
                    }
                }
            }
            __builtin_amdgcn_wave_barrier();   // keep the tile's stores ahead of its loads
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                const v4i fd = *reinterpret_cast<const v4i*>(rd_dig + 4 * DSGC_GPITCH * s);
                const v4i fc = *reinterpret_cast<const v4i*>(rd_code + 4 * DSGC_GPITCH * s);
                accA[h] = __builtin_amdgcn_mfma_i32_16x16x64_i8(fd, fc, accA[h], 0, 0, 0);
                accB[h] = __builtin_amdgcn_mfma_i32_16x16x64_i8(fc, fc, accB[h], 0, 0, 0);
            }
            __builtin_amdgcn_wave_barrier();   // and the next stores behind these loads
        }
    };

    {
        // Wave-uniform trip count (the MFMAs need the whole wave): lanes beyond the end carry zeros,
        // which add nothing to A or B.  The next iteration's 16 bytes are requested before this
        // iteration's arithmetic starts.
        const int units = (int)((n4 + 63) >> 6);
        int u = w * (int)gridDim.x + (int)blockIdx.x;      // this wave's current wave-iteration
        float4 f = f_first;
        // (waits for the first data here: inside the loop the wait would be for the load just issued)
        asm volatile("" : "+v"(f.x), "+v"(f.y), "+v"(f.z), "+v"(f.w));
        int knext = 0;                                     // (lane 0) the number of the one after it, asked for an iteration ahead
        auto draw = [&]() {
            if (lane == 0) knext = __hip_atomic_fetch_add(&s_next, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        };
        draw();
        while (u < units) {
            for (int it = 0; it < DSGC_FLUSH_ITERS && u < units; ++it) {
                const int un = __builtin_amdgcn_readfirstlane(knext) * (int)gridDim.x + (int)blockIdx.x;
                const size_t inext = (size_t)un * 64 + lane;
                const float4 fn = (inext < n4) ? g4[inext] : make_float4(0.f, 0.f, 0.f, 0.f);
                draw();
                const float vv[4] = {f.x, f.y, f.z, f.w};
                group(vv, (uint32_t)u * 256u + 4u * (uint32_t)lane);
                f = fn;
                u = un;
            }
            if (u < units) flush();
        }
    }
    if (blockIdx.x == 0 && w == 0 && (n & 3)) {
        // ragged tail (wave-uniform branch): lane 0 carries the last 1..3 elements, zeros elsewhere
        float vv[4] = {0.0f, 0.0f, 0.0f, 0.0f};
        if (lane == 0)
            for (int e = 0; e < (int)(n & 3); ++e) vv[e] = g[(n4 << 2) + e];
        group(vv, (uint32_t)(n4 << 2) + 4u * (uint32_t)lane);
    }
    flush();

    // block totals -> one of the accumulator sets
    __syncthreads();
    if (threadIdx.x < 3 * JC) {
        const int j = threadIdx.x / 3, q = threadIdx.x - 3 * j;
        if (j < jn) {
            const int grp = (int)(blockIdx.x % DSGC_GROUPS);
            __hip_atomic_fetch_add(&acc[((size_t)grp * DSGC_JPAD + j0 + j) * 3 + q], s_tot[threadIdx.x],
                                   __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    }
    // All data moves through device-scope atomics (performed at the memory side) and is read back
    // with device-scope atomic loads, so no cache write-back is needed: it is enough that this
    // block's additions have been acknowledged before its ticket is drawn: every thread waits for
    // its outstanding memory operations, then the barrier.  (The memory model's own way to say this,
    // a device-scope release fence per thread in front of the barrier and an acquire fence in the
    // last block, was measured: each release fence writes the whole L2 of its XCD back; with 768 blocks of
    // 256 threads they stretched the sweep from 58 to 75 us with the GPU to itself and to 126 us beside another
    // stream's kernels, whose dirty lines they flush.  What the wait below relies on is only that an
    // atomic's vmcnt decrement means it has been performed, which the return path of a device-scope
    // atomic guarantees.)
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (threadIdx.x == 0)
        s_last = __hip_atomic_fetch_add(ticket, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == gridDim.x * gridDim.y - 1
                     ? 1u : 0u;
    __syncthreads();
    if (!s_last) return;
    float Mn = M;
    if (STOCH) fp32_round_nearest_mode(Mn);   // the clip value below is a default-mode product

    // ---- last block: sum the sets, Eq.6 per candidate, smallest deviation (ties: smallest j, i.e.
    // the largest clip value for decreasing ratios).  Every addition is in a fixed order. ----------
    long long (*const f_part)[DSGC_JPAD][3] = reinterpret_cast<long long (*)[DSGC_JPAD][3]>(s_tile);
    double* const f_g = reinterpret_cast<double*>(s_tile + sizeof(long long) * 4 * DSGC_JPAD * 3);
    static_assert(sizeof(long long) * 4 * DSGC_JPAD * 3 + sizeof(double) * 4 <= 4 * DSGC_TILE, "fits the tiles of the smallest block");
    {
        const int j = threadIdx.x & 63, part = threadIdx.x >> 6;
        if (part < 4) {
        // G: the absmax pass's per-block sums of squares, at most one per thread (asked for ahead of the sets)
        static_assert(kAbsmaxPartials <= 256, "one partial sum of squares per thread");
        double gs = (int)threadIdx.x < nparts ? partG[threadIdx.x] : 0.0;
        long long t[3] = {0, 0, 0};
        if (j < n_cand) {
            long long v[DSGC_GROUPS / 4][3];
#pragma unroll
            for (int k = 0; k < DSGC_GROUPS / 4; ++k)
#pragma unroll
                for (int q = 0; q < 3; ++q)
                    v[k][q] = (long long)__hip_atomic_load(&acc[((size_t)(4 * k + part) * DSGC_JPAD + j) * 3 + q],
                                                           __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
            for (int k = 0; k < DSGC_GROUPS / 4; ++k)
#pragma unroll
                for (int q = 0; q < 3; ++q) t[q] += v[k][q];
        }
#pragma unroll
        for (int q = 0; q < 3; ++q) f_part[part][j][q] = t[q];
        gs = wave_sum(gs);
        if (j == 0) f_g[part] = gs;
        }
    }
    __syncthreads();
    if (threadIdx.x < 64) {
        const int j = threadIdx.x;
        double d = 0.0;
        if (j < n_cand) {
            long long t[3];
#pragma unroll
            for (int q = 0; q < 3; ++q) t[q] = (f_part[0][j][q] + f_part[1][j][q]) + (f_part[2][j][q] + f_part[3][j][q]);
            // A = (sumH * 2^22 + sumL) * 2^(e-44); the integer totals are exact, the conversions round once
            const double At = ldexp((double)t[0] * 4194304.0 + (double)t[1], e2 - 44);
            const double Bt = (double)t[2];
            const double Gt = (f_g[0] + f_g[1]) + (f_g[2] + f_g[3]);
            if (Gt == 0.0) d = 0.0;
            else if (Bt == 0.0) d = 1.0;
            else d = 1.0 - At / (sqrt(Gt) * sqrt(Bt));
            if (dev_all_out) dev_all_out[j] = d;
        }
        // The winner, over the lanes: a candidate replaces the best so far only with a strictly smaller deviation,
        // walking j upwards -- i.e. the smallest (d, j) in lexicographic order, where a deviation that is not
        // a number never wins, except candidate 0's, which then is never replaced.
        const double inf = __builtin_huge_val();
        double bd = (j < n_cand && d == d) ? d : (j == 0 ? -inf : inf);
        int bj = j;
        auto better = [&](double od, int oj) {
            if (od < bd || (od == bd && oj < bj)) { bd = od; bj = oj; }
        };
        better(dpp_of<kDppSwap1>(bd), dpp_word<kDppSwap1>(bj));
        better(dpp_of<kDppSwap2>(bd), dpp_word<kDppSwap2>(bj));
        better(dpp_of<kDppRor4>(bd), dpp_word<kDppRor4>(bj));
        better(dpp_of<kDppRor8>(bd), dpp_word<kDppRor8>(bj));
        const double rd[4] = {lane_of(bd, 0), lane_of(bd, 16), lane_of(bd, 32), lane_of(bd, 48)};
        const int rj[4] = {__builtin_amdgcn_readlane(bj, 0), __builtin_amdgcn_readlane(bj, 16), __builtin_amdgcn_readlane(bj, 32),
                           __builtin_amdgcn_readlane(bj, 48)};
#pragma unroll
        for (int r = 0; r < 4; ++r) better(rd[r], rj[r]);
        const int best = (Mn == 0.0f) ? 0 : bj;
        const double dbest = lane_of(d, best);
        if (j == 0) {
            *clip_out = __fmul_rn(Mn, ratios[best]);
            *dev_out = dbest;
        }
    }
}

// Threads per block and blocks.  Up to 1024 wave-iterations (262 K elements) a wave has one of them and the sweep is a chain of
// memory round trips: blocks of four waves spread them over more compute units (65 K elements: 9.8 us, 12.4 with 16
// waves per block).  Above, 16 waves per block, one block per compute unit: fewer blocks also leave fewer atomic
// additions and tickets at the end (0.8 M elements: 17.0 us with four waves per block, 13.7 with 16).
static int dsgc_threads(size_t units) { return units <= 1024 ? 256 : DSGC_MAX_THREADS; }

hipError_t launch_dsgc(const float* g, size_t n, const float* ratios, int n_cand, int stochastic,
                       uint64_t seed, const DsgcWs& ws, int nparts_absmax, float* clip_out,
                       double* dev_out, double* dev_all_out, hipStream_t st) {
    const int nchunks = (n_cand + DSGC_JC - 1) / DSGC_JC;
    const size_t units = (n / 4 + 63) / 64;
    const int threads = dsgc_threads(units), waves = threads / 64;
    // every candidate chunk walks the same x-grid
    const size_t cap = (DSGC_MAX_BLOCKS + nchunks - 1) / nchunks;
    size_t blocks = (units + waves - 1) / waves;
    blocks = blocks < 1 ? 1 : blocks > cap ? cap : blocks;
    const uint32_t slo = seed_key_x(seed), shi = seed_key_a(seed);
    const size_t lds = (size_t)waves * DSGC_TILE;
    dim3 grid((unsigned)blocks, nchunks);
    static std::atomic<unsigned long long> done_st, done_nr;
    const hipError_t e = raise_dynamic_lds(stochastic ? (const void*)dsgc_sweep_kernel<true> : (const void*)dsgc_sweep_kernel<false>,
                                           DSGC_MAX_THREADS / 64 * DSGC_TILE, stochastic ? done_st : done_nr);
    if (e != hipSuccess) return e;
    KernelTimer kt(KID_DSGC_SWEEP, st);
    if (stochastic)
        launch_timed(kt, (dsgc_sweep_kernel<true>), grid, dim3(threads), lds, st, g, n, ratios, n_cand,
                           ws.absmax_part, nparts_absmax, slo, shi, ws.acc, ws.ticket, ws.partG, clip_out,
                           dev_out, dev_all_out);
    else
        launch_timed(kt, (dsgc_sweep_kernel<false>), grid, dim3(threads), lds, st, g, n, ratios, n_cand,
                           ws.absmax_part, nparts_absmax, slo, shi, ws.acc, ws.ticket, ws.partG, clip_out,
                           dev_out, dev_all_out);
    return hipGetLastError();
}

static_assert(kDsgcAccWords == (size_t)DSGC_GROUPS * DSGC_JPAD * 3, "accumulator layout known to the C-ABI layer");
size_t dsgc_acc_words() { return kDsgcAccWords; }

}  // namespace int8t
