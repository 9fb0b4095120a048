// Device-side building blocks of the one-token kernel for 1- and 2-bit weights on the matrix cores: codes as 4-bit floating
// point numbers, activations as four 8-bit ones.
//
// Why.  On the dot product unit a block of 32 weights costs 16 dot products beside its transposition, whatever the width of
// the codes, and a 2-bit tile 123 vector instructions (1 bit: 110).  v_mfma_f32_16x16x128_f8f6f4 multiplies 16 rows x 128 columns of
// codes with 16 rows of activations in one instruction that runs beside the vector pipe; what is left are exchanges between
// lanes, the transposition and 5 or 6 multiply-adds per 16 rows: 84 instructions per tile for 2 bits, 69 for 1 bit, in the loop.
// 32 launches of a 7B layer set, uint2 g64: 430 -> 416 us (63.2 MB in 13.0 us = 4.9 TB/s), of a 3.8B one, 1 bit: 265 -> 249 (without
// the scaling of the blocks: 413 and 248).  What bounds them now is the memory system and, for 2 bits, digits and products of waves
// that start together (a launch with neither: 11.7 of 13.0 us), for 1 bit the start and end of a launch (6.5 of 7.7).
//
// Codes.  The numbers 0, 1, 2, 3 in the low bits of an E2M1 number (4 bits) are 0, 0.5, 1, 1.5: codes of 1 and 2 bits in
// nibbles are operands as they are (times 2).
//
// Activations.  An fp16 number is its high byte, which is an E5M2 number (sign, exponent, 2 of 10 mantissa bits), and a rest;
// the rest times 4 is an fp16 number that starts again with its leading bit, and so on: x = d0 + d1 / 4 + d2 / 32 + d3 / 256.  But of 8
// neighbouring products of a row the instruction keeps only what is at least 2^-13 of the largest (measured; beyond these 8 all 24
// bits are kept), cut towards zero.  So every 32-column block is first scaled by a power of two that brings its largest magnitude
// into 2^-7 .. 2^-6, where the last place of E5M2's subnormals, 2^-16, ends a digit before the cut does; the bits below it go
// to the next digit, which starts two or three places lower, and the last one ends where fp16 does, at 2^-24.  So the split is exact and
// nothing is cut; what is rounded are activations below 2^-7 of their block's largest, by the scaling, to the nearest 2^-24.
//
// Precision.  Sums are fp32.  rms error against 64 bits in units of rms(y), all formats and block sizes, for normal activations and with 1 % of the
// channels x 20 to x 4000, of both signs or one: 2.05 - 2.12e-4, the fp16 result alone (the rest is at most 0.2e-4).  Fixed point numbers of 16 bits per quantization block (the dot product unit): 2.2 - 2.6e-4 with such channels.
// The same digits without the scaling: 2.1 - 3.0e-4, and with channels x 1000 / x 4000 of one sign 6e-4 / 1.1e-3, nearly all of it towards zero.
//
// Rows.  The first operand has 16 rows: row 4 b + v is digit v of the tile's 32-column block b, zero in the other blocks'
// columns, so lane group g of a product (lanes 16 g ..) has the four digits' sums of block g, for weight row lane % 16.  That is
// one layout for quantization blocks of 32, 64 and 128; a row's sums meet across the lane groups at the end of the segment.
#pragma once
#include "tman_digits_device.h"

namespace tman {

typedef int v8i_t __attribute__((ext_vector_type(8)));
typedef float v4f_t __attribute__((ext_vector_type(4)));

constexpr int kFp4BytesPerKTile = 512;  // 16 rows x 32 columns
constexpr int kFp4SumBytes = 32;        // (sum, step) of the tile's four 32-column blocks
constexpr int kFp4Zeros = 16;

// The factor between (sum of code value x activation - what the zero takes) as the lanes add it up and y.
template <bool HZ>
constexpr float kFp4Factor = HZ ? 2.f : 4.f;

// 4 x 4 transposition of 16-lane groups and registers: group R comes with w[b], group g leaves with w[r] = what group r had in w[g].
__device__ __forceinline__ void group_transpose(uint32_t (&w)[4]) {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const u32x2 v = __builtin_amdgcn_permlane32_swap(w[h], w[h + 2], false, false);
        w[h] = v.x, w[h + 2] = v.y;
    }
#pragma unroll
    for (int h = 0; h < 4; h += 2) {
        const u32x2 v = __builtin_amdgcn_permlane16_swap(w[h], w[h + 1], false, false);
        w[h] = v.x, w[h + 1] = v.y;
    }
}

// P blocks per quad of lanes: lane f of it holds, of block i, activations 4f .. 4f + 3 (h[i][0], h[i][1]) and 16 + 4f .. .  Digits
// go to `ld[i]` + 32 * digit (the lane's 8 bytes of the block's rows in LDS), sum and step of the block to `ls[i]`.  Returns whether an
// activation is not finite (those count as zero here, see add_nonfinite).  All lanes take part, and all store: the addresses of
// those whose numbers nobody reads point to where nothing is kept yet.
// (Several blocks at once, in one basic block: what a block's digits have to wait for, its largest magnitude and the scale, is a
// chain of 20 instructions.  One block after the other, stores under a branch: 420 and 250 us.)
template <bool HZ, int P>
__device__ __forceinline__ bool store_fp8_digits(uint32_t (&h)[P][4], int lane, const uint32_t (&ld)[P], const uint32_t (&ls)[P]) {
    typedef uint16_t u16x2 __attribute__((ext_vector_type(2)));
    uint32_t mx[P];
    auto largest = [&] {  // of the blocks; magnitudes compare like their bit patterns
#pragma unroll
        for (int i = 0; i < P; ++i) {
            auto magnitudes = [&](int k) { return __builtin_bit_cast(u16x2, h[i][k] & 0x7fff7fffu); };
            const u16x2 m = __builtin_elementwise_max(__builtin_elementwise_max(magnitudes(0), magnitudes(1)), __builtin_elementwise_max(magnitudes(2), magnitudes(3)));
            mx[i] = max_over_lanes<4>(max((uint32_t)m.x, (uint32_t)m.y));
        }
    };
    largest();
    bool nonfinite = false;
#pragma unroll
    for (int i = 0; i < P; ++i) nonfinite |= mx[i] >= 0x7c00u;
    if (__builtin_expect(__builtin_amdgcn_ballot_w64(nonfinite) != 0, 0)) {
#pragma unroll
        for (int i = 0; i < P; ++i)
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                if ((h[i][k] & 0x7c00u) == 0x7c00u) h[i][k] &= 0xffff0000u;
                if ((h[i][k] & 0x7c000000u) == 0x7c000000u) h[i][k] &= 0xffffu;
            }
        largest();
    }
    const uint32_t halves = lane & 1 ? 0x03020706u : 0x05040100u;
    const bool up = lane & 2;
    const float one = opaque(1.f);  // (one mixed-precision instruction per activation)
#pragma unroll
    for (int i = 0; i < P; ++i) {
        // Exponent field e: magnitudes below 2^(e - 14), in steps of 2^(e - 8) below 2^-6.  (1 / step is a subnormal fp16 number from
        // e = 23 on.)
        const uint32_t step_bits = (max(mx[i] & 0x7c00u, 0x400u) << 13) + (119u << 23), inv_bits = (254u << 23) - step_bits;
        const float inv = __builtin_bit_cast(float, inv_bits);
        const _Float16 scale = (_Float16)inv;
        const half2_t scales = {scale, scale};
        float sum = 0.f;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const half2_t v = __builtin_bit_cast(half2_t, h[i][k]);
            sum = fmaf((float)v.x, one, sum);
            sum = fmaf((float)v.y, one, sum);
        }
        sum += __builtin_bit_cast(float, dpp_u32<0xB1>(__builtin_bit_cast(uint32_t, sum)));
        sum += __builtin_bit_cast(float, dpp_u32<0x4E>(__builtin_bit_cast(uint32_t, sum)));
        const float s = HZ ? sum * (inv * 0.5f) : sum * 0.25f;  // half the sum in steps, a quarter of the sum
        store_lds<u32x2>(ls[i], u32x2{__builtin_bit_cast(uint32_t, s), step_bits});
        // Lane o of the quad takes numbers 4f + o: halves of words are exchanged with the lane that differs in bit 0, words with the one
        // that differs in bit 1; x[p] = numbers 8p + o and 8p + 4 + o.
        half2_t x[4];
#pragma unroll
        for (int p = 0; p < 4; p += 2) {
            const uint32_t w0 = __builtin_amdgcn_perm(dpp_u32<0xB1>(h[i][p]), h[i][p], halves), w1 = __builtin_amdgcn_perm(dpp_u32<0xB1>(h[i][p + 1]), h[i][p + 1], halves);
            const uint32_t got = dpp_u32<0x4E>(up ? w0 : w1);
            x[p] = __builtin_bit_cast(half2_t, up ? got : w0) * scales;
            x[p + 1] = __builtin_bit_cast(half2_t, up ? w1 : got) * scales;
        }
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            uint32_t w[2];
#pragma unroll
            for (int q = 0; q < 2; ++q) w[q] = __builtin_amdgcn_perm(__builtin_bit_cast(uint32_t, x[2 * q + 1]), __builtin_bit_cast(uint32_t, x[2 * q]), 0x07050301u);
            store_lds<u32x2>(ld[i] + v * 32, u32x2{w[0], w[1]});
            if (v < 3) {
                const _Float16 by = v == 0 ? (_Float16)4.f : (_Float16)8.f;
#pragma unroll
                for (int p = 0; p < 4; ++p) x[p] = (x[p] - __builtin_bit_cast(half2_t, __builtin_bit_cast(uint32_t, x[p]) & 0xff00ff00u)) * by;
            }
        }
    }
    return nonfinite;
}

// Codes of 32 weights as E2M1 numbers of half their value, word o, field f = weight 4f + o.
template <int B>
__device__ __forceinline__ void planes_to_fp4(const uint32_t (&p)[B], uint32_t (&c)[4]) {
    planes_to_codes<B>(p, c);
    uint32_t mask = B == 2 ? 0x33333333u : 0x11111111u;
    asm("" : "+s"(mask));
#pragma unroll
    for (int o = 0; o < 4; ++o) c[o] &= mask;
}

// Codes times activations of one tile (`st`: lane = row): y[r] += scale (sum - zero S) of block lane / 16 and weight row
// 16 r + lane % 16.  `lo` and `hi`: LDS addresses of the lane's 16 bytes of the first operand in columns 16 g .. and 64 + 16 g ..
// (the zeros, where they are another block's); `ls`: of the tile's block
// sums and steps.
// (Lanes that load what they multiply - four requests of 8 bytes a lane and four for the parameters instead of two and one
// whole ones - save the exchanges and lose a quarter: 16.2 us a launch against 12.6, uint2 g64.)
template <int B, int GQ, bool HZ, typename Next>
__device__ __forceinline__ void multiply_fp4(const Stage<B, 1, GemvCfg<B, 1, GQ, HZ>::MPL>& st, uint32_t lo, uint32_t hi, uint32_t ls,
                                             int lane, float (&y)[4], Next next) {
    using Cfg = GemvCfg<B, 1, GQ, HZ>;
    const u32x4 xl = load_lds<u32x4>(lo), xh = load_lds<u32x4>(hi);
    const u32x2 block = load_lds<u32x2>(ls + (lane >> 4) * 8);
    const v8i_t x = {(int)xl.x, (int)xl.y, (int)xl.z, (int)xl.w, (int)xh.x, (int)xh.y, (int)xh.z, (int)xh.w};
    if constexpr (B == 1) {
        next();
        __builtin_amdgcn_sched_barrier(0);  // (digits and the next tile are requested before the wait for this one)
    }
    uint32_t plane[B][4], meta[4];
#pragma unroll
    for (int b = 0; b < 4; ++b) {
        const int v = (b * 32) / Cfg::CH, ksub = ((b * 32) % Cfg::CH) / 32, mo = (b * 32 / GQ) * Cfg::MSZ;
#pragma unroll
        for (int i = 0; i < B; ++i) plane[i][b] = word_of(st.c[v], ksub * B + i);
        meta[b] = (mo % 4) ? st.meta[mo / 4] >> 16 : st.meta[mo / 4];
    }
#pragma unroll
    for (int i = 0; i < B; ++i) group_transpose(plane[i]);
    group_transpose(meta);
    v4f_t d[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        uint32_t p[B], c[4];
#pragma unroll
        for (int i = 0; i < B; ++i) p[i] = plane[i][r];
        planes_to_fp4<B>(p, c);
        const v8i_t w = {(int)c[0], (int)c[1], (int)c[2], (int)c[3], 0, 0, 0, 0};
        // formats: 1 = E5M2 activations, 4 = E2M1 codes; no scales
        d[r] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(x, w, v4f_t{0.f, 0.f, 0.f, 0.f}, 1, 4, 0, 0, 0, 0);
    }
    const uint32_t sum_w = block.x, step_w = block.y;  // (copied out before the casts)
    const float S = __builtin_bit_cast(float, sum_w), step = __builtin_bit_cast(float, step_w);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        float t = fmaf(d[r][1], 0.25f, d[r][0]);
        t = fmaf(d[r][2], 0.03125f, t);
        t = fmaf(d[r][3], 0.00390625f, t);
        const float sc = half_bits_to_float(meta[r] & 0xffffu);
        if constexpr (HZ) {  // (two mixed-precision instructions and a multiply-add)
            t = fmaf(-half_bits_to_float(meta[r] >> 16), S, t);
            y[r] = fmaf(fmaf(sc, step, 0.f), t, y[r]);
        } else {
            t = fmaf(t, step, -S);
            y[r] = fmaf(sc, t, y[r]);
        }
    }
    if constexpr (B != 1) next();
}

}  // namespace tman
