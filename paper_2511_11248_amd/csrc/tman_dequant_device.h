// Two-level dequantization of the bit-serial layout in registers (Sec. 4.1 "Fused LUT-based dequantization"):
// level 1 turns the bit-plane words of 32 weights into 4-bit codes, level 2 turns a code into the fp16 weight
// with its quantization block's scale and zero baked in.  Shared by the prefill kernel and the small-batch
// matrix-core kernel; both feed the result to MFMA instructions.
#pragma once
#include <hip/hip_fp16.h>

#include "tman_internal.h"

namespace tman {

typedef _Float16 half2_t __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

// (a & mask) | (b & ~mask) and (a & mask) | k as single instructions.  v_bitop3_b32 with all operands in vector registers is one
// of the instructions that two waves of a SIMD issue side by side: 1.07-1.12 ns an instruction from two waves on; 1.85-1.95 for
// v_bfi_b32, for v_and_or_b32 and for itself with a mask in a scalar register.
__device__ __forceinline__ uint32_t in_vgpr(uint32_t constant) {
    asm("" : "+v"(constant));
    return constant;
}
__device__ __forceinline__ uint32_t bfi(uint32_t mask, uint32_t a, uint32_t b) {
    return __builtin_amdgcn_bitop3_b32(in_vgpr(mask), a, b, 0xCA);
}
__device__ __forceinline__ uint32_t and_or(uint32_t a, uint32_t mask, uint32_t k) {
    return __builtin_amdgcn_bitop3_b32(a, in_vgpr(mask), in_vgpr(k), 0xEA);
}

// Level 1: bit planes of 32 weights -> four words of eight 4-bit fields; word o, field f = weight 4f + o.
// For fewer than four planes the upper bits of a field hold bits of other weights; level 2 masks them.
template <int B>
__device__ __forceinline__ void planes_to_codes(const uint32_t (&p)[B], uint32_t (&out)[4]) {
    if constexpr (B == 4) {
        // pair planes (0,1) and (2,3) into 2-bit fields of even / odd weights, then pair those into nibbles
        const uint32_t a = bfi(0x55555555u, p[0], p[1] << 1);  // field e: low two code bits of weight 2e
        const uint32_t b = bfi(0x55555555u, p[0] >> 1, p[1]);  // same for weight 2e + 1
        const uint32_t c = bfi(0x55555555u, p[2], p[3] << 1);  // high two code bits of weight 2e
        const uint32_t d = bfi(0x55555555u, p[2] >> 1, p[3]);
        out[0] = bfi(0x33333333u, a, c << 2);  // weights 4f
        out[2] = bfi(0x33333333u, a >> 2, c);  // weights 4f + 2
        out[1] = bfi(0x33333333u, b, d << 2);  // weights 4f + 1
        out[3] = bfi(0x33333333u, b >> 2, d);  // weights 4f + 3
    } else if constexpr (B == 2) {
        const uint32_t a = bfi(0x55555555u, p[0], p[1] << 1);
        const uint32_t b = bfi(0x55555555u, p[0] >> 1, p[1]);
        out[0] = a;
        out[2] = a >> 2;
        out[1] = b;
        out[3] = b >> 2;
    } else {
#pragma unroll
        for (int o = 0; o < 4; ++o) out[o] = p[0] >> o;
    }
}

// raw data of one 32-weight block of a stage for one lane (= one row)
template <int B>
struct WRegs {
    uint32_t plane[B];
    uint32_t meta;  // scale (low 16 bits) and zero (high 16 bits) of the block's quantization group
};

// Level 2 for one lane's 32 weights; writes them as fp16, in column order, into its row of the LDS
// weight tile (`wrow` already points at the block's 64 bytes).
//
// Field f of code word o (weight 4f + o) is turned into an fp16 number without moving it to bit 0:
// a nibble at mantissa bits 0..3 of 0x6400 reads 1024 + c, one at bits 4..7 reads 1024 + 16c.  Fields
// f and f + 4 sit 16 bits apart, so one AND-OR makes two such numbers; a single shift by 8 brings
// fields 2, 3, 6, 7 into reach.  The affine map (c - zero) * scale is then one fp32 FMA per weight:
// (1024 + c) * s - (1024 + z) * s   or   (1024 + 16c) * s/16 - (64 + z) * s   (the second, constant
// term is itself rounded to fp32 when the block's constants are prepared), and the conversion of two of them to fp16 puts weights
// 4f + o and 4f + o + 1 (from the same field of two code words) side by side.
template <int B, bool HZ>
struct Dequant {
    uint32_t codes[4];
    float mul[2], bias[2];  // [0]: nibble at mantissa bits 0..3, [1]: at bits 4..7
    half2_t P[4][4];        // [o][d]: halves = fields d and d + 4 of code word o, as 1024 + c or 1024 + 16c

    // part 1: level 1 and the block's constants
    __device__ __forceinline__ void start(const WRegs<B>& r) {
        planes_to_codes<B>(r.plane, codes);
        const float s = (float)__builtin_bit_cast(_Float16, (uint16_t)(r.meta & 0xffffu));
        if constexpr (HZ) {
            const float z = (float)__builtin_bit_cast(_Float16, (uint16_t)(r.meta >> 16));
            mul[0] = s;
            bias[0] = -(1024.f + z) * s;
            mul[1] = s * 0.0625f;
            bias[1] = -(64.f + z) * s;
        } else {
            mul[0] = 2.f * s;  // (2c - 1) * s
            bias[0] = -2049.f * s;
            mul[1] = s * 0.125f;
            bias[1] = -129.f * s;
        }
    }
    // part 2: codes -> fp16 integers
    __device__ __forceinline__ void insert() {
        constexpr uint32_t kCodeMask = (1u << B) - 1u;
        constexpr uint32_t kMaskLo = kCodeMask | (kCodeMask << 16), kMaskHi = kMaskLo << 4;
#pragma unroll
        for (int o = 0; o < 4; ++o) {
            const uint32_t c = codes[o], c8 = codes[o] >> 8;
            P[o][0] = __builtin_bit_cast(half2_t, and_or(c, kMaskLo, 0x64006400u));
            P[o][1] = __builtin_bit_cast(half2_t, and_or(c, kMaskHi, 0x64006400u));
            P[o][2] = __builtin_bit_cast(half2_t, and_or(c8, kMaskLo, 0x64006400u));
            P[o][3] = __builtin_bit_cast(half2_t, and_or(c8, kMaskHi, 0x64006400u));
        }
    }
    // part 3: 16-byte piece q (weights 8q .. 8q + 7 = fields 2q, 2q + 1) as four pairs of fp16
    __device__ __forceinline__ u32x4 piece(int q) const {
        u32x4 out;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int f = 2 * q + (i >> 1), o = (i & 1) * 2, d = f & 3, t = d & 1;
            const _Float16 va = (f >> 2) ? P[o][d].y : P[o][d].x;
            const _Float16 vb = (f >> 2) ? P[o + 1][d].y : P[o + 1][d].x;
            // two v_fma_mix_f32 and one v_cvt_pk_f16_f32 (5.6 ns): v_fma_mixlo_f16 and _mixhi_f16, which would round
            // themselves, issue at half rate (7.0 ns)
            float a = fmaf((float)va, mul[t], bias[t]), b = fmaf((float)vb, mul[t], bias[t]);
            asm("" : "+v"(a));
            asm("" : "+v"(b));
            half2_t w;
            w.x = (_Float16)a;
            w.y = (_Float16)b;
            out[i] = __builtin_bit_cast(uint32_t, w);
        }
        return out;
    }
    // ... written to its place in an LDS row
    __device__ __forceinline__ void emit(int q, uint8_t* wrow) const { *reinterpret_cast<u32x4*>(wrow + q * 16) = piece(q); }
};

template <int B, bool HZ>
__device__ __forceinline__ void dequant_to_lds(const WRegs<B>& r, uint8_t* wrow) {
    Dequant<B, HZ> dq;
    dq.start(r);
    dq.insert();
#pragma unroll
    for (int q = 0; q < 4; ++q) dq.emit(q, wrow);
}

// Elements of type T of an output tile, consecutive lanes to consecutive elements of a row: `live` rows of TM / (elements per T).
template <typename T, int TM, int OUT_ROW, int THREADS>
__device__ __forceinline__ void store_elements(_Float16* y, int M, const uint8_t* otile, int m0, int n0, int live, int tid) {
    constexpr int kPer = sizeof(T) / 2, kRowItems = TM / kPer;
#pragma unroll 4
    for (int i = tid; i < live * kRowItems; i += THREADS) {
        const int n = i / kRowItems, m = i % kRowItems * kPer;
        if (m0 + m < M)
            *reinterpret_cast<T*>(y + (size_t)(n0 + n) * M + m0 + m) = *reinterpret_cast<const T*>(otile + n * OUT_ROW + m * 2);
    }
}

// Stores an fp16 output tile kept in LDS as [token][row].  Rows of y that are 16-byte aligned: 16-byte pieces, coalesced; a whole tile
// takes four pieces of a thread at a time, so that their reads and stores overlap.  Other rows of y: words or elements, each store of a
// wave a piece of one or two rows.  (Element by element of a thread's own 16 bytes a store touched eight or more lines, which counts most
// where few threads store a tile: 19022 x 256 N = 93, 256 x 96 tiles 13.3 -> 9.7 us; 15731 x 320 N = 1997, 256 x 256 tiles 70.3 -> 37.7.)
template <int TM, int TN, int OUT_ROW, int THREADS>
__device__ __forceinline__ void store_tile(_Float16* y, int M, int N, const uint8_t* otile, int m0, int n0, int tid) {
    constexpr int kPieces = TN * (TM / 8);
    if (M % 8 != 0 || !aligned16(y)) {
        const int live = N - n0 < TN ? N - n0 : TN;
        if (M % 2 == 0 && ((uintptr_t)y & 3) == 0) store_elements<uint32_t, TM, OUT_ROW, THREADS>(y, M, otile, m0, n0, live, tid);
        else store_elements<uint16_t, TM, OUT_ROW, THREADS>(y, M, otile, m0, n0, live, tid);
        return;
    }
    if (m0 + TM <= M && n0 + TN <= N) {
#pragma unroll 4
        for (int piece = tid; piece < kPieces; piece += THREADS) {
            const int n = piece / (TM / 8), c8 = piece % (TM / 8);
            *reinterpret_cast<u32x4*>(y + (size_t)(n0 + n) * M + m0 + c8 * 8) =
                *reinterpret_cast<const u32x4*>(otile + n * OUT_ROW + c8 * 16);
        }
        return;
    }
    for (int piece = tid; piece < kPieces; piece += THREADS) {
        const int n = piece / (TM / 8), c8 = piece % (TM / 8);
        const int gn = n0 + n, gm = m0 + c8 * 8;
        if (gn < N && gm < M)  // (M is a multiple of 8)
            *reinterpret_cast<u32x4*>(y + (size_t)gn * M + gm) = *reinterpret_cast<const u32x4*>(otile + n * OUT_ROW + c8 * 16);
    }
}

}  // namespace tman
