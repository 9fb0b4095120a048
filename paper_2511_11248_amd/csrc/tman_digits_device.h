// Device-side building blocks of the decoding kernels that multiply codes with integer activations on the 4-bit dot
// product unit: activations as 16-bit fixed-point numbers split into four signed 4-bit digits, weights as 4-bit codes,
// v_dot8c_i32_i4 (eight products and their sum in one vector instruction).
//
// Why digits instead of table lookups.  A lookup costs 2.6 vector instructions and one LDS read per 4 weights and
// bit-plane (an address, the addition, the index preparation), so 4-bit weights cost 2.6 instructions each and the
// lookup kernel was bound by vector issue.  Here a block of 32 weights costs its bit transposition (17 instructions
// for 4-bit codes, 10 for 2-bit ones) and 16 dot products: 1.03 and 0.81 instructions per weight, no gather from LDS.
//
// Digits.  Every quantization block gets a power-of-two step 2^e, the smallest for which all |x| / 2^e <= 30583, the
// largest number that four digits d_i in -8 .. 7 hold: X = round_to_nearest_even(x / 2^e) = sum 16^i d_i (the nibbles
// of X + 0x8888, each exclusive-or 8).  Against fp16 table entries, which round every sum of four activations to 11
// bits, only activations below 1/14 of their block's largest are rounded at all.  (With |x| / 2^e < 2^14, a step twice
// as large for seven maxima out of eight, blocks of 128 with channels of 100 to 1000 times the others came out up to 4 %
// worse than through fp16 tables: rms error 3.4e-4 to 3.5e-4 of rms(y) for all formats; now 2.5e-4.)  All products and
// sums inside a block are exact integers (|sum| <= 30583 * 15 * 128 < 2^26).
//
// Order.  The bit transposition leaves weight 4f + o of a 32-weight block in field f of word o, so digit word
// (o, i) holds digit i of activations 4f + o.  A block's 16 digit words are read from LDS by ONE ds_read_b32 per
// lane - lane l takes word l % 16 - and every dot product picks its word with the DPP row broadcast: an LDS read
// that delivered each word to all lanes would take 32 cycles per block and compute unit, as long as the arithmetic.
#pragma once
#include "tman_dequant_device.h"
#include "tman_gemv_device.h"

namespace tman {

constexpr int kDigitBytesPerKTile = 256;  // 4 blocks x 16 words
constexpr int kDigitMetaBytes = 16;       // per quantization block: sum of X (float), step (float), 8 * sum of X (int)

// acc[i] += sum over the block's 32 weights of code * (digit i), for the four digits.  `dg` holds digit word l % 16 of
// the block in lane l, word o * 4 + i = digit i of activations 4f + o.
// (s_nop: a VGPR written by a vector instruction may be read through DPP two wait states later, and the result of a
// dot product by another kind of vector instruction three later; the compiler does not look into the block.)
__device__ __forceinline__ void dot_block(int (&acc)[4], uint32_t dg, const uint32_t (&c)[4]) {
#define TMAN_DOT(i, o, w) "v_dot8c_i32_i4_dpp %" #i ", %4, %" #o " row_newbcast:" #w " row_mask:0xf bank_mask:0xf\n"
    asm("s_nop 1\n"
        TMAN_DOT(0, 5, 0) TMAN_DOT(1, 5, 1) TMAN_DOT(2, 5, 2) TMAN_DOT(3, 5, 3)
        TMAN_DOT(0, 6, 4) TMAN_DOT(1, 6, 5) TMAN_DOT(2, 6, 6) TMAN_DOT(3, 6, 7)
        TMAN_DOT(0, 7, 8) TMAN_DOT(1, 7, 9) TMAN_DOT(2, 7, 10) TMAN_DOT(3, 7, 11)
        TMAN_DOT(0, 8, 12) TMAN_DOT(1, 8, 13) TMAN_DOT(2, 8, 14) TMAN_DOT(3, 8, 15)
        "s_nop 3\n"
        : "+v"(acc[0]), "+v"(acc[1]), "+v"(acc[2]), "+v"(acc[3])
        : "v"(dg), "v"(c[0]), "v"(c[1]), "v"(c[2]), "v"(c[3]));
#undef TMAN_DOT
}

// Codes of 32 weights as signed 4-bit fields, word o, field f = weight 4f + o: the code itself for 1 and 2 bits,
// code - 8 for 4 bits (made good with 8 times the block's sum of X).
template <int B>
__device__ __forceinline__ void planes_to_signed_codes(const uint32_t (&p)[B], uint32_t (&out)[4]) {
    if constexpr (B == 4) {
        const uint32_t q[4] = {p[0], p[1], p[2], ~p[3]};  // code ^ 8, read as a signed nibble, is code - 8
        planes_to_codes<4>(q, out);
    } else {
        planes_to_codes<B>(p, out);
#pragma unroll
        for (int o = 0; o < 4; ++o) out[o] &= B == 2 ? 0x33333333u : 0x11111111u;
    }
}

// A DPP move of a 32-bit word.
template <int CTRL>
__device__ __forceinline__ uint32_t dpp_u32(uint32_t v) {
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, 0xF, 0xF, true);
}

// Largest value and sum over blocks of W consecutive lanes (W = 4, 8 or 16), in every lane of the block.
template <int W>
__device__ __forceinline__ uint32_t max_over_lanes(uint32_t v) {
    v = max(v, dpp_u32<0xB1>(v));  // lane ^ 1
    v = max(v, dpp_u32<0x4E>(v));  // lane ^ 2
    if constexpr (W >= 8) v = max(v, dpp_u32<0x141>(v));   // the other quad of 8 lanes
    if constexpr (W >= 16) v = max(v, dpp_u32<0x140>(v));  // the other half of 16 lanes
    return v;
}
template <int W>
__device__ __forceinline__ int isum_over_lanes(int v) {
    v += (int)dpp_u32<0xB1>((uint32_t)v);
    v += (int)dpp_u32<0x4E>((uint32_t)v);
    if constexpr (W >= 8) v += (int)dpp_u32<0x141>((uint32_t)v);
    if constexpr (W >= 16) v += (int)dpp_u32<0x140>((uint32_t)v);
    return v;
}

// 4 x 4 transposition over a quad of lanes: lane f comes with r[o], lane o leaves with r[f].
__device__ __forceinline__ void quad_transpose(uint32_t (&r)[4], int lane) {
    const bool odd = lane & 1, up = lane & 2;
#pragma unroll
    for (int h = 0; h < 4; h += 2) {  // 2 x 2 blocks: lanes differing in bit 0, registers differing in bit 0
        const uint32_t got = dpp_u32<0xB1>(odd ? r[h] : r[h + 1]);
        r[h] = odd ? got : r[h];
        r[h + 1] = odd ? r[h + 1] : got;
    }
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const uint32_t got = dpp_u32<0x4E>(up ? r[h] : r[h + 2]);
        r[h] = up ? got : r[h];
        r[h + 2] = up ? r[h + 2] : got;
    }
}

// From 16-bit numbers to digit words, for a quad of lanes that holds one 32-weight block: lane f (of 4) comes with
// r[o] = number 4f + o of the block in the low half, 16 + 4f + o in the high half (as X + 0x8888), and leaves with
// r[i] = digit word (o = its lane, i): a 4 x 4 transposition over the quad, then one of nibbles.
__device__ __forceinline__ void digit_words(uint32_t (&r)[4], int lane) {
    quad_transpose(r, lane);
    // r[f] now holds the numbers 4f + o and 4 (f + 4) + o of this lane's o; nibble i of each goes to word i
    const uint32_t a0 = bfi(0x00FF00FFu, r[0], r[2] << 8), a1 = bfi(0x00FF00FFu, r[1], r[3] << 8);
    const uint32_t b0 = bfi(0xFF00FF00u, r[2], r[0] >> 8), b1 = bfi(0xFF00FF00u, r[3], r[1] >> 8);
    r[0] = bfi(0x0F0F0F0Fu, a0, a1 << 4) ^ 0x88888888u;
    r[1] = bfi(0xF0F0F0F0u, a1, a0 >> 4) ^ 0x88888888u;
    r[2] = bfi(0x0F0F0F0Fu, b0, b1 << 4) ^ 0x88888888u;
    r[3] = bfi(0xF0F0F0F0u, b1, b0 >> 4) ^ 0x88888888u;
}

// Sum of the lane's eight numbers from its digit words (digit i counts 16^i).
__device__ __forceinline__ int sum_of_digits(const uint32_t (&w)[4]) {
    int s = 0;
#pragma unroll
    for (int i = 3; i >= 0; --i) s = (s << 4) + __builtin_amdgcn_sdot8((int)w[i], 0x11111111, 0, false);
    return s;
}

// The sums of the four digits, put together (modulo 2^32): three shift-adds (left to itself the compiler makes two shifts,
// a shift-add and an addition of three).
__device__ __forceinline__ uint32_t join_digits(const int (&acc)[4]) {
    uint32_t s = ((uint32_t)acc[3] << 4) + (uint32_t)acc[2];
    asm("" : "+v"(s));
    s = (s << 4) + (uint32_t)acc[1];
    asm("" : "+v"(s));
    return (s << 4) + (uint32_t)acc[0];
}

// Numbers of a quad of lanes -> digits in LDS.  Lane f (of 4) of a quad holds of one 32-weight block, in r[o], number
// 4f + o (low half) and 16 + 4f + o (high half), as X + 0x8888.  The lane's four words of the block go to `ld`, and the
// first lane of every quantization block (GQ / 8 lanes) stores the block's (sum of X, step, 8 * sum) at `lm`.  `i`: index
// of the lane in the segment.  All lanes take part in the exchanges; with `live` false nothing is stored.
template <int GQ>
__device__ __forceinline__ void store_digits(uint32_t (&r)[4], float step, int i, bool live, uint32_t ld, uint32_t lm) {
    constexpr int LPG = GQ / 8;  // lanes per quantization block
    digit_words(r, i & 3);
    const int sum = isum_over_lanes<LPG>(sum_of_digits(r));
    if (live) {
        store_lds<u32x4>(ld, u32x4{r[0], r[1], r[2], r[3]});
        if (i % LPG == 0)
            store_lds<u32x4>(lm, u32x4{__builtin_bit_cast(uint32_t, (float)sum), __builtin_bit_cast(uint32_t, step),
                                       (uint32_t)sum << 3, 0u});
    }
}

// fp16 activations of the lane (xa: 4f .. 4f + 3, xb: 16 + 4f ..) -> numbers in the form store_digits takes and the
// step of their quantization block.  Returns whether one of them is not finite (those count as zero here, see
// add_nonfinite).
template <int GQ>
__device__ __forceinline__ bool quantize_block(const u32x2& xa, const u32x2& xb, uint32_t (&r)[4], float& step) {
    uint32_t h[4] = {xa.x, xa.y, xb.x, xb.y};  // activations in pairs
    auto largest = [&]() {                     // magnitudes compare like their bit patterns
        uint32_t m = 0;
#pragma unroll
        for (int k = 0; k < 4; ++k) m = max(m, max(h[k] & 0x7fffu, (h[k] >> 16) & 0x7fffu));
        return m;
    };
    uint32_t mx = largest();
    const bool nonfinite = mx >= 0x7c00u;
    if (__builtin_expect(nonfinite, 0)) {
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            if ((h[k] & 0x7c00u) == 0x7c00u) h[k] &= 0xffff0000u;
            if ((h[k] & 0x7c000000u) == 0x7c000000u) h[k] &= 0xffffu;
        }
        mx = largest();
    }
    // The block's largest magnitude is (1024 + f) * 2^(e - 25), e its exponent field: 16 (1024 + f) steps of 2^(e - 29)
    // if that is at most 30583, f <= 887, else 8 (1024 + f) steps twice as large.  Adding 136 = 1023 - 887 to the bit
    // pattern carries into the exponent in the second case: step 2^(eb - 29) (subnormals: that of e = 1).
    const uint32_t eb = max((max_over_lanes<GQ / 8>(mx) + 136u) >> 10, 1u);
    const float up = __builtin_bit_cast(float, (156u - eb) << 23);  // 2^(29 - eb)
    step = __builtin_bit_cast(float, (98u + eb) << 23);             // 2^(eb - 29)
    // x * 2^(29 - eb) rounded to an integer by adding 1.5 * 2^23: the low 16 bits of the sum are X (+ 0x8888)
    constexpr float kMagic = 12582912.f + 34952.f;
    uint32_t n[4][2];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const half2_t v = __builtin_bit_cast(half2_t, h[k]);
        n[k][0] = __builtin_bit_cast(uint32_t, fmaf((float)v.x, up, kMagic));
        n[k][1] = __builtin_bit_cast(uint32_t, fmaf((float)v.y, up, kMagic));
    }
#pragma unroll
    for (int o = 0; o < 4; ++o) r[o] = __builtin_amdgcn_perm(n[2 + o / 2][o & 1], n[o / 2][o & 1], 0x05040100u);
    return nonfinite;
}

// The same for integer activations (14-bit numbers in pairs, step 1).
__device__ __forceinline__ void bias_block(const u32x2& xa, const u32x2& xb, uint32_t (&r)[4]) {
    typedef uint16_t u16x2 __attribute__((ext_vector_type(2)));
    const uint32_t h[4] = {xa.x, xa.y, xb.x, xb.y};
#pragma unroll
    for (int o = 0; o < 4; ++o) {
        const uint32_t both = __builtin_amdgcn_perm(h[2 + o / 2], h[o / 2], o & 1 ? 0x07060302u : 0x05040100u);
        const u16x2 v = __builtin_bit_cast(u16x2, both) + (uint16_t)0x8888;
        r[o] = __builtin_bit_cast(uint32_t, v);
    }
}

// Codes times activations of one tile block for the lane's row.  `dbase` is the LDS address of the tile's digit words
// plus 4 (lane % 16), `mbase` of its blocks' records.  The accumulators run on over blocks and tiles, and a block's sum is
// what they gained (`before`: their joined value so far; integers modulo 2^32), one subtraction instead of clearing four
// registers per block.
// Vector instructions per tile for 1 bit, blocks of 32 / 64: 147 -> 127, 121 -> 111 (with the shorter join_digits and the
// scale read as fp16 by the multiplication).
// `next` requests the wave's next tile: when this one is done, into its stage, or (1 bit) before the wait for this one, into
// another stage.
template <int B, int GQ, bool HZ, typename Next>
__device__ __forceinline__ void consume_weights_digits(const Stage<B, 1, GemvCfg<B, 1, GQ, HZ>::MPL>& s, uint32_t dbase,
                                                       uint32_t mbase, int (&acc)[4], uint32_t& before, float& y, Next next) {
    using Cfg = GemvCfg<B, 1, GQ, HZ>;
    constexpr int BPG = GQ / 32;  // 32-weight blocks per quantization block
    uint32_t dg[4];
    // a block's record: (sum of X, step), and 8 * sum for 4 bits.  (Of a 16-byte read whose last words nobody uses the
    // compiler lets the next read overwrite those, and waits for each.)
    typedef std::conditional_t<B == 4, u32x4, u32x2> record_t;
    record_t gm[Cfg::GPT];
#pragma unroll
    for (int b = 0; b < 4; ++b) dg[b] = load_lds<uint32_t>(dbase + b * 64);
#pragma unroll
    for (int gi = 0; gi < Cfg::GPT; ++gi) gm[gi] = load_lds<record_t>(mbase + gi * kDigitMetaBytes);
    if constexpr (B == 1) {
        next();
        __builtin_amdgcn_sched_barrier(0);  // (digits and the next tile are requested before the wait for this one)
    }
#pragma unroll
    for (int gi = 0; gi < Cfg::GPT; ++gi) {
#pragma unroll
        for (int b = gi * BPG; b < (gi + 1) * BPG; ++b) {
            const int v = (b * 32) / Cfg::CH, ksub = ((b * 32) % Cfg::CH) / 32;
            uint32_t p[B], c[4];
#pragma unroll
            for (int i = 0; i < B; ++i) p[i] = word_of(s.c[v], ksub * B + i);
            planes_to_signed_codes<B>(p, c);
            dot_block(acc, dg[b], c);
        }
        const int mo = gi * Cfg::MSZ;
        const uint32_t mw = s.meta[mo / 4];
        const float scale = half_bits_to_float((mo % 4) ? (mw >> 16) : (mw & 0xffffu));
        const uint32_t gs_w = gm[gi].x, step_w = gm[gi].y;  // (copied out before the casts)
        const float gs = __builtin_bit_cast(float, gs_w), step = __builtin_bit_cast(float, step_w);
        const uint32_t now = join_digits(acc);
        uint32_t own = now - before;
        before = now;
        if constexpr (B == 4) own += gm[gi].z;  // fields hold code - 8
        const float a = (float)(int)own;
        const float sc = fmaf(scale, step, 0.f);  // (one mixed-precision instruction)
        if constexpr (HZ) {
            const float z = half_bits_to_float(mw >> 16);
            y = fmaf(sc, fmaf(-z, gs, a), y);
        } else {
            y = fmaf(sc, fmaf(2.f, a, -gs), y);
        }
    }
    if constexpr (B != 1) next();
}

// Activations that are not finite take no part in the integer arithmetic (their X is 0); their products with the
// lane's weights of tile t are added here one by one, (code - zero) * scale * x in fp32, so that infinities and NaN come
// out as in the sum over all columns.  Reached only when the segment has such an activation.  `fetch` gives the bits
// of activation k; the lanes look at two columns each, so a tile without one costs two loads (with a load per column
// one infinity made four launches of a 7B layer set, uint4 g128, 411 us instead of 79).
template <int B, int GQ, bool HZ, typename Fetch>
__device__ __forceinline__ float add_nonfinite(const uint8_t* tile, Fetch fetch, int K, int t, int lane, float y) {
    using Cfg = GemvCfg<B, 1, GQ, HZ>;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const int k0 = t * kKTile + h * 64;
        const uint32_t mine = k0 + lane < K ? fetch(k0 + lane) : 0u;
        uint64_t left = __builtin_amdgcn_ballot_w64((mine & 0x7c00u) == 0x7c00u);
        for (; left; left &= left - 1) {
            const int j = __builtin_ctzll(left), b = 2 * h + j / 32;
            const int v = (b * 32) / Cfg::CH, ksub = ((b * 32) % Cfg::CH) / 32;
            uint32_t c = 0;
#pragma unroll
            for (int i = 0; i < B; ++i)
                c |= ((load_global<uint32_t>(tile, v * 1024 + lane * 16 + (ksub * B + i) * 4) >> (j % 32)) & 1u) << i;
            const uint32_t mo = B * 1024 + lane * Cfg::MPL + ((h * 64 + j) / GQ) * Cfg::MSZ;
            const float sc = half_bits_to_float(load_global<uint16_t>(tile, mo));
            const float wt = HZ ? ((float)c - half_bits_to_float(load_global<uint16_t>(tile, mo + 2))) * sc : (2.f * (float)c - 1.f) * sc;
            y += wt * half_bits_to_float((uint32_t)__builtin_amdgcn_readlane((int)mine, j));
        }
    }
    return y;
}

}  // namespace tman
