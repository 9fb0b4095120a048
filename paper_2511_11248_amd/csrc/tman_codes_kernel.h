// The product of codes and a handful of tokens on the matrix cores, as a template over the weight format, the number of
// tokens and where the activations come from (as such: tman_mpgemm for 2 .. 32 tokens; out of lookup tables: tman_mpgemv and
// tman_mpgemv_i16 for 2 .. 8 tokens, see lookups_stay).
//
// The matrix cores multiply the codes themselves, as exact fp16 numbers off + c (the code inserted into the mantissa of a
// power of two), and a quantization block's scale and zero are applied to its sums:
//   y[n][m] += s[m] * (acc[n][m] - (off + z[m]) * S[n]),   acc = sum (off + c) x,  S = sum x over the block.
// The offset costs 1 to 4 bits of the fp32 accumulator; weights are not rounded to fp16, so the sums are closer to the
// exact ones than those of dequantized weights or of 16-bit table entries (rms 2.1e-4 of rms(y), the fp16 result alone,
// from 2.9e-4 and 3.6e-4).
//
// The activations are the FIRST operand and the weights the second, so that a lane's accumulators belong to ONE row of W
// and the registers to tokens: a block's scale and zero are one value per lane and row group.  S comes from a product of
// the activations with ones, in the accumulators' own layout.
//
// Roles of the lanes.  v_mfma_f32_16x16x32 (and 32x32x16) takes, per operand, 8 numbers of K from each group of 16 (32)
// lanes.  Which columns those are is free as long as both operands agree, so lane group g takes whole 32-column blocks: of
// the rows 16 r + i (32 r + i) block g (blocks g and 2 + g), which a lane loads, transposes to codes and multiplies without
// exchanging anything with other lanes.  (With a row of its own per lane, as in the other kernels, a tile cost 32 exchanges
// of registers and 32 v_perm for the activations.)  A product then sums over 128 (64) columns.  Where that is more
// than a quantization block, rows 0 .. 7 and 8 .. 15 of the first operand hold the same 8 tokens, each with the other's
// columns left out, so that the sums of two quantization blocks come out in different registers or lanes.
// 16 x 16: blocks of 128 with up to 16 tokens, blocks of 64 with up to 8; 32 x 32 otherwise.
//
// What bounds it (7B uint4 g128, 8 tokens: 107.5 MB in 23.6 us = 4.55 TB/s, with a row per lane and 32 x 32 products 27.0).
// Not vector issue (about 250 instructions per tile block), which runs beside the matrix cores: without the
// transposition the time is the same.  Without the products it falls by a fifth, without the activations by a fifth:
// the clock under HBM and matrix load, and the wait for the activations behind the weights.  So rows of a product without
// a token are zeros (numbers there cost 5 %), the smaller product is used where it can be, and the activations of a tile are
// requested once per wave in full lines (two requests of 1 KB for 8 tokens; a request per operand, three quarters of its
// lanes beyond the tokens, made 8).
#pragma once
#include "tman_dequant_device.h"
#include "tman_gemv_device.h"

namespace tman {

typedef float float4v_t __attribute__((ext_vector_type(4)));
typedef float float16_t __attribute__((ext_vector_type(16)));

constexpr int kSmallTokens = TMAN_MAX_SMALL_TOKENS;  // 32: the token extent of one MFMA
constexpr int kRedStride = kRows + 4;                  // floats per token in the LDS reduction buffer (bank spread)

// The offset: 64 for 4 bits (a nibble at mantissa bits 4..7 needs three shifts per code word; at bits 6..9, as 16 + c, it
// would need four), 4 for 2 bits (bits 8..9), 2 for 1 bit (bit 9): small against the codes, because what the offset
// adds to the sums is lost to their precision.  Level 1 leaves weights k and k + 16 of a 32-column block in the halves of
// one register; the activations are paired to match.
template <int B>
constexpr float kCodeOffset = B == 4 ? 64.f : B == 2 ? 4.f : 2.f;
template <int B>
__device__ __forceinline__ void codes_to_half_pairs(const uint32_t (&p)[B], uint32_t (&w)[16]) {
    // (Constants the compiler cannot look through, so that each pair is one v_and_or_b32; not in an asm block, because the
    // products read these registers at once and the compiler has to see which instruction wrote them to keep the wait
    // states between the two.)
    uint32_t mask = B == 4 ? 0x00F000F0u : B == 2 ? 0x03000300u : 0x02000200u;
    uint32_t base = B == 4 ? 0x54005400u : B == 2 ? 0x44004400u : 0x40004000u;
    asm("" : "+s"(mask));
    asm("" : "+v"(base));
    auto place = [](uint32_t v, int from, int to) { return from < to ? v << (to - from) : v >> (from - to); };
    if constexpr (B == 1) {
#pragma unroll
        for (int k = 0; k < 16; ++k) w[k] = (place(p[0], k, 9) & mask) | base;
    } else {
        uint32_t c[4];  // word o, field f: weight 4f + o; fields f and f + 4 are 16 bits apart
        planes_to_codes<B>(p, c);
#pragma unroll
        for (int f = 0; f < 4; ++f)
#pragma unroll
            for (int o = 0; o < 4; ++o) w[4 * f + o] = (place(c[o], 4 * f, B == 4 ? 4 : 8) & mask) | base;
    }
}

// The lane's row of tile block t (in `st`) times the activations of one token (`fetch` gives the bits
// of activation k), weight by weight.
template <int B, int GQ, bool HZ, typename Fetch>
__device__ __forceinline__ float add_products(const Stage<B, 1, GemvCfg<B, 1, GQ, HZ>::MPL>& st, Fetch fetch, int K, int t,
                                              int lane, float sum) {
    using Cfg = GemvCfg<B, 1, GQ, HZ>;
    uint32_t xv[2];  // lane l holds columns l and 64 + l of the tile
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int k = t * kKTile + i * 64 + lane;
        xv[i] = k < K ? fetch(k) : 0u;
    }
#pragma unroll
    for (int b = 0; b < 4; ++b) {
        if (t * kKTile + b * 32 >= K) break;  // (uniform)
        const int v = (b * 32) / Cfg::CH, ksub = ((b * 32) % Cfg::CH) / 32;
        uint32_t p[B], c[4];
#pragma unroll
        for (int i = 0; i < B; ++i) p[i] = word_of(st.c[v], ksub * B + i);
        planes_to_codes<B>(p, c);
        const int mo = (b * 32 / GQ) * Cfg::MSZ;
        const uint32_t mw = (mo % 4) ? st.meta[mo / 4] >> 16 : st.meta[mo / 4];
        const float sc = half_bits_to_float(mw & 0xffffu), z = HZ ? half_bits_to_float(mw >> 16) : 0.f;
#pragma unroll 1
        for (int f = 0; f < 8; ++f) {
#pragma unroll
            for (int o = 0; o < 4; ++o) {  // weight 4f + o is field f of word o
                const float code = (float)((c[o] >> (4 * f)) & ((1u << B) - 1u));
                const float wt = HZ ? (code - z) * sc : (2.f * code - 1.f) * sc;
                sum += wt * half_bits_to_float((uint32_t)__builtin_amdgcn_readlane((int)xv[b / 2], (b % 2) * 32 + 4 * f + o));
            }
        }
    }
    return sum;
}

// Output of one row block: thread -> (token, rows r8 .. r8 + 7 of the block) with the sums of the workgroup's K segment.
// `STRIDE`: tokens per segment and row block in the workspace.
template <int STRIDE>
__device__ __forceinline__ void finish_tokens(const GemvDesc& d, int rb, int seg, int n_seg, int token, int r8, int M, int N,
                                              const float (&sum)[8]) {
    __shared__ int last_flag;
    const int m0 = rb * kRows + r8;
    _Float16* out = static_cast<_Float16*>(d.y);
    const bool wide = M % 8 == 0 && aligned16(out);  // 16-byte aligned rows of y
    auto store_rows = [&](const float (&v)[8]) {
        if (token >= N) return;
        _Float16* dst = out + (size_t)token * M + m0;
        if (wide && m0 + 8 <= M) {
            half8_t h;
#pragma unroll
            for (int e = 0; e < 8; ++e) h[e] = (_Float16)v[e];
            *reinterpret_cast<half8_t*>(dst) = h;
        } else {
#pragma unroll
            for (int e = 0; e < 8; ++e)
                if (m0 + e < M) dst[e] = (_Float16)v[e];
        }
    };
    if (n_seg == 1) {
        store_rows(sum);
        return;
    }

    // K longer than one segment: publish this segment's sums, take a ticket; the last one adds in segment order
    float* base_p = d.partial + (size_t)rb * n_seg * STRIDE * kRows;
    float* mine = base_p + (size_t)seg * STRIDE * kRows + token * kRows + r8;
    if (token < N) {
#pragma unroll
        for (int e = 0; e < 8; ++e) __hip_atomic_store(mine + e, sum[e], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // the sums have reached device-coherent memory
    __syncthreads();
    int32_t* ticket = d.tickets + rb;
    if (threadIdx.x == 0) last_flag = __hip_atomic_fetch_add(ticket, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == n_seg - 1;
    __syncthreads();
    if (!last_flag) return;
    float total[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) total[e] = 0.f;
    if (token < N) {
        for (int p = 0; p < n_seg; ++p) {
            const float* src_p = base_p + (size_t)p * STRIDE * kRows + token * kRows + r8;
            float v[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) v[e] = __hip_atomic_load(src_p + e, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
            for (int e = 0; e < 8; ++e) total[e] += v[e];
        }
    }
    store_rows(total);
    if (threadIdx.x == 0) __hip_atomic_store(ticket, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// LDS per wave: partial sums of 8 NT tokens, before that a tile's activations (2 KB NT); and the zeros that rows of the
// product without a token are read from.
constexpr uint32_t codes_wave_bytes(int nt) { return 8 * nt * kRedStride * 4; }
constexpr uint32_t codes_zero_bytes(int nt) { return nt < 4 ? nt * 1536 : 0; }
constexpr uint32_t codes_lds_bytes(int nt) { return kWaves * codes_wave_bytes(nt) + codes_zero_bytes(nt); }

// NT: rows of the first operand / 8, rounded up.  TNP: 0, or the tokens (padded to 2, 4 or 8) of the tables the activations are
// taken from; INT: integer tables, whose 14-bit activations are two rows each, a multiple of 8 and a rest of -4 .. 3.
template <int B, int GQ, bool HZ, int NT, int TNP, bool INT, bool SINGLE, typename Args, typename... Fields>
__global__ void __launch_bounds__(kWaves * 64, 3) mpgemm_codes_kernel(Fields... fields) {
    const Args a{fields...};
    using Cfg = GemvCfg<B, 1, GQ, HZ>;
    static_assert(GQ >= 64 || NT <= 2, "blocks of 32: 16 rows");
    static_assert(TNP == 0 || NT == (INT && TNP == 8 ? 2 : 1), "tables: 8 tokens");
    constexpr int kRest = TNP == 8 ? 8 : 4;  // integers: row of the rest less the token's first row
    constexpr bool kSixteen = (GQ == 128 && NT <= 2) || (GQ == 64 && NT == 1);
    constexpr int R = kSixteen ? 4 : 2;        // row groups of a tile block
    constexpr int kGroup = kRows / R;          // lanes per row group, rows and columns of a product
    constexpr int Q = kSixteen ? 1 : 2;        // 32-column blocks per lane and row group
    constexpr int V = kSixteen ? 4 : 4 * NT;   // registers of a product that hold tokens (per quantization block)
    constexpr int D = !kSixteen && NT > 1 ? 1 : 2;  // weight tile blocks in flight per wave
    typedef std::conditional_t<kSixteen, float4v_t, float16_t> acc_t;
    extern __shared__ __attribute__((aligned(128))) uint8_t lds_c[];  // see codes_lds_bytes

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);

    int wg_local;
    const GemvDesc d = desc_of_workgroup(a, wg_local);
    const int n_seg = d.n_seg, n_ktiles = d.n_ktiles;
    // Exits: surplus workgroups of the grid, and (single call) a blob packed for another shape or layout, which is
    // reported and leaves y alone (a batch is checked when its descriptor table is written).
    int n_wg = d.n_row_blocks * n_seg;
    if constexpr (SINGLE) {
        if (!header_matches(d.tiles, d.M, d.K, B, GQ, HZ ? 1 : 0)) {
            if (wg_local == 0 && tid == 0) report_header_mismatch(a.status);
            n_wg = 0;
        }
    }
    if (wg_local >= n_wg) return;
    int rb = (int)__umulhi((uint32_t)wg_local, d.seg_recip), seg = wg_local - rb * n_seg;
    if (seg >= n_seg) ++rb, seg -= n_seg;
    const int k0 = seg * d.seg_tiles;
    const int k1 = min(k0 + d.seg_tiles, n_ktiles);
    const int t0 = k0 + wave;  // the waves take the segment's tiles in turn
    const int N = d.N, K = d.K, M = d.M;
    const uint8_t* const row = d.tiles + (size_t)rb * n_ktiles * Cfg::TB;
    const int part = lane / kGroup, ri = lane % kGroup;

    // Weights: of rows kGroup r + ri, block 2 q + part (32 x 32) or part (16 x 16) and the parameters that go with it.
    constexpr int kMetaBytes = kSixteen ? Cfg::MSZ : Cfg::MPL;
    struct Codes {
        uint32_t p[R][Q][B];
        uint32_t meta[R][(kMetaBytes + 3) / 4];
    };
    auto issue_w = [&](Codes& s, bool live, int kt) {
        const rsrc_t rw = make_rsrc(row, live ? (uint32_t)(n_ktiles * Cfg::TB) : 0u);
        const int so = kt * Cfg::TB;
        const int at = ri * 16 + (part * 32 / Cfg::CH) * 1024 + (part * 32 % Cfg::CH) / 32 * B * 4;
        const int mo = B * 1024 + ri * Cfg::MPL + (kSixteen && GQ == 64 ? (part >> 1) * Cfg::MSZ : 0);
#pragma unroll
        for (int r = 0; r < R; ++r) {
#pragma unroll
            for (int q = 0; q < Q; ++q) {
                const int off = at + r * kGroup * 16 + (q * 64 / Cfg::CH) * 1024 + (q * 64 % Cfg::CH) / 32 * B * 4;
                if constexpr (B == 4) {
                    const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(rw, off, so, kStreamAux);
                    s.p[r][q][0] = v.x, s.p[r][q][1] = v.y, s.p[r][q][2] = v.z, s.p[r][q][3] = v.w;
                } else if constexpr (B == 2) {
                    const u32x2 v = __builtin_amdgcn_raw_buffer_load_b64(rw, off, so, kStreamAux);
                    s.p[r][q][0] = v.x, s.p[r][q][1] = v.y;
                } else {
                    s.p[r][q][0] = __builtin_amdgcn_raw_buffer_load_b32(rw, off, so, kStreamAux);
                }
            }
            const int off = mo + r * kGroup * Cfg::MPL;
            if constexpr (kMetaBytes == 2) {
                s.meta[r][0] = __builtin_amdgcn_raw_buffer_load_b16(rw, off, so, kStreamAux);
            } else if constexpr (kMetaBytes == 4) {
                s.meta[r][0] = __builtin_amdgcn_raw_buffer_load_b32(rw, off, so, kStreamAux);
            } else if constexpr (kMetaBytes == 8) {
                const u32x2 v = __builtin_amdgcn_raw_buffer_load_b64(rw, off, so, kStreamAux);
                s.meta[r][0] = v.x, s.meta[r][1] = v.y;
            } else {
                const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(rw, off, so, kStreamAux);
                s.meta[r][0] = v.x, s.meta[r][1] = v.y, s.meta[r][2] = v.z, s.meta[r][3] = v.w;
            }
        }
    };

    // Activations of a tile, requested one tile ahead and left in the wave's own part of the LDS as operands: 16 bytes are the
    // pairs (k, k + 16) of four columns k of one token; chunk 4 b + j holds columns 32 b + 4 j .. of all tokens, token n at
    // place n ^ (2 b + j / 2), which spreads what a store writes over all banks.
    constexpr uint32_t kChunk = 128 * NT;
    const uint32_t lr = static_cast<uint32_t>(reinterpret_cast<uintptr_t>((lds_ptr<uint8_t>)lds_c));
    const uint32_t lx = lr + (uint32_t)(wave * codes_wave_bytes(NT));
    // As such: lane 8 n + q requests, of token n (and n + 8 ..), columns 32 (q / 2) + 8 (q % 2) .. + 7 and the same + 16.  Tokens
    // beyond N lie past the end of the resource and read as zero; so do columns beyond K, which are sent there.
    const int xq = lane & 7, xn = lane >> 3, xcol = (xq >> 1) * 32 + (xq & 1) * 8;
    const uint32_t xlane = ((uint32_t)xn * (uint32_t)K + (uint32_t)xcol) * 2u;
    constexpr uint32_t kOutside = 0xFFFFFF00u;
    // Out of tables: lane 2 T + h requests, of table T (columns 4 T ..), entries 1 << h and 4 << h, which are activations h and
    // 2 + h, of all tokens; the number of a token goes to its half of a pair.
    typedef std::conditional_t<TNP == 8, u32x4, std::conditional_t<TNP == 4, u32x2, uint32_t>> entry_t;
    const int tab = lane >> 1, th = lane & 1;
    const uint32_t tlane = (uint32_t)(tab * 16 + 1 + th) * 2u * TNP;
    const uint32_t tput = lx + (uint32_t)(4 * (tab >> 3) + (tab & 3)) * kChunk + (uint32_t)(2 * (tab >> 3) + ((tab & 3) >> 1)) * 16u +
                          (uint32_t)(th * 4 + ((tab >> 2) & 1) * 2);
    struct XRegs {
        u32x4 a[NT], b[NT];
        entry_t t[2];
    };
    auto issue_x = [&](XRegs& x, bool live, int kt) {
        if constexpr (TNP == 0) {
            const rsrc_t r = make_rsrc(d.lut_t, live ? (uint32_t)N * (uint32_t)K * 2u : 0u);
            const bool inside = GQ == 128 || kt * kKTile + xcol < K;
#pragma unroll
            for (int i = 0; i < NT; ++i) {
                const uint32_t off = inside ? xlane + (uint32_t)(kt * kKTile * 2) + (uint32_t)(i * 8) * (uint32_t)K * 2u : kOutside;
                x.a[i] = __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, 0);
                x.b[i] = __builtin_amdgcn_raw_buffer_load_b128(r, off + 32, 0, 0);
            }
        } else {  // (tables beyond K hold zeros)
            constexpr uint32_t kSlice = kTableBytesPerKTile * TNP;
            const rsrc_t r = make_rsrc(d.lut_t + (size_t)kt * kSlice, live ? kSlice : 0u);
            const uint32_t far = tlane + (uint32_t)((4 << th) - (1 << th)) * 2u * TNP;
            if constexpr (TNP == 8) {
                x.t[0] = __builtin_amdgcn_raw_buffer_load_b128(r, tlane, 0, 0);
                x.t[1] = __builtin_amdgcn_raw_buffer_load_b128(r, far, 0, 0);
            } else if constexpr (TNP == 4) {
                x.t[0] = __builtin_amdgcn_raw_buffer_load_b64(r, tlane, 0, 0);
                x.t[1] = __builtin_amdgcn_raw_buffer_load_b64(r, far, 0, 0);
            } else {
                x.t[0] = __builtin_amdgcn_raw_buffer_load_b32(r, tlane, 0, 0);
                x.t[1] = __builtin_amdgcn_raw_buffer_load_b32(r, far, 0, 0);
            }
        }
    };
    auto put_x = [&](const XRegs& x) {
        wave_lds_sync();  // (the wave's reads of the previous tile come first)
        if constexpr (TNP == 0) {
            const uint32_t at = lx + (uint32_t)(2 * xq) * kChunk + (uint32_t)((xn ^ xq) * 16);
#pragma unroll
            for (int i = 0; i < NT; ++i)
#pragma unroll
                for (int j = 0; j < 2; ++j) {
                    u32x4 c;
#pragma unroll
                    for (int e = 0; e < 2; ++e) {
                        c[2 * e] = __builtin_amdgcn_perm(x.b[i][2 * j + e], x.a[i][2 * j + e], 0x05040100u);
                        c[2 * e + 1] = __builtin_amdgcn_perm(x.b[i][2 * j + e], x.a[i][2 * j + e], 0x07060302u);
                    }
                    store_lds<u32x4>(at + i * 128 + j * kChunk, c);
                }
        } else {
            uint32_t w[2][TNP / 2 ? TNP / 2 : 1];
#pragma unroll
            for (int m = 0; m < 2; ++m) __builtin_memcpy(w[m], &x.t[m], sizeof(w[m]));
            auto put = [&](int slot, int m, uint16_t v) { store_lds<uint16_t>((tput ^ (uint32_t)(slot % 8 * 16)) + slot / 8 * 128 + m * 8, v); };
#pragma unroll
            for (int n = 0; n < TNP; ++n)
#pragma unroll
                for (int m = 0; m < 2; ++m) {
                    if constexpr (INT) {
                        typedef int16_t i16x2 __attribute__((ext_vector_type(2)));
                        const i16x2 v = __builtin_bit_cast(i16x2, w[m][n / 2]), a = (v + (int16_t)4) & (int16_t)~7, b = v - a;
                        put(n, m, __builtin_bit_cast(uint16_t, (_Float16)a[n & 1]));
                        put(n + kRest, m, __builtin_bit_cast(uint16_t, (_Float16)b[n & 1]));
                    } else {
                        put(n, m, (uint16_t)(n & 1 ? w[m][n / 2] >> 16 : w[m][n / 2]));
                    }
                }
        }
        wave_lds_sync();
    };
    // Operand for the j-th four columns (and + 16) of the lanes' blocks (q): a lane is row ri of the product, slot ri of the activations, or
    // where two quantization blocks come apart slot ri % (8 NT) of block ri / (8 NT).  What is left out and rows without a token
    // are read from a piece of zeros.
    constexpr bool kApart = GQ == 32 || (GQ == 64 && kSixteen);
    const uint32_t zeros = lr + kWaves * codes_wave_bytes(NT);
    const int slot = kApart ? ri % (8 * NT) : ri;
    const bool empty = (kApart && ri / (8 * NT) != (kSixteen ? part >> 1 : part)) || slot >= 8 * NT ||
                       (TNP > 0 && (INT ? slot % kRest >= TNP || slot >= 2 * kRest : slot >= TNP));
    const uint32_t x_get = empty ? zeros : lx + (uint32_t)part * 4 * kChunk + (uint32_t)((ri >> 3) % NT) * 128;
    const uint32_t x_place = ((uint32_t)ri & 7u) ^ (uint32_t)(2 * part);
    if constexpr (NT < 4) {
        // (every wave writes all the zeros, before it reads any)
#pragma unroll
        for (int i = 0; i < (int)codes_zero_bytes(NT) / 512; ++i)
            store_lds<u32x2>(zeros + i * 512 + lane * 8, u32x2{0, 0});
    }
    auto get_x = [&](int q, int j) {
        return __builtin_bit_cast(half8_t, load_lds<u32x4>(x_get + (x_place ^ (uint32_t)(4 * q + j / 2)) * 16 + (8 * q + j) * kChunk));
    };

    auto product = [](half8_t x, half8_t c, const acc_t& s) -> acc_t {
        if constexpr (kSixteen) return __builtin_amdgcn_mfma_f32_16x16x32_f16(x, c, s, 0, 0, 0);
        else return __builtin_amdgcn_mfma_f32_32x32x16_f16(x, c, s, 0, 0, 0);
    };
    acc_t none;
#pragma unroll
    for (int v = 0; v < (kSixteen ? 4 : 16); ++v) none[v] = 0.f;
    half8_t ones;
#pragma unroll
    for (int e = 0; e < 8; ++e) ones[e] = (_Float16)1.f;
    acc_t acc[R], S;
    float y[R][V], check = 0.f;
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
        for (int v = 0; v < V; ++v) y[r][v] = 0.f;

    // acc[r][v]: row kGroup r + ri of the weights, row 4 part + v (16 x 16) or 8 (v / 4) + 4 part + v % 4 of the first operand; the
    // registers of the quantization block begin at v0, its parameters at byte mo.
    auto finish_block = [&](const Codes& st, int v0, int mo) {
        if constexpr (!INT)
#pragma unroll
            for (int v = 0; v < V; ++v) check = fmaf(S[v0 + v], 0.f, check);  // NaN from the first sum that is not finite on
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const uint32_t mw = (mo % 4) ? st.meta[r][mo / 4] >> 16 : st.meta[r][mo / 4];
            const float sc = half_bits_to_float(mw & 0xffffu) * (HZ ? 1.f : 2.f);
            const float z_off = HZ ? -kCodeOffset<B> - half_bits_to_float(mw >> 16) : -kCodeOffset<B> - 0.5f;
#pragma unroll
            for (int v = 0; v < V; ++v) {
                // sign form: (2c - 1) s = 2 s ((off + c) - (off + 1/2))
                const float t_v = fmaf(z_off, S[v0 + v], acc[r][v0 + v]);
                y[r][v] = fmaf(sc, t_v, y[r][v]);
            }
        }
    };
    auto multiply = [&](const Codes& st) {
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            uint32_t w[R][16];
#pragma unroll
            for (int r = 0; r < R; ++r) codes_to_half_pairs<B>(st.p[r][q], w[r]);
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const half8_t x = get_x(q, j);
                const bool clear = j == 0 && (q == 0 || GQ < 128);
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    const half8_t c = __builtin_bit_cast(half8_t, u32x4{w[r][4 * j], w[r][4 * j + 1], w[r][4 * j + 2], w[r][4 * j + 3]});
                    acc[r] = product(x, c, clear ? none : acc[r]);
                }
                S = product(x, ones, clear ? none : S);
            }
            if constexpr (GQ == 32) {
                finish_block(st, 0, 2 * q * Cfg::MSZ);
                finish_block(st, V, (2 * q + 1) * Cfg::MSZ);
            } else if (GQ == 64 || q == Q - 1) {
                finish_block(st, 0, GQ == 64 && !kSixteen ? q * Cfg::MSZ : 0);
            }
            if constexpr (Q == 2) __builtin_amdgcn_sched_barrier(0);  // (bounds the registers)
        }
    };

    // The first tile is requested alone behind its activations, the second (D == 2) when those are in: with both at once the
    // first products waited for the second tiles of every wave of the chip.
    Codes stg[D];
    XRegs xr;
    issue_x(xr, t0 < k1, t0);
    issue_w(stg[0], t0 < k1, t0);
    put_x(xr);
    issue_x(xr, t0 + kWaves < k1, t0 + kWaves);
    if constexpr (D == 2) issue_w(stg[1], t0 + kWaves < k1, t0 + kWaves);
    for (int base = t0; base < k1; base += D * kWaves) {
#pragma unroll
        for (int s = 0; s < D; ++s) {
            const int t = base + s * kWaves;
            if (t < k1) {
                multiply(stg[s]);
                issue_w(stg[s], t + D * kWaves < k1, t + D * kWaves);
                put_x(xr);
                issue_x(xr, t + 2 * kWaves < k1, t + 2 * kWaves);
            }
        }
    }

    // The four quarters of the segment meet in LDS, [wave][token][row].
    if constexpr (kSixteen && kApart) {  // lanes part and part + 2 have the same tokens
#pragma unroll
        for (int r = 0; r < R; ++r)
#pragma unroll
            for (int v = 0; v < V; ++v) y[r][v] += __shfl_xor(y[r][v], 32, 64);
    }
    const int tpart = kSixteen && kApart ? part & 1 : part;  // token of y[r][v]: 8 (v / 4) + 4 tpart + v % 4
    wave_lds_sync();
    if (4 * tpart < 8 * NT && (tpart == part || !kApart)) {
#pragma unroll
        for (int r = 0; r < R; ++r)
#pragma unroll
            for (int v = 0; v < V; ++v)
                store_lds<float>(lx + ((8 * (v / 4) + 4 * tpart + v % 4) * kRedStride + kGroup * r + ri) * 4, y[r][v]);
    }
    if (!INT && __builtin_expect(__builtin_amdgcn_ballot_w64(check != check) != 0, 0)) {
        // An infinity times (off + c) less an infinite sum is always NaN: the tokens with an activation that is not finite
        // in this wave's tiles, whose sums are not finite in any row, are summed again weight by weight, (c - z) s x
        // in fp32, lane = row; the others keep their sums.  One infinity in 8 tokens makes four launches of a 7B layer
        // set (uint4 g128) 235 instead of 121 us.  (A wave's LDS operations are executed in order.)
        uint32_t again = 0;
#pragma unroll
        for (int v = 0; v < V; ++v) {
            uint64_t m = __builtin_amdgcn_ballot_w64(!(fabsf(y[0][v]) < __builtin_inff()));
#pragma unroll
            for (int p = 0; p < R; ++p, m >>= kGroup)
                if (m & ((1ull << kGroup) - 1)) again |= 1u << (8 * (v / 4) + 4 * (kSixteen && kApart ? p & 1 : p) + v % 4);
        }
        again &= N < 32 ? (1u << N) - 1u : ~0u;
#pragma unroll 1
        for (; again; again &= again - 1) {
            const int n = __builtin_ctz(again);
            auto fetch = [&](int k) -> uint32_t {
                if constexpr (TNP == 0) return load_global<uint16_t>(d.lut_t + (size_t)n * K * 2, (uint32_t)k * 2u);
                else return load_global<uint16_t>(d.lut_t, (((uint32_t)(k / kLutGroup) * 16u + (1u << (k % kLutGroup))) * TNP + n) * 2u);
            };
            float sum = 0.f;
            Streams src;
            src.w = row;
            src.t = src.s = nullptr;
            src.w_bytes = (uint32_t)(n_ktiles * Cfg::TB);
            src.t_bytes = src.s_bytes = 0;
            Stage<B, 1, Cfg::MPL> next;
            issue_weights<B, 1, GQ, HZ>(next, src, t0 < k1, t0, lane);
#pragma unroll 1
            for (int t = t0; t < k1; t += kWaves) {
                const auto st = next;
                issue_weights<B, 1, GQ, HZ>(next, src, t + kWaves < k1, t + kWaves, lane);
                sum = add_products<B, GQ, HZ>(st, fetch, K, t, lane, sum);
            }
            store_lds<float>(lx + (n * kRedStride + lane) * 4, sum);
        }
    }
    __syncthreads();
    // thread -> token tid / 8, rows 8 (tid % 8) .. + 7
    const int token = tid >> 3, r8 = (tid & 7) * 8;
    const bool mine = token < N;
    float sum[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) sum[e] = 0.f;
    if (mine) {
#pragma unroll
        for (int w = 0; w < kWaves; ++w)
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const uint32_t at = lr + w * codes_wave_bytes(NT) + (token * kRedStride + r8 + e) * 4;
                sum[e] += load_lds<float>(at);
                if constexpr (INT) sum[e] += load_lds<float>(at + kRest * kRedStride * 4);
            }
        if constexpr (INT) {  // the token's power-of-two step, behind the block sums of the tables
            const float step = ldexpf(1.f, load_global<int>(d.lut_s + (size_t)n_ktiles * Cfg::GPT * TNP * 4, (uint32_t)token * 4u));
#pragma unroll
            for (int e = 0; e < 8; ++e) sum[e] *= step;
        }
    }
    finish_tokens<TNP ? TNP : kSmallTokens>(d, rb, seg, n_seg, token, r8, M, N, sum);
}

// ---------------------------------------------------------------------------------------------
// launch

template <int B, int GQ, bool HZ, int NT, int TNP, bool INT, bool SINGLE, typename Args>
static int launch_codes(const Args& a, int n_wg, hipStream_t st) {
    const dim3 grid((unsigned)n_wg, __is_same(Args, OrderedArgs) ? 1u : (unsigned)a.n_gemv);
    with_fields(a, [&](auto... f) {
        hipLaunchKernelGGL((mpgemm_codes_kernel<B, GQ, HZ, NT, TNP, INT, SINGLE, Args, decltype(f)...>), grid, dim3(kWaves * 64),
                           codes_lds_bytes(NT), st, f...);
    });
    return launch_status();
}

// 2 to 8 tokens out of tables
template <int B, bool HZ, int TNP, bool INT, bool SINGLE, typename Args>
static int launch_codes_tables_group(int group, const Args& a, int n_wg, hipStream_t st) {
    constexpr int NT = INT && TNP == 8 ? 2 : 1;
    switch (group) {
        case 32: return launch_codes<B, 32, HZ, NT, TNP, INT, SINGLE>(a, n_wg, st);
        case 64: return launch_codes<B, 64, HZ, NT, TNP, INT, SINGLE>(a, n_wg, st);
        default: return launch_codes<B, 128, HZ, NT, TNP, INT, SINGLE>(a, n_wg, st);
    }
}
template <int TNP, bool INT, bool SINGLE, typename Args>
static int launch_codes_tables(int bits, int has_zero, int group, const Args& a, int n_wg, hipStream_t st) {
    if (bits == 1) {
        return has_zero ? launch_codes_tables_group<1, true, TNP, INT, SINGLE>(group, a, n_wg, st)
                        : launch_codes_tables_group<1, false, TNP, INT, SINGLE>(group, a, n_wg, st);
    }
    if (bits == 2) return launch_codes_tables_group<2, true, TNP, INT, SINGLE>(group, a, n_wg, st);
    return launch_codes_tables_group<4, true, TNP, INT, SINGLE>(group, a, n_wg, st);
}

}  // namespace tman
