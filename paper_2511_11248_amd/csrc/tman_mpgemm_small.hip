// mpGEMM for a handful of tokens (2 .. 32): two-level table dequantization in registers feeding the matrix
// cores (Sec. 4.1 "Fused LUT-based dequantization", Sec. 4.2), organised like the decoding kernel because with
// so few tokens the product is bound by the weight stream, not by the matrix cores.
//
// Why not the lookup kernel for 4 or 8 tokens: a lookup then returns 8 or 16 bytes per lane and the vector
// lookups are bound by LDS bandwidth (16 bytes per lane and lookup), three to four times the time the weight
// stream needs.  Dequantizing a weight once and multiplying it with all tokens in one MFMA costs the same
// vector work for 2 tokens as for 32.
//
// Mapping.  The weights stay in the bit-serial layout the decoding kernel streams (lane = row of a 64-row
// tile block, 16-byte chunks of bit-plane words, group scales and zeros behind them): a wave requests whole
// tile blocks exactly as mpgemv_kernel does.  Per 32-column step it dequantizes the lane's 32 weights into
// four 16-byte pieces of 8 fp16 (level 1: bit-field transposition, level 2: the block's affine map as one
// FMA on a code placed in an fp16 mantissa).  v_mfma_f32_32x32x16_f16 wants, per operand, lane l to hold row
// l % 32 and the 8 columns of half l / 32; a lane holds ONE row and all columns, so two pieces (a, b) are
// exchanged between the wave's halves with v_permlane32_swap: one result has rows 0..31 with columns a | b,
// the other rows 32..63 with columns a | b -- two ready operands from four swaps.  The activations of the same
// 16 columns come straight from memory (L2): lane l reads 16 bytes of token l % 32 at column half l / 32;
// tokens beyond N and columns beyond K lie outside the buffer resource and read as zero.
// Accumulators: 64 rows x 32 tokens per wave in fp32.
//
// Scheduling is that of the decoding kernels: a workgroup of four waves owns a row block and a K segment, the
// four quarters meet in LDS, segments of a long K meet through the workspace (tickets, partial sums added in
// segment order, so results do not depend on timing).
#include <vector>

#include "tman_dequant_device.h"
#include "tman_gemv_device.h"

namespace tman {

typedef float float16_t __attribute__((ext_vector_type(16)));
typedef uint32_t u32x2v __attribute__((ext_vector_type(2)));

constexpr int kSmallTokens = TMAN_MAX_SMALL_TOKENS;  // 32: the token extent of one MFMA
constexpr int kRedStride = kRows + 4;                  // floats per token in the LDS reduction buffer (bank spread)

GemvPlan plan_small(const Layout& L) {
    // a dequantized tile takes about as long as a looked-up tile of one token: the same segment lengths
    GemvPlan p = plan_segments(L, 1, current_tiling().small_seg_tiles);
    p.np = kSmallTokens;
    p.partial_bytes = p.n_seg > 1 ? (size_t)L.n_row_blocks * p.n_seg * kSmallTokens * kRows * sizeof(float) : 0;
    return p;
}

void fill_desc_small(GemvDesc& d, const Layout& L, const void* packed, const void* x, int N, void* y, void* workspace) {
    fill_desc_plan(d, L, plan_small(L), packed, x, N, y, workspace);
    d.lut_s = nullptr;
}

// Output of one row block: thread -> (token, rows r8 .. r8 + 7 of the block) with the sums of the workgroup's K segment.
__device__ __forceinline__ void finish_tokens(const GemvDesc& d, int rb, int seg, int n_seg, int token, int r8, int M, int N,
                                              const float (&sum)[8]) {
    __shared__ int last_flag;
    const int m0 = rb * kRows + r8;
    _Float16* out = static_cast<_Float16*>(d.y);
    auto store_rows = [&](const float (&v)[8]) {
        if (token >= N) return;
        _Float16* dst = out + (size_t)token * M + m0;
        if (m0 + 8 <= M && (M % 8) == 0) {
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
    float* base_p = d.partial + (size_t)rb * n_seg * kSmallTokens * kRows;
    float* mine = base_p + (size_t)seg * kSmallTokens * kRows + token * kRows + r8;
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
            const float* src_p = base_p + (size_t)p * kSmallTokens * kRows + token * kRows + r8;
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

template <int B, int GQ, bool HZ, bool SINGLE, typename Args>
__global__ void __launch_bounds__(kWaves * 64) mpgemm_small_kernel(Args a) {
    using Cfg = GemvCfg<B, 1, GQ, HZ>;
    constexpr int D = 2;  // weight tile blocks in flight per wave
    __shared__ __attribute__((aligned(16))) float red[kWaves][kSmallTokens][kRedStride];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);

    int g, wg_local;
    workgroup_of<SINGLE>(a, g, wg_local);
    const GemvDesc& d = desc_of<SINGLE>(a, g);
    const int n_seg = uniform(d.n_seg), n_ktiles = uniform(d.n_ktiles);
    // Exits: surplus workgroups of the grid, and (single call) a blob packed for another shape or layout, which
    // is reported and leaves y alone (a batch is checked when its descriptor table is written).
    int n_wg = uniform(d.n_row_blocks) * n_seg;
    if constexpr (SINGLE) {
        if (!header_matches(uniform(d.tiles), uniform(d.M), uniform(d.K), B, GQ, HZ ? 1 : 0)) {
            if (wg_local == 0 && tid == 0) report_header_mismatch(a.status);
            n_wg = 0;
        }
    }
    if (wg_local >= n_wg) return;
    const int rb = uniform(wg_local / n_seg), seg = uniform(wg_local % n_seg);
    const int seg_tiles = uniform(d.seg_tiles);
    const int k0 = seg * seg_tiles;
    const int k1 = min(k0 + seg_tiles, n_ktiles);
    const int per_wave = (k1 - k0 + kWaves - 1) / kWaves;
    const int t0 = min(k0 + wave * per_wave, k1);  // this wave's K tiles [t0, t1)
    const int t1 = min(t0 + per_wave, k1);
    const int N = uniform(d.N), K = uniform(d.K), M = uniform(d.M);
    Streams src;
    src.w = uniform(d.tiles) + (size_t)rb * n_ktiles * Cfg::TB;
    src.t = src.s = nullptr;
    src.w_bytes = (uint32_t)(n_ktiles * Cfg::TB);
    src.t_bytes = src.s_bytes = 0;

    // Activations: lane l reads token l % 32, column half l / 32 of each 16-column step.  A token beyond N lies
    // past the end of the resource (N * K * 2 bytes); a column beyond K is sent there explicitly, because inside
    // the buffer it would be the next token's data.
    const rsrc_t rx = make_rsrc(uniform(d.lut_t), (uint32_t)N * (uint32_t)K * 2u);
    const uint32_t xlane = (uint32_t)(lane & 31) * (uint32_t)K * 2u + (uint32_t)(lane >> 5) * 16u;
    const int kcol_lane = (lane >> 5) * 8;
    constexpr uint32_t kOutside = 0xFFFFFFF0u;
    // The activations of a tile are requested in two halves of 64 columns, each half a tile ahead of its use.
    struct XHalf {
        u32x4 v[4];  // step s (16 columns) of the half
    };
    auto issue_x = [&](XHalf& xh, bool live, int kt, int half) {
        const rsrc_t r = live ? rx : make_rsrc(uniform(d.lut_t), 0u);
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            const int c0 = kt * kKTile + half * 64 + s * 16;
            const uint32_t off = c0 + kcol_lane < K ? xlane + (uint32_t)c0 * 2u : kOutside;
            xh.v[s] = __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, 0);
        }
    };

    float16_t acc[2];
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[h][v] = 0.f;

    // One 32-column step: the lane's 32 weights of block kb32 of the tile, against steps 2 (kb32 % 2) and + 1
    // of the activation half.
    auto step32 = [&](const Stage<B, 1, Cfg::MPL>& cur, const XHalf& xh, int kb32) {
        WRegs<B> r;
        const int v = (kb32 * 32) / Cfg::CH, ksub = ((kb32 * 32) % Cfg::CH) / 32;
#pragma unroll
        for (int i = 0; i < B; ++i) r.plane[i] = word_of(cur.c[v], ksub * B + i);
        const int mo = ((kb32 * 32) / GQ) * Cfg::MSZ;
        const uint32_t mw = cur.meta[mo / 4];
        r.meta = HZ ? mw : ((mo % 4) ? (mw >> 16) : (mw & 0xffffu));
        Dequant<B, HZ> dq;
        dq.start(r);
        dq.insert();
#pragma unroll
        for (int pair = 0; pair < 2; ++pair) {
            const u32x4 pa = dq.piece(2 * pair), pb = dq.piece(2 * pair + 1);
            u32x4 lo, hi;  // operands of rows 0..31 and rows 32..63: columns pa | pb
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const u32x2v sw = __builtin_amdgcn_permlane32_swap(pa[e], pb[e], false, false);
                lo[e] = sw.x;
                hi[e] = sw.y;
            }
            const half8_t xo = __builtin_bit_cast(half8_t, xh.v[(kb32 & 1) * 2 + pair]);
            acc[0] = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(half8_t, lo), xo, acc[0], 0, 0, 0);
            acc[1] = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(half8_t, hi), xo, acc[1], 0, 0, 0);
        }
    };

    Stage<B, 1, Cfg::MPL> st[D] = {};
    XHalf xa, xb;
#pragma unroll
    for (int s = 0; s < D; ++s) issue_weights<B, 1, GQ, HZ>(st[s], src, t0 + s < t1, t0 + s, lane);
    issue_x(xa, t0 < t1, t0, 0);
    issue_x(xb, t0 < t1, t0, 1);
    for (int base = t0; base < t1; base += D) {
#pragma unroll
        for (int s = 0; s < D; ++s) {
            const int t = base + s;
            if (t < t1) {
                step32(st[s], xa, 0);
                step32(st[s], xa, 1);
                issue_x(xa, t + 1 < t1, t + 1, 0);
                step32(st[s], xb, 2);
                step32(st[s], xb, 3);
                issue_x(xb, t + 1 < t1, t + 1, 1);
                issue_weights<B, 1, GQ, HZ>(st[s], src, t + D < t1, t + D, lane);
            }
        }
    }

    // The four quarters of the segment meet in LDS.  acc[h][v] is row 32 h + 8 (v / 4) + 4 (lane / 32) + v % 4 of
    // the row block for token lane % 32: four consecutive rows per group of four registers.
    {
        const int token = lane & 31, hh = lane >> 5;
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                float* dst = &red[wave][token][32 * h + 8 * q + 4 * hh];
#pragma unroll
                for (int e = 0; e < 4; ++e) dst[e] = acc[h][4 * q + e];
            }
    }
    __syncthreads();
    // thread -> token tid / 8, rows 8 (tid % 8) .. + 7
    const int token = tid >> 3, r8 = (tid & 7) * 8;
    float sum[8];
#pragma unroll
    for (int e = 0; e < 8; ++e)
        sum[e] = ((red[0][token][r8 + e] + red[1][token][r8 + e]) + red[2][token][r8 + e]) + red[3][token][r8 + e];

    finish_tokens(d, rb, seg, n_seg, token, r8, M, N, sum);
}

// ---------------------------------------------------------------------------------------------
// The same product with the scales and zeros taken out of the weights.  The kernel above spends two thirds of its
// vector instructions on the affine map of every weight (82 per 32 weights, 385 per tile block with the rest).  Here the
// matrix cores multiply the codes themselves, as exact fp16 numbers off + c (the code inserted into the mantissa of a
// power of two), and a quantization block's scale and zero are applied to its sums:
//   y[n][m] += s[m] * (acc[n][m] - (off + z[m]) * S[n]),   acc = sum (off + c) x,  S = sum x over the block.
// The offset costs 1 to 4 bits of the fp32 accumulator; weights are no longer rounded to fp16, so the sums are closer to
// the exact ones than before (rms 2.1e-4 of rms(y), the fp16 result alone, from 2.9e-4).
//
// The activations are the FIRST operand and the weights the second, so that a lane's accumulators belong to ONE row of W
// (lane % 32) and the registers to tokens: a block's scale and zero are one value per lane and 32-row half, and with 8
// tokens only 4 of 16 registers hold tokens that exist.  That is 8 NT fused multiply-adds per half and block (NT = tokens
// / 8 rounded up).  Level 1 leaves weights k and k + 16 of a 32-column step in the halves of one register; the
// activations are paired to match (8 v_perm per step).  S comes from a third product, of the activations with ones, in the
// accumulators' own layout (summing it ahead, once per workgroup, put 3 to 6 us in front of every workgroup).
// About 263 vector instructions per tile block in the loop for uint4 g128 and 8 tokens.  What bounds it now: registers for three waves per
// SIMD (two tiles in flight: 5 % better than one; with two waves per SIMD it loses 15 %), so latency, then the
// vector pipe; 107.5 MB (7B uint4 g128, N = 8) in 28.7 - 29.5 us = 3.7 TB/s, from 35.0 (bench run: 31.1 - 31.8, from 39.3).
// The offset: 64 for 4 bits (a nibble at mantissa bits 4..7 needs three shifts per code word; at bits 6..9, as 16 + c, it
// would need four), 4 for 2 bits (bits 8..9), 2 for 1 bit (bit 9): small against the codes, because what the offset
// adds to the sums is lost to their precision.
template <int B>
constexpr float kCodeOffset = B == 4 ? 64.f : B == 2 ? 4.f : 2.f;
template <int B>
__device__ __forceinline__ void codes_to_half_pairs(const uint32_t (&p)[B], uint32_t (&w)[16]) {
    constexpr uint32_t kMask = B == 4 ? 0x00F000F0u : B == 2 ? 0x03000300u : 0x02000200u;
    constexpr uint32_t kBase = B == 4 ? 0x54005400u : B == 2 ? 0x44004400u : 0x40004000u;
    auto place = [](uint32_t v, int from, int to) { return from < to ? v << (to - from) : v >> (from - to); };
    if constexpr (B == 1) {
#pragma unroll
        for (int k = 0; k < 16; ++k) w[k] = and_or(place(p[0], k, 9), kMask, kBase);
    } else {
        uint32_t c[4];  // word o, field f: weight 4f + o; fields f and f + 4 are 16 bits apart
        planes_to_codes<B>(p, c);
#pragma unroll
        for (int f = 0; f < 4; ++f)
#pragma unroll
            for (int o = 0; o < 4; ++o) w[4 * f + o] = and_or(place(c[o], 4 * f, B == 4 ? 4 : 8), kMask, kBase);
    }
}

// The lane's row of tile block t (in `st`) times the activations of one token (row x), weight by weight.
template <int B, int GQ, bool HZ>
__device__ __forceinline__ float add_products(const Stage<B, 1, GemvCfg<B, 1, GQ, HZ>::MPL>& st, const uint8_t* x, int K, int t,
                                              int lane, float sum) {
    using Cfg = GemvCfg<B, 1, GQ, HZ>;
    uint32_t xv[2];  // lane l holds columns l and 64 + l of the tile
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int k = t * kKTile + i * 64 + lane;
        xv[i] = k < K ? load_global<uint16_t>(x, (uint32_t)k * 2u) : 0u;
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

template <int B, int GQ, bool HZ, int NT, bool SINGLE, typename Args>
__global__ void __launch_bounds__(kWaves * 64, 3) mpgemm_codes_kernel(Args a) {
    using Cfg = GemvCfg<B, 1, GQ, HZ>;
    constexpr int kTok = 8 * NT;
    constexpr int D = 2;  // weight tile blocks in flight per wave
    extern __shared__ __attribute__((aligned(16))) uint8_t lds_c[];  // partial sums of the waves

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);

    int g, wg_local;
    workgroup_of<SINGLE>(a, g, wg_local);
    const GemvDesc d = desc_value<SINGLE>(a, g);
    const int n_seg = d.n_seg, n_ktiles = d.n_ktiles;
    // Exits as in mpgemm_small_kernel.
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
    Streams src;
    src.w = d.tiles + (size_t)rb * n_ktiles * Cfg::TB;
    src.t = src.s = nullptr;
    src.w_bytes = (uint32_t)(n_ktiles * Cfg::TB);
    src.t_bytes = src.s_bytes = 0;

    // Activations: lane l reads token l % 32, 8 columns of half l / 32 of each 16-column step.  Tokens beyond N lie past
    // the end of the resource and read as zero.  Columns beyond K may read the next token's activations: they belong
    // to quantization blocks beyond K, whose sums are dropped.
    const rsrc_t rx = make_rsrc(d.lut_t, (uint32_t)N * (uint32_t)K * 2u);
    const uint32_t xlane = (uint32_t)(lane & 31) * (uint32_t)K * 2u + (uint32_t)(lane >> 5) * 16u;
    struct XHalf {
        u32x4 v[4];  // 16-column steps of half a tile
    };
    auto issue_x = [&](XHalf& xh, bool live, int kt, int half) {
        const rsrc_t r = live ? rx : make_rsrc(d.lut_t, 0u);
        const uint32_t off = xlane + (uint32_t)(kt * kKTile * 2);
#pragma unroll
        for (int s = 0; s < 4; ++s) xh.v[s] = __builtin_amdgcn_raw_buffer_load_b128(r, off + half * 128 + s * 32, 0, 0);
    };

    Stage<B, 1, Cfg::MPL> stg[D] = {};
    XHalf xa, xb;
#pragma unroll
    for (int s = 0; s < D; ++s) issue_weights<B, 1, GQ, HZ>(stg[s], src, t0 + s * kWaves < k1, t0 + s * kWaves, lane);
    issue_x(xa, t0 < k1, t0, 0);
    issue_x(xb, t0 < k1, t0, 1);

    const uint32_t lr = static_cast<uint32_t>(reinterpret_cast<uintptr_t>((lds_ptr<uint8_t>)lds_c));
    float16_t zero16;
#pragma unroll
    for (int v = 0; v < 16; ++v) zero16[v] = 0.f;
    half8_t ones;
#pragma unroll
    for (int e = 0; e < 8; ++e) ones[e] = (_Float16)1.f;
    float16_t acc[2], S;
    float y[2][4 * NT], check = 0.f;
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int v = 0; v < 4 * NT; ++v) y[h][v] = 0.f;

    // one 32-column step of the tile; `first`: the first step of its quantization block
    auto step32 = [&](const Stage<B, 1, Cfg::MPL>& st, const XHalf& xh, int kb32, bool first) {
        uint32_t p[B], w[16], x[8];
        const int v = (kb32 * 32) / Cfg::CH, ksub = ((kb32 * 32) % Cfg::CH) / 32;
#pragma unroll
        for (int i = 0; i < B; ++i) p[i] = word_of(st.c[v], ksub * B + i);
        codes_to_half_pairs<B>(p, w);
        const u32x4 va = xh.v[(kb32 & 1) * 2], vb = xh.v[(kb32 & 1) * 2 + 1];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            x[2 * e] = __builtin_amdgcn_perm(vb[e], va[e], 0x05040100u);
            x[2 * e + 1] = __builtin_amdgcn_perm(vb[e], va[e], 0x07060302u);
        }
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            // lanes 0..31 take columns 4j .. 4j + 3 (and + 16), lanes 32..63 columns 8 + 4j ..
            u32x4 lo, hi;  // rows 0..31 and rows 32..63
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const u32x2v sw = __builtin_amdgcn_permlane32_swap(w[4 * j + e], w[8 + 4 * j + e], false, false);
                lo[e] = sw.x;
                hi[e] = sw.y;
            }
            const half8_t xo = __builtin_bit_cast(half8_t, u32x4{x[4 * j], x[4 * j + 1], x[4 * j + 2], x[4 * j + 3]});
            const bool clear = first && j == 0;
            acc[0] = __builtin_amdgcn_mfma_f32_32x32x16_f16(xo, __builtin_bit_cast(half8_t, lo), clear ? zero16 : acc[0], 0, 0, 0);
            acc[1] = __builtin_amdgcn_mfma_f32_32x32x16_f16(xo, __builtin_bit_cast(half8_t, hi), clear ? zero16 : acc[1], 0, 0, 0);
            S = __builtin_amdgcn_mfma_f32_32x32x16_f16(xo, ones, clear ? zero16 : S, 0, 0, 0);
        }
    };
    // acc[h][v]: row 32 h + lane % 32, token 8 (v / 4) + 4 (lane / 32) + v % 4
    auto finish_block = [&](const Stage<B, 1, Cfg::MPL>& st, int t, int gi) {
        if (t * kKTile + gi * GQ >= K) return;  // (uniform)
        const int mo = gi * Cfg::MSZ;
        const uint32_t mw = (mo % 4) ? st.meta[mo / 4] >> 16 : st.meta[mo / 4];
        const u32x2v m2 = __builtin_amdgcn_permlane32_swap(mw, mw, false, false);
        const uint32_t m_of[2] = {m2.x, m2.y};
#pragma unroll
        for (int v = 0; v < 4 * NT; ++v) check = fmaf(S[v], 0.f, check);  // NaN from the first sum that is not finite on
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const float sc = half_bits_to_float(m_of[h] & 0xffffu) * (HZ ? 1.f : 2.f);
            const float z_off = HZ ? -kCodeOffset<B> - half_bits_to_float(m_of[h] >> 16) : -kCodeOffset<B> - 0.5f;
#pragma unroll
            for (int v = 0; v < 4 * NT; ++v) {
                // sign form: (2c - 1) s = 2 s ((off + c) - (off + 1/2))
                const float t_v = fmaf(z_off, S[v], acc[h][v]);
                y[h][v] = fmaf(sc, t_v, y[h][v]);
            }
        }
    };

    for (int base = t0; base < k1; base += D * kWaves) {
#pragma unroll
        for (int s = 0; s < D; ++s) {
            const int t = base + s * kWaves;
            if (t < k1) {
#pragma unroll
                for (int b = 0; b < 4; ++b) {
                    step32(stg[s], b < 2 ? xa : xb, b, (b * 32) % GQ == 0);
                    if ((b * 32 + 32) % GQ == 0) finish_block(stg[s], t, b * 32 / GQ);
                    if (b == 1) issue_x(xa, t + kWaves < k1, t + kWaves, 0);
                }
                issue_x(xb, t + kWaves < k1, t + kWaves, 1);
                issue_weights<B, 1, GQ, HZ>(stg[s], src, t + D * kWaves < k1, t + D * kWaves, lane);
            }
        }
    }

    // the four quarters of the segment meet in LDS, [wave][token][row]
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int v = 0; v < 4 * NT; ++v)
            store_lds<float>(lr + ((wave * kTok + 8 * (v / 4) + 4 * (lane >> 5) + v % 4) * kRedStride + 32 * h + (lane & 31)) * 4,
                             y[h][v]);
    if (__builtin_expect(__builtin_amdgcn_ballot_w64(check != check) != 0, 0)) {
        // An infinity times (off + c) less an infinite sum is always NaN: the tokens with an activation that is not finite
        // in this wave's tiles, whose sums are not finite in any row, are summed again weight by weight, (c - z) s x
        // in fp32, lane = row; the others keep their sums.  One infinity in 8 tokens makes four launches of a 7B layer
        // set (uint4 g128) 235 instead of 121 us (5.8 ms when every token was summed again, a bit and a column at a
        // time; 146 in the kernel above, which needs no second sum).  (A wave's LDS stores are executed in order.)
        uint32_t again = 0;
#pragma unroll
        for (int v = 0; v < 4 * NT; ++v) {
            const uint64_t m = __builtin_amdgcn_ballot_w64(!(fabsf(y[0][v]) < __builtin_inff()));
            again |= (m & 0xffffffffu ? 1u << (8 * (v / 4) + v % 4) : 0u) | (m >> 32 ? 1u << (8 * (v / 4) + 4 + v % 4) : 0u);
        }
#pragma unroll 1
        for (; again; again &= again - 1) {
            const int n = __builtin_ctz(again);
            const uint8_t* const x = d.lut_t + (size_t)n * K * 2;
            float sum = 0.f;
            issue_weights<B, 1, GQ, HZ>(stg[0], src, t0 < k1, t0, lane);
#pragma unroll 1
            for (int t = t0; t < k1; t += kWaves) {
                const auto st = stg[0];
                issue_weights<B, 1, GQ, HZ>(stg[0], src, t + kWaves < k1, t + kWaves, lane);
                sum = add_products<B, GQ, HZ>(st, x, K, t, lane, sum);
            }
            store_lds<float>(lr + ((wave * kTok + n) * kRedStride + lane) * 4, sum);
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
            for (int e = 0; e < 8; ++e) sum[e] += load_lds<float>(lr + ((w * kTok + token) * kRedStride + r8 + e) * 4);
    }
    finish_tokens(d, rb, seg, n_seg, token, r8, M, N, sum);
}

// ---------------------------------------------------------------------------------------------
// launch

// Which kernel: the one that multiplies codes where what it does per quantization block (16 NT multiply-adds) is less than
// the affine map of the weights costs: every group for up to 8 tokens, blocks of 64 or 128 for up to 16, blocks of 128
// for up to 32.  Measured on layer sets of width 4096 / MLP 11008, us per launch before -> now: uint4 N = 4, blocks of
// 128 / 64 / 32: 35.4 -> 27.9, 36.0 -> 29.1, 41.3 -> 31.1; N = 16, 128 / 64: 39.0 -> 33.1, 40.1 -> 35.7; N = 32, 128: 45.3 ->
// 43.2; uint2 g64 N = 4: 30.4 -> 25.0; 1 bit g128 N = 4: 28.3 -> 21.5 (width 2048: 2 to 15 % less).  Blocks of 32 with 16
// tokens and blocks of 64 with 32 would do as much work in both kernels.
template <int NT>
constexpr int kCodesLdsBytes = kWaves * 8 * NT * kRedStride * 4;

template <int B, int GQ, bool HZ, bool SINGLE, typename Args>
static int launch_small_cfg(const Args& a, int N, int n_wg, hipStream_t st) {
    const dim3 grid((unsigned)n_wg, __is_same(Args, OrderedArgs) ? 1u : (unsigned)a.n_gemv), block(kWaves * 64);
    if (N <= 8) {
        hipLaunchKernelGGL((mpgemm_codes_kernel<B, GQ, HZ, 1, SINGLE, Args>), grid, block, kCodesLdsBytes<1>, st, a);
        return launch_status();
    } else if (N <= 16) {
        if constexpr (GQ >= 64) {
            hipLaunchKernelGGL((mpgemm_codes_kernel<B, GQ, HZ, 2, SINGLE, Args>), grid, block, kCodesLdsBytes<2>, st, a);
            return launch_status();
        }
    } else if constexpr (GQ >= 128) {
        hipLaunchKernelGGL((mpgemm_codes_kernel<B, GQ, HZ, 4, SINGLE, Args>), grid, block, kCodesLdsBytes<4>, st, a);
        return launch_status();
    }
    hipLaunchKernelGGL((mpgemm_small_kernel<B, GQ, HZ, SINGLE, Args>), grid, block, 0, st, a);
    return launch_status();
}

template <int B, bool HZ, bool SINGLE, typename Args>
static int launch_small_group(int group, const Args& a, int N, int n_wg, hipStream_t st) {
    switch (group) {
        case 32: return launch_small_cfg<B, 32, HZ, SINGLE>(a, N, n_wg, st);
        case 64: return launch_small_cfg<B, 64, HZ, SINGLE>(a, N, n_wg, st);
        default: return launch_small_cfg<B, 128, HZ, SINGLE>(a, N, n_wg, st);
    }
}

template <bool SINGLE, typename Args>
static int launch_small_format(int bits, int has_zero, int group, const Args& a, int N, int n_wg,
                               hipStream_t st) {
    if (bits == 1) {
        return has_zero ? launch_small_group<1, true, SINGLE>(group, a, N, n_wg, st)
                        : launch_small_group<1, false, SINGLE>(group, a, N, n_wg, st);
    }
    if (bits == 2) return launch_small_group<2, true, SINGLE>(group, a, N, n_wg, st);
    return launch_small_group<4, true, SINGLE>(group, a, N, n_wg, st);
}

int launch_mpgemm_small(const Layout& L, const void* packed, const void* x, int N, void* y, void* workspace,
                        hipStream_t st) {
    KernelArgs<true> a;
    fill_desc_small(a.single, L, packed, x, N, y, workspace);
    a.n_gemv = 1;
    a.status = device_status_word();
    if (!a.status) return TMAN_ERR_LAUNCH;
    return launch_small_format<true>(L.bits, L.has_zero, L.group, a, N, plan_small(L).n_workgroups, st);
}

int launch_mpgemm_small_batch(int bits, int group, int has_zero, int N, const GemvDesc* descs_dev, int n_gemv,
                              int max_workgroups, hipStream_t st) {
    KernelArgs<false> a;
    a.descs = descs_dev;
    a.n_gemv = n_gemv;
    a.row_blocks = 1;
    return launch_small_format<false>(bits, has_zero, group, a, N, max_workgroups, st);
}

// The numbered launch of a batch (see order_workgroups_of), up to four workgroups per compute unit: what is resident of
// mpgemm_small_kernel, whose reduction buffer takes 34.8 KB of LDS.  Of mpgemm_codes_kernel three are (registers), but
// numbering, largest workgroups first, pays up to four for it too, and never costs: eight launches of a layer set of width
// 4096 and MLP width 14336 (896 workgroups), plain grid -> numbered, uint4 g128 N = 8 309 -> 275 us, g64 N = 16 358 -> 318,
// uint2 g64 N = 4 267 -> 236, 1 bit 233 -> 202; 992 workgroups 364 -> 354; 832 equal ones 284 / 285.
constexpr int kSmallResident = (int)(160u * 1024u / (sizeof(float) * kWaves * kSmallTokens * kRedStride + 64));
int ordered_workgroups_small(int count, const Layout* L, int n_units) {
    if (count > 8) return 0;
    std::vector<GemvPlan> plans(count);
    for (int g = 0; g < count; ++g) plans[g] = plan_small(L[g]);
    return ordered_workgroups_of(count, L, plans.data(), n_units, kSmallResident);
}
bool order_workgroups_small(int count, const Layout* L, int n_units, std::vector<uint16_t>* order) {
    if (count > 8) return false;
    std::vector<GemvPlan> plans(count);
    for (int g = 0; g < count; ++g) plans[g] = plan_small(L[g]);
    return order_workgroups_of(count, L, plans.data(), n_units, kSmallResident, order);
}
int launch_mpgemm_small_ordered(int bits, int group, int has_zero, int N, const GemvDesc* descs_dev, int n_gemv,
                                const uint16_t* order_dev, int n_wg, hipStream_t st) {
    OrderedArgs a;
    a.descs = descs_dev;
    a.order = order_dev;
    a.n_gemv = n_gemv;
    return launch_small_format<false>(bits, has_zero, group, a, N, n_wg, st);
}

}  // namespace tman
