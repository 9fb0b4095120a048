// mpGEMM for a handful of tokens (up to 32): which kernel, how K is cut, and the kernel for 17 to 32 tokens with quantization
// blocks of 32 and 64.  The others multiply the codes themselves (tman_codes_kernel.h; see launch_small_cfg).
//
// With so few tokens the product is bound by the weight stream, so both kernels are organised like the decoding kernels.  The one
// here is two-level table dequantization in registers feeding the matrix cores (Sec. 4.1 "Fused LUT-based dequantization",
// Sec. 4.2): a weight is dequantized once and multiplied with all tokens in one MFMA.
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

#include "tman_codes_kernel.h"

namespace tman {

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

template <int B, int GQ, bool HZ, bool SINGLE, typename Args, typename... Fields>
__global__ void __launch_bounds__(kWaves * 64) mpgemm_small_kernel(Fields... fields) {
    const Args a{fields...};
    using Cfg = GemvCfg<B, 1, GQ, HZ>;
    constexpr int D = 2;  // weight tile blocks in flight per wave
    __shared__ __attribute__((aligned(16))) float red[kWaves][kSmallTokens][kRedStride];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);

    int wg_local;
    const GemvDesc d = desc_of_workgroup(a, wg_local);
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
                const u32x2 sw = __builtin_amdgcn_permlane32_swap(pa[e], pb[e], false, false);
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

    finish_tokens<kSmallTokens>(d, rb, seg, n_seg, token, r8, M, N, sum);
}

// ---------------------------------------------------------------------------------------------
// launch

// Which kernel: the one that multiplies codes, except for 17 to 32 tokens with blocks below 128, where its accumulators do
// not fit the registers of three waves per SIMD (uint4 g64 N = 32: 132 us against 46).  Layer sets of width 4096 / MLP
// 11008, us per launch, dequantized weights -> codes: uint4 N = 4, blocks of 128 / 64 / 32: 35 / 36 / 41 -> 22.2 / 24.5 / 26.9;
// N = 16: 39 / 40 / 45 -> 27.6 / 29.1 / 35.6; N = 32, 128: 45 -> 34.7; uint2 g64 N = 4 30 -> 19.0; 1 bit g128 N = 4 28 -> 16.3.
// Where a launch leaves most units idle, two kinds of single GEMVs are slower than the kernels before (dequantized weights; codes with
// a row per lane), which round more or are slower everywhere else: blocks of 32 with 9 to 16 tokens, 4096 x 4096, N = 16, 1 / 2
// / 4 bits 13.3 / 13.8 / 14.9 -> 14.6 / 14.3 / 14.8, 4096 x 11008 20.3 / 20.8 / 22.2 -> 21.6 / 21.3 / 22.2 (error 2.9e-4 -> 2.1e-4; a layer
// set 32 / 34.5 / 44.5 -> 28.5 / 29.5 / 34.5); 2 bits, blocks of 128, 17 tokens 12.0 -> 12.6 (N = 32 12.8 both; a layer set 27.6 -> 26.2, 38.5 -> 30.5).
// (1 bit, blocks of 128, more than 16 tokens: three registers are spilled; forms without, which make the codes in pieces, are 2
// to 4 % slower.)
template <int B, int GQ, bool HZ, bool SINGLE, typename Args>
static int launch_small_cfg(const Args& a, int N, int n_wg, hipStream_t st) {
    if (N <= 8) return launch_codes<B, GQ, HZ, 1, 0, false, SINGLE>(a, n_wg, st);
    if (N <= 16) return launch_codes<B, GQ, HZ, 2, 0, false, SINGLE>(a, n_wg, st);
    if constexpr (GQ >= 128) {
        return launch_codes<B, GQ, HZ, 4, 0, false, SINGLE>(a, n_wg, st);
    } else {
        const dim3 grid((unsigned)n_wg, __is_same(Args, OrderedArgs) ? 1u : (unsigned)a.n_gemv), block(kWaves * 64);
        with_fields(a, [&](auto... f) {
            hipLaunchKernelGGL((mpgemm_small_kernel<B, GQ, HZ, SINGLE, Args, decltype(f)...>), grid, block, 0, st, f...);
        });
        return launch_status();
    }
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
// numbering, largest workgroups first, pays up to four for it too, and never costs (measured with a row of W per lane): eight launches of a layer set of width
// 4096 and MLP width 14336 (896 workgroups), plain grid -> numbered, uint4 g128 N = 8 309 -> 275 us, g64 N = 16 358 -> 318,
// uint2 g64 N = 4 267 -> 236, 1 bit 233 -> 202; 992 workgroups 364 -> 354; 832 equal ones 284 / 285.
int ordered_workgroups_small(int count, const Layout* L, int n_units) {
    if (count > 8) return 0;
    std::vector<GemvPlan> plans(count);
    for (int g = 0; g < count; ++g) plans[g] = plan_small(L[g]);
    return ordered_workgroups_of(count, L, plans.data(), n_units, kCodesResident);
}
bool order_workgroups_small(int count, const Layout* L, int n_units, std::vector<uint16_t>* order) {
    if (count > 8) return false;
    std::vector<GemvPlan> plans(count);
    for (int g = 0; g < count; ++g) plans[g] = plan_small(L[g]);
    return order_workgroups_of(count, L, plans.data(), n_units, kCodesResident, order);
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
