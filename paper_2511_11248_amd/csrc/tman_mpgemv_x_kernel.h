// The one-token decoding kernel on the 4-bit dot product unit or (on_matrix_cores) the matrix cores, as a template over the
// weight format and the source of the activations; what it does and why is said in tman_mpgemv_x.hip.
#pragma once
#include "tman_codes_kernel.h"
#include "tman_digits_device.h"
#include "tman_fp4_device.h"
#include "tman_mpgemv_kernel.h"

namespace tman {

// Which formats multiply on the matrix cores (tman_fp4_device.h) instead of the dot product unit: 1 and 2 bits, whose codes are 4-bit
// numbers as they are, with fp16 activations.  4 bits would be two such products beside a longer transposition, and their
// launches wait for memory already (without any computing 20.0 us against 19.2); integer activations
// stay integers.
constexpr bool on_matrix_cores(int bits, TokenSource src) { return bits <= 2 && src != TokenSource::kTablesI16; }

// LDS of a workgroup whose segment has `seg_tiles` tiles: digits and sums or quantization blocks (`gpt` per tile) of the
// activations, then the partial sums (two sets where a workgroup takes several row blocks) and a word per wave: at most 19,488 bytes
constexpr unsigned x_lds_bytes(int seg_tiles, int gpt, bool matrix, int sets = 1) {
    const int tile = matrix ? kFp4BytesPerKTile + kFp4SumBytes : kDigitBytesPerKTile + gpt * kDigitMetaBytes;
    return (unsigned)(seg_tiles * tile + sets * kWaves * kRows * 4 + kWaves * 4 + (matrix ? kFp4Zeros : 0));
}
// Workgroups of a large 1-bit batch take several row blocks with one set of digits (batch_row_blocks).
template <int B, typename Args>
constexpr bool several_row_blocks = B == 1 && std::is_same_v<Args, KernelArgs<false>>;

// The 8 activations of a lane: numbers 4f .. 4f + 3 (a) and 16 + 4f .. (b) of its 32-column block.
struct LaneActs {
    u32x2 a, b;
};

// The four activations out of one table.
__device__ __forceinline__ void load_table(rsrc_t rt, int off, u32x2& x) {
    const u32x4 lo = __builtin_amdgcn_raw_buffer_load_b128(rt, off, 0, 0);
    const uint32_t e8 = __builtin_amdgcn_raw_buffer_load_b32(rt, off + 16, 0, 0);
    const uint32_t e01 = lo.x, e23 = lo.y, e45 = lo.z;
    x = u32x2{__builtin_amdgcn_perm(e23, e01, 0x05040302u), __builtin_amdgcn_perm(e8, e45, 0x05040100u)};
}

template <int B, int GQ, bool HZ, TokenSource SRC, bool SINGLE, typename Args, typename... Fields>
__global__ void __launch_bounds__(kWaves * 64, 4) mpgemv_x_kernel(Fields... fields) {
    const Args a{fields...};
    using Cfg = GemvCfg<B, 1, GQ, HZ>;
    constexpr bool kSeveral = several_row_blocks<B, Args>;
    constexpr bool kMatrix = on_matrix_cores(B, SRC);
    extern __shared__ __attribute__((aligned(1024))) uint8_t lds_x[];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);

    int wg_local;
    const GemvDesc d = desc_of_workgroup(a, wg_local);
    const int n_seg = d.n_seg, n_ktiles = d.n_ktiles;
    // Exits: surplus workgroups of the grid, and (single call) a blob packed for another shape or layout, which is
    // reported and leaves y alone; a batch is checked when its descriptor table is written, which empties the
    // descriptor of such a GEMV.  One exit for both, before any other memory request.
    int n_wg = d.n_row_blocks * n_seg;
    if constexpr (kSeveral) n_wg = (d.n_row_blocks + a.row_blocks - 1) / a.row_blocks * n_seg;
    if constexpr (SINGLE) {
        if (!header_matches(d.tiles, d.M, d.K, B, GQ, HZ ? 1 : 0)) {
            if (wg_local == 0 && tid == 0) report_header_mismatch(a.status);
            n_wg = 0;
        }
    }
    if (wg_local >= n_wg) return;
    // row block and segment: quotient by the reciprocal floor((2^32 - 1) / n_seg), which falls short by at most one
    int rb = (int)__umulhi((uint32_t)wg_local, (uint32_t)d.seg_recip), seg = wg_local - rb * n_seg;
    if (seg >= n_seg) ++rb, seg -= n_seg;
    int rb_end = rb + 1;
    if constexpr (kSeveral) {
        rb *= a.row_blocks;
        rb_end = min(rb + a.row_blocks, d.n_row_blocks);
    }
    const int k0 = seg * d.seg_tiles;
    const int k1 = min(k0 + d.seg_tiles, n_ktiles);
    Streams src;
    src.w = d.tiles + (size_t)rb * n_ktiles * Cfg::TB;
    src.t = src.s = nullptr;
    src.w_bytes = (uint32_t)(n_ktiles * Cfg::TB);
    src.t_bytes = src.s_bytes = 0;

    const uint32_t ld = static_cast<uint32_t>(reinterpret_cast<uintptr_t>((lds_ptr<uint8_t>)lds_x));
    // quantization blocks, or sums and steps of 32-column blocks
    const uint32_t lm = ld + (uint32_t)(d.seg_tiles * (kMatrix ? kFp4BytesPerKTile : kDigitBytesPerKTile));
    const uint32_t lr = lm + (uint32_t)(d.seg_tiles * (kMatrix ? kFp4SumBytes : Cfg::GPT * kDigitMetaBytes));  // partial sums [wave][row]
    const uint32_t lf = lr + (kSeveral ? 2 : 1) * kWaves * kRows * 4;  // a word per wave, then (matrix cores) zeros

    float y[1] = {0.f};
    // matrix cores: the lane's sums for weight rows 16 r + lane % 16, and where its part of the first operand is (see multiply_fp4)
    float y4[4] = {0.f, 0.f, 0.f, 0.f};
    const int xb = (lane >> 2) & 3, xg = lane >> 4;  // row 4 xb + digit, columns of lane group xg
    const bool x_mine = (xb & 1) == xg >> 1;
    const uint32_t x_at = ld + (uint32_t)((lane & 15) * 32 + (xg & 1) * 16), zeros = lf + kWaves * 4;
    const uint32_t x_lo = x_mine && xb < 2 ? x_at : zeros, x_lo_step = x_mine && xb < 2 ? kFp4BytesPerKTile : 0u;
    const uint32_t x_hi = x_mine && xb >= 2 ? x_at : zeros, x_hi_step = x_mine && xb >= 2 ? kFp4BytesPerKTile : 0u;
    int acc[4] = {0, 0, 0, 0};  // running sums of the digits, and their joined value (see consume_weights_digits)
    uint32_t before = 0;
    // the four sums of a row meet in LDS, the first wave adds them
    auto publish = [&](uint32_t set) {
        store_lds<float>(set + (wave * kRows + lane) * 4, y[0]);
        __syncthreads();
    };
    auto finish = [&](uint32_t set) {
        y[0] = 0.f;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) y[0] += load_lds<float>(set + (w * kRows + lane) * 4);
        float factor[1] = {1.f};
        if constexpr (SRC == TokenSource::kTablesI16)  // the token's power-of-two step, behind the block sums of the tables
            factor[0] = ldexpf(1.f, uniform(*reinterpret_cast<const int*>(d.lut_s + (size_t)n_ktiles * Cfg::GPT * 4)));
        finish_rows<1>(d, rb, seg, n_seg, lane, y, factor);
    };
    // The activations are requested first and the first weight tiles right behind them: a wave's loads return in
    // the order they were issued, so activations queued behind weight tiles (which come from HBM) would hold the
    // digits back until those tiles are in; this way the digits are made while the weights travel.
    // Four lanes share a block of 32 columns; a pass is 64 blocks, 16 tiles.
    constexpr int kPasses = (kGemvXSegmentTiles * kKTile / 8 + kWaves * 64 - 1) / (kWaves * 64);
    LaneActs xv[kPasses];  // (a pass beyond the segment reads what nobody uses; x beyond K reads as zero)
    if constexpr (SRC == TokenSource::kActivations) {
        const uint32_t x_start = (uint32_t)(k0 * kKTile * 2);  // k0 < n_ktiles, so this lies inside x
        // (the resource starts at the segment's first activation and ends with x, K * 2 bytes less the segment's start: a
        // lane's own offset decides what is read)
        const rsrc_t rx = make_rsrc(d.lut_t + x_start, (uint32_t)d.K * 2u - x_start);
#pragma unroll
        for (int i = 0; i < kPasses; ++i) {
            const int off = (i * kWaves * 64 + (tid & ~3)) * 16 + (tid & 3) * 8;
            xv[i].a = __builtin_amdgcn_raw_buffer_load_b64(rx, off, 0, 0);
            xv[i].b = __builtin_amdgcn_raw_buffer_load_b64(rx, off + 32, 0, 0);
        }
    } else {
        // table j = activations 4j .. 4j + 3: 16 entries of two bytes; entry 1 << t is activation 4j + t
        constexpr int kTable = 32;
        const uint32_t t_start = (uint32_t)k0 * (uint32_t)(kTablesPerKTile * kTable);
        const rsrc_t rt = make_rsrc(d.lut_t + t_start, (uint32_t)n_ktiles * (uint32_t)(kTablesPerKTile * kTable) - t_start);
#pragma unroll
        for (int i = 0; i < kPasses; ++i) {
            const int off = ((i * kWaves * 64 + (tid & ~3)) * 2 + (tid & 3)) * kTable;
            load_table(rt, off, xv[i].a);
            load_table(rt, off + 4 * kTable, xv[i].b);
        }
    }
    __builtin_amdgcn_sched_barrier(0);
    // One bit: the next tile is requested before the wait for the current one, otherwise when the current one is done.
    // A 1-bit tile is 1.3 to 2 KB and 70 vector instructions, so a wave waits longer than it computes: on the dot product unit, with the request
    // at the end of a tile (where the last use of a zero kept it) 16 launches of a layer set of width 1024 took 131 us,
    // else 92; width 3072 145 -> 130, 4096 184 -> 170 (zeros, blocks of 64); on the matrix cores 3.8B layer sets 277 -> 247.  2 and 4
    // bits: more streams in flight cost more than they hide (uint2 g64 +1 %; see tman_mpgemv_x.hip).
    constexpr int kStages = B == 1 ? 2 : 1;
    Stage<B, 1, Cfg::MPL> st[kStages] = {};
    auto issue = [&](auto& s, bool live, int t) { issue_weights<B, 1, GQ, HZ>(s, src, live, t, lane); };
    issue(st[0], k0 + wave < k1, k0 + wave);
    __builtin_amdgcn_sched_barrier(0);

    // digits of the segment: lane -> four lanes per 32-column block, sixteen per tile
    const int n_lanes = (k1 - k0) * (kKTile / 8);
    bool nonfinite = false;
    if constexpr (kMatrix) {
        auto passes = [&](auto count) {
            constexpr int P = decltype(count)::value;
            uint32_t h[P][4], to[P], ts[P];
#pragma unroll
            for (int i = 0; i < P; ++i) {
                const int j = i * kWaves * 64 + tid;
                const bool live = j < n_lanes;
                h[i][0] = live ? xv[i].a.x : 0u, h[i][1] = live ? xv[i].a.y : 0u, h[i][2] = live ? xv[i].b.x : 0u, h[i][3] = live ? xv[i].b.y : 0u;
                // (the partial sums' place is free until all digits are there)
                to[i] = live ? ld + (uint32_t)((j >> 2) * 128 + (j & 3) * 8) : lr;
                ts[i] = live && (j & 3) == 0 ? lm + (uint32_t)((j >> 2) * 8) : lr + 128;
            }
            nonfinite = store_fp8_digits<HZ, P>(h, lane, to, ts);
        };
        static_assert(kPasses == 2, "one or two passes");
        if (kWaves * 64 + wave * 64 < n_lanes) passes(std::integral_constant<int, 2>{});
        else if (wave * 64 < n_lanes) passes(std::integral_constant<int, 1>{});
    } else {
#pragma unroll
        for (int i = 0; i < kPasses; ++i) {
            if (i * kWaves * 64 + wave * 64 >= n_lanes) break;  // (this wave has none)
            const int j = i * kWaves * 64 + tid, tile = j >> 4;
            const bool live = j < n_lanes;
            uint32_t r[4];
            float step = 1.f;
            if constexpr (SRC == TokenSource::kTablesI16)
                bias_block(xv[i].a, xv[i].b, r);
            else
                nonfinite |= quantize_block<GQ>(xv[i].a, xv[i].b, r, step) && live;
            store_digits<GQ>(r, step, j, live, ld + (uint32_t)(tile * kDigitBytesPerKTile + (j & 15) * 16),
                             lm + (uint32_t)((tile * Cfg::GPT + (j & 15) / (GQ / 8)) * kDigitMetaBytes));
        }
    }
    if constexpr (kMatrix)
        if (tid == 0) store_lds<u32x4>(zeros, u32x4{0, 0, 0, 0});
    if constexpr (SRC != TokenSource::kTablesI16)
        store_lds<uint32_t>(lf + wave * 4, __builtin_amdgcn_ballot_w64(nonfinite) != 0 ? 1u : 0u);
    __syncthreads();

    for (int r = 0;; r ^= 1) {  // the row blocks of the workgroup (one, unless kSeveral)
        // the waves take the tiles in turn
        for (int t0 = k0 + wave; t0 < k1; t0 += kStages * kWaves) {
#pragma unroll
            for (int s = 0; s < kStages; ++s) {
                const int t = t0 + s * kWaves;
                if (t < k1) {
                    auto next = [&] { issue(st[(s + 1) % kStages], t + kWaves < k1, t + kWaves); };
                    if constexpr (kMatrix) {
                        const uint32_t at = (uint32_t)(t - k0);
                        multiply_fp4<B, GQ, HZ>(st[s], x_lo + at * x_lo_step, x_hi + at * x_hi_step, lm + at * kFp4SumBytes, lane, y4, next);
                    } else {
                        consume_weights_digits<B, GQ, HZ>(
                            st[s], ld + (uint32_t)((t - k0) * kDigitBytesPerKTile + (lane & 15) * 4),
                            lm + (uint32_t)((t - k0) * Cfg::GPT * kDigitMetaBytes), acc, before, y[0], next);
                    }
                }
            }
        }
        if constexpr (kMatrix) {  // the lane groups' sums of a row meet; lane 16 r + i takes row 16 r + i
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                y4[r] += __shfl_xor(y4[r], 16, 64);
                y4[r] += __shfl_xor(y4[r], 32, 64);
            }
            y[0] = kFp4Factor<HZ> * (lane < 32 ? (lane < 16 ? y4[0] : y4[1]) : (lane < 48 ? y4[2] : y4[3]));
        }
        if constexpr (SRC != TokenSource::kTablesI16) {
            const u32x4 f = load_lds<u32x4>(lf);
            if (uniform((int)(f.x | f.y | f.z | f.w))) {
                auto fetch = [&](int k) -> uint32_t {
                    if constexpr (SRC == TokenSource::kActivations) return load_global<uint16_t>(d.lut_t, (uint32_t)k * 2u);
                    else return load_global<uint16_t>(d.lut_t, ((uint32_t)(k / kLutGroup) * 16u + (1u << (k % kLutGroup))) * 2u);
                };
                for (int t = k0 + wave; t < k1; t += kWaves)
                    y[0] = add_nonfinite<B, GQ, HZ>(src.w + (size_t)t * Cfg::TB, fetch, d.K, t, lane, y[0]);
            }
        }
        if constexpr (!kSeveral) {
            break;
        } else {
            // the next row block's first tile travels while this one's four sums meet in LDS, in one of two sets: a wave
            // writes a set again only after the barrier that follows its last reading
            const bool more = rb + 1 < rb_end;
            src.w += (size_t)n_ktiles * Cfg::TB;
            issue(st[0], more && k0 + wave < k1, k0 + wave);
            publish(lr + (uint32_t)(r * kWaves * kRows * 4));
            if (wave == 0) finish(lr + (uint32_t)(r * kWaves * kRows * 4));
            if (!more) return;
            y[0] = 0.f;
#pragma unroll
            for (int q = 0; q < 4; ++q) y4[q] = 0.f;
            ++rb;
        }
    }
    publish(lr);
    if (wave == 0) finish(lr);
}

// ---------------------------------------------------------------------------------------------
// launch

template <int B, int GQ, bool HZ, TokenSource SRC, bool SINGLE, typename Args>
static int launch_x_cfg(const Args& a, const dim3& grid, int max_seg_tiles, hipStream_t st) {
    constexpr int kSets = several_row_blocks<B, Args> ? 2 : 1;
    static_assert(x_lds_bytes(kGemvXSegmentTiles, kKTile / GQ, on_matrix_cores(B, SRC), kSets) <= 64 * 1024, "LDS of a launch that does not ask for more");
    with_fields(a, [&](auto... f) {
        hipLaunchKernelGGL((mpgemv_x_kernel<B, GQ, HZ, SRC, SINGLE, Args, decltype(f)...>), grid, dim3(kWaves * 64),
                           x_lds_bytes(max_seg_tiles, kKTile / GQ, on_matrix_cores(B, SRC), kSets), st, f...);
    });
    return launch_status();
}

template <int B, bool HZ, TokenSource SRC, bool SINGLE, typename Args>
static int launch_x_group(int group, const Args& a, int n_wg, int max_seg_tiles, hipStream_t st) {
    const dim3 grid((unsigned)n_wg, __is_same(Args, OrderedArgs) ? 1u : (unsigned)a.n_gemv);
    switch (group) {
        case 32: return launch_x_cfg<B, 32, HZ, SRC, SINGLE>(a, grid, max_seg_tiles, st);
        case 64: return launch_x_cfg<B, 64, HZ, SRC, SINGLE>(a, grid, max_seg_tiles, st);
        default: return launch_x_cfg<B, 128, HZ, SRC, SINGLE>(a, grid, max_seg_tiles, st);
    }
}

template <TokenSource SRC, bool SINGLE, typename Args>
static int launch_x_tokens(int np, int bits, int has_zero, int group, const Args& a, int n_wg, int max_seg_tiles, hipStream_t st) {
    if constexpr (SRC != TokenSource::kActivations) {
        constexpr bool INT = SRC == TokenSource::kTablesI16;
        if (np > 1 && lookups_stay(bits, np, INT)) return launch_lookups<SINGLE, INT>(np, bits, has_zero, group, a, n_wg, st);
        if (np == 2) return launch_codes_tables<2, INT, SINGLE>(bits, has_zero, group, a, n_wg, st);
        if (np == 4) return launch_codes_tables<4, INT, SINGLE>(bits, has_zero, group, a, n_wg, st);
        if (np == 8) return launch_codes_tables<8, INT, SINGLE>(bits, has_zero, group, a, n_wg, st);
    }
    if (bits == 1) {
        return has_zero ? launch_x_group<1, true, SRC, SINGLE>(group, a, n_wg, max_seg_tiles, st)
                        : launch_x_group<1, false, SRC, SINGLE>(group, a, n_wg, max_seg_tiles, st);
    }
    if (bits == 2) return launch_x_group<2, true, SRC, SINGLE>(group, a, n_wg, max_seg_tiles, st);
    return launch_x_group<4, true, SRC, SINGLE>(group, a, n_wg, max_seg_tiles, st);
}

// A single GEMV, a numbered batch and a batch on the plain grid from one source of activations.
template <TokenSource SRC>
static int launch_x_single(const Layout& L, int N, const void* packed, const void* x, void* y, void* workspace, hipStream_t st) {
    KernelArgs<true> a;
    const GemvPlan p = plan_decode(L, N, N > 1 && fills_device(plan_tables(L, N).n_workgroups));
    fill_desc_plan(a.single, L, p, packed, x, N, y, workspace);
    a.n_gemv = 1;
    a.status = device_status_word();
    if (!a.status) return TMAN_ERR_LAUNCH;
    return launch_x_tokens<SRC, true>(p.np, L.bits, L.has_zero, L.group, a, p.n_workgroups, p.seg_tiles, st);
}
template <TokenSource SRC>
static int launch_x_batch(const DecodeBatch& b, hipStream_t st) {
    if (b.order) {
        OrderedArgs a;
        a.descs = b.descs;
        a.order = b.order;
        a.n_gemv = b.n_gemv;
        return launch_x_tokens<SRC, false>(padded_tokens(b.N), b.bits, b.has_zero, b.group, a, b.n_workgroups, b.max_seg_tiles, st);
    }
    KernelArgs<false> a;
    a.descs = b.descs;
    a.n_gemv = b.n_gemv;
    a.row_blocks = b.row_blocks;
    return launch_x_tokens<SRC, false>(padded_tokens(b.N), b.bits, b.has_zero, b.group, a, b.n_workgroups, b.max_seg_tiles, st);
}

}  // namespace tman
