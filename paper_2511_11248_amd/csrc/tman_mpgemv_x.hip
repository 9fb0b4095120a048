// Decoding mpGEMV of ONE token: tman_mpgemv_x (activations in), and tman_mpgemv / tman_mpgemv_i16 for one token
// (tables in).
//
// y[m] = sum_G scale[m][G] * (sum_{k in G} q[m][k] x[k] - zero[m][G] * S[G]) (Sec. 2.2).  The lookups of Sec. 4.3 turn
// the inner sum into one table read per 4 weights and bit-plane; on this chip that costs 2.6 vector instructions and
// an LDS read each, and the kernel built that way was bound by vector issue (7B layer sets: uint2 g64 14.7 us, uint4
// g128 24.2 us per launch).  Here the sum is taken in integers: the activations of a quantization block become 16-bit
// fixed-point numbers, split into four signed 4-bit digits, and v_dot8c_i32_i4 multiplies eight codes with one digit
// (see tman_digits_device.h for the instruction counts and the precision).
//
// A workgroup of four waves owns one row block (64 rows, one per lane) and one K segment of at most 32 tiles.  It
// makes the digits of its segment itself (8 KB of activations -> 8 KB of digit words in LDS) while its first weight
// tiles are on their way, so a decode step needs no launch for a precompute.  Given tables, it takes the activations
// out of them: the entries of patterns 1, 2, 4 and 8 are the four activations themselves.  The sums of the four waves
// meet in LDS, segments of a long K through the workspace (tickets, fixed order of addition).
//
// What bounds it: the weight stream.  63.2 MB (7B uint2 g64) in 13.4 us = 4.7 TB/s, 107.5 MB (uint4 g128) in 19.3
// us = 5.6 TB/s; reading alone reaches 6.0-6.15 TB/s, and about 1 us at the start (descriptor, first activations)
// and 1.5 us at the end (exchange between segments) are not covered.  What helped beside the digits, measured in
// turn on the uint2 / uint4 launch: the waves of a workgroup take its tiles in turn instead of a quarter each, so that
// a workgroup reads one contiguous stream (uint4 20.6 -> 20.1 us); ONE tile in flight per wave instead of two or three
// (uint2 14.2 -> 13.6 us with two against one, 15.2 with three: more streams in flight cost more in the memory
// system than they hide); no issue priorities (uint2 14.3 -> 13.9 us: they balanced vector work, which no longer
// bounds); K up to 4096 as one segment also for 4-bit weights (uint4 20.7 -> 19.6 us).
#include <algorithm>
#include <vector>

#include "tman_digits_device.h"

namespace tman {

// LDS of a workgroup whose segment has `seg_tiles` tiles: digit words and at most 4 quantization blocks per tile, then
// (16-byte aligned) the partial sums and a word per wave
static unsigned x_lds_bytes(int seg_tiles) {
    return (unsigned)seg_tiles * (kDigitBytesPerKTile + 4 * kDigitMetaBytes) + kWaves * kRows * 4 + kWaves * 4;
}

// Segments (measured on the 7B and 3.8B layer sets): a K that one workgroup can take whole - up to 32 tiles and 160 KB
// of packed weights per row block - is one segment, which spares the exchange of partial sums; a longer K is cut into
// equal segments of at most 17 tiles.
GemvPlan plan_gemv_x(const Layout& L) {
    const tman_tiling_t t = current_tiling();
    int whole = t.decode_x_whole_bytes / L.tile_bytes;
    if (whole > t.decode_x_seg_tiles) whole = t.decode_x_seg_tiles;
    if (whole < 1) whole = 1;
    return plan_segments(L, 1, L.n_ktiles <= whole ? whole : t.decode_x_long_seg_tiles);
}

void fill_desc_x(GemvDesc& d, const Layout& L, const void* packed, const void* x, void* y, void* workspace) {
    fill_desc_plan(d, L, plan_gemv_x(L), packed, x, 1, y, workspace);
}

// The 8 activations of a lane: numbers 4f .. 4f + 3 (a) and 16 + 4f .. (b) of its 32-column block.
struct LaneActs {
    u32x2 a, b;
};

template <int B, int GQ, bool HZ, TokenSource SRC, bool SINGLE, typename Args>
__global__ void __launch_bounds__(kWaves * 64) mpgemv_x_kernel(Args a) {
    using Cfg = GemvCfg<B, 1, GQ, HZ>;
    extern __shared__ __attribute__((aligned(1024))) uint8_t lds_x[];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);

    int g, wg_local;
    workgroup_of<SINGLE>(a, g, wg_local);
    const GemvDesc d = desc_value<SINGLE>(a, g);  // (one load: the fields are needed one after the other)
    const int n_seg = d.n_seg, n_ktiles = d.n_ktiles;
    // Exits: surplus workgroups of the grid, and (single call) a blob packed for another shape or layout, which is
    // reported and leaves y alone; a batch is checked when its descriptor table is written, which empties the
    // descriptor of such a GEMV.  One exit for both, before any other memory request.
    int n_wg = d.n_row_blocks * n_seg;
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
    const int seg_tiles = d.seg_tiles;
    const int k0 = seg * seg_tiles;
    const int k1 = min(k0 + seg_tiles, n_ktiles);
    Streams src;
    src.w = d.tiles + (size_t)rb * n_ktiles * Cfg::TB;
    src.t = src.s = nullptr;
    src.w_bytes = (uint32_t)(n_ktiles * Cfg::TB);
    src.t_bytes = src.s_bytes = 0;

    const uint32_t ld = static_cast<uint32_t>(reinterpret_cast<uintptr_t>((lds_ptr<uint8_t>)lds_x));
    const uint32_t lm = ld + (uint32_t)seg_tiles * kDigitBytesPerKTile;     // quantization blocks
    const uint32_t lr = lm + (uint32_t)seg_tiles * Cfg::GPT * kDigitMetaBytes;  // partial sums [wave][row]
    const uint32_t lf = lr + kWaves * kRows * 4;                            // a word per wave

    // The activations are requested first and the first weight tiles right behind them: a wave's loads return in
    // the order they were issued, so activations queued behind weight tiles (which come from HBM) would hold the
    // digits back until those tiles are in; this way the digits are made while the weights travel.
    // Four lanes share a block of 32 columns; a pass is 64 blocks, 16 tiles.
    constexpr int kPasses = kGemvXSegmentTiles * kKTile / (8 * kWaves * 64);
    static_assert(kPasses * 8 * kWaves * 64 == kGemvXSegmentTiles * kKTile, "whole passes");
    LaneActs xv[kPasses];  // (a pass beyond the segment reads what nobody uses; x beyond K reads as zero)
    if constexpr (SRC == TokenSource::kActivations) {
        const uint32_t x_start = (uint32_t)(k0 * kKTile * 2);  // k0 < n_ktiles, so this lies inside x
        // (the range check of a buffer load covers the per-lane offset only, not the scalar offset, so the resource
        // starts at the segment's first activation and ends with x: K * 2 bytes less the segment's start)
        const rsrc_t rx = make_rsrc(d.lut_t + x_start, (uint32_t)d.K * 2u - x_start);
#pragma unroll
        for (int i = 0; i < kPasses; ++i) {
            const int off = (i * kWaves * 64 + (tid & ~3)) * 16 + (tid & 3) * 8;
            xv[i].a = __builtin_amdgcn_raw_buffer_load_b64(rx, off, 0, 0);
            xv[i].b = __builtin_amdgcn_raw_buffer_load_b64(rx, off + 32, 0, 0);
        }
    } else {
        // table j = activations 4j .. 4j + 3: 16 entries of two bytes; entry 1 << t is activation 4j + t
        const uint32_t t_start = (uint32_t)k0 * kTableBytesPerKTile;
        const rsrc_t rt = make_rsrc(d.lut_t + t_start, (uint32_t)n_ktiles * kTableBytesPerKTile - t_start);
        auto table = [&](int off) {
            const u32x4 lo = __builtin_amdgcn_raw_buffer_load_b128(rt, off, 0, 0);
            const uint32_t e8 = __builtin_amdgcn_raw_buffer_load_b32(rt, off + 16, 0, 0);
            const uint32_t e01 = lo.x, e23 = lo.y, e45 = lo.z;
            return u32x2{__builtin_amdgcn_perm(e23, e01, 0x05040302u), __builtin_amdgcn_perm(e8, e45, 0x05040100u)};
        };
#pragma unroll
        for (int i = 0; i < kPasses; ++i) {
            const int off = ((i * kWaves * 64 + (tid & ~3)) * 2 + (tid & 3)) * 32;
            xv[i].a = table(off);
            xv[i].b = table(off + 4 * 32);
        }
    }
    __builtin_amdgcn_sched_barrier(0);
    Stage<B, 1, Cfg::MPL> st = {};
    issue_weights<B, 1, GQ, HZ>(st, src, k0 + wave < k1, k0 + wave, lane);
    __builtin_amdgcn_sched_barrier(0);

    // digits of the segment: lane -> four lanes per 32-column block
    const int n_lanes = (k1 - k0) * (kKTile / 8);
    bool nonfinite = false;
#pragma unroll
    for (int i = 0; i < kPasses; ++i) {
        if (i * kWaves * 64 >= n_lanes) break;
        const int j = i * kWaves * 64 + tid;
        uint32_t r[4];
        float step = 1.f;
        if constexpr (SRC == TokenSource::kTablesI16)
            bias_block(xv[i].a, xv[i].b, r);
        else
            nonfinite |= quantize_block<GQ>(xv[i].a, xv[i].b, r, step) && j < n_lanes;
        store_digits<GQ>(r, step, j, j < n_lanes, ld, lm);
    }
    if constexpr (SRC != TokenSource::kTablesI16)
        store_lds<uint32_t>(lf + wave * 4, __builtin_amdgcn_ballot_w64(nonfinite) != 0 ? 1u : 0u);
    __syncthreads();

    float y = 0.f;
    for (int t = k0 + wave; t < k1; t += kWaves) {
        consume_weights_digits<B, GQ, HZ>(st, ld + (t - k0) * kDigitBytesPerKTile + (lane & 15) * 4,
                                          lm + (t - k0) * Cfg::GPT * kDigitMetaBytes, y);
        issue_weights<B, 1, GQ, HZ>(st, src, t + kWaves < k1, t + kWaves, lane);
    }
    if constexpr (SRC != TokenSource::kTablesI16) {
        const u32x4 f = load_lds<u32x4>(lf);
        if (uniform((int)(f.x | f.y | f.z | f.w))) {
            auto fetch = [&](int k) -> uint32_t {
                if constexpr (SRC == TokenSource::kActivations) return load_global<uint16_t>(d.lut_t, (uint32_t)k * 2u);
                else return load_global<uint16_t>(d.lut_t, ((uint32_t)(k / kLutGroup) * 16u + (1u << (k % kLutGroup))) * 2u);
            };
            for (int t = k0 + wave; t < k1; t += kWaves)
                y = add_nonfinite<B, GQ, HZ>(src.w + (size_t)t * Cfg::TB, fetch, d.K, t, lane, y);
        }
    }

    store_lds<float>(lr + (wave * kRows + lane) * 4, y);
    __syncthreads();
    if (wave != 0) return;
    y = 0.f;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) y += load_lds<float>(lr + (w * kRows + lane) * 4);
    float yy[1] = {y};
    float factor[1] = {1.f};
    if constexpr (SRC == TokenSource::kTablesI16)  // the token's power-of-two step, behind the block sums of the tables
        factor[0] = ldexpf(1.f, uniform(*reinterpret_cast<const int*>(d.lut_s + (size_t)n_ktiles * Cfg::GPT * 4)));
    finish_rows<1>(d, rb, seg, n_seg, lane, yy, factor);
}

// ---------------------------------------------------------------------------------------------
// launch

template <int B, bool HZ, TokenSource SRC, bool SINGLE, typename Args>
static int launch_x_group(int group, const Args& a, int n_wg, int max_seg_tiles, hipStream_t st) {
    const dim3 grid((unsigned)n_wg, __is_same(Args, OrderedArgs) ? 1u : (unsigned)a.n_gemv), block(kWaves * 64);
    const unsigned lds = x_lds_bytes(max_seg_tiles);
    switch (group) {
        case 32: hipLaunchKernelGGL((mpgemv_x_kernel<B, 32, HZ, SRC, SINGLE, Args>), grid, block, lds, st, a); break;
        case 64: hipLaunchKernelGGL((mpgemv_x_kernel<B, 64, HZ, SRC, SINGLE, Args>), grid, block, lds, st, a); break;
        default: hipLaunchKernelGGL((mpgemv_x_kernel<B, 128, HZ, SRC, SINGLE, Args>), grid, block, lds, st, a); break;
    }
    return launch_status();
}

template <TokenSource SRC, bool SINGLE, typename Args>
static int launch_x_format(int bits, int has_zero, int group, const Args& a, int n_wg, int max_seg_tiles, hipStream_t st) {
    if (bits == 1) {
        return has_zero ? launch_x_group<1, true, SRC, SINGLE>(group, a, n_wg, max_seg_tiles, st)
                        : launch_x_group<1, false, SRC, SINGLE>(group, a, n_wg, max_seg_tiles, st);
    }
    if (bits == 2) return launch_x_group<2, true, SRC, SINGLE>(group, a, n_wg, max_seg_tiles, st);
    return launch_x_group<4, true, SRC, SINGLE>(group, a, n_wg, max_seg_tiles, st);
}

template <bool SINGLE, typename Args>
static int launch_x_source(TokenSource source, int bits, int has_zero, int group, const Args& a, int n_wg, int max_seg_tiles,
                           hipStream_t st) {
    switch (source) {
        case TokenSource::kActivations:
            return launch_x_format<TokenSource::kActivations, SINGLE>(bits, has_zero, group, a, n_wg, max_seg_tiles, st);
        case TokenSource::kTables:
            return launch_x_format<TokenSource::kTables, SINGLE>(bits, has_zero, group, a, n_wg, max_seg_tiles, st);
        default:
            return launch_x_format<TokenSource::kTablesI16, SINGLE>(bits, has_zero, group, a, n_wg, max_seg_tiles, st);
    }
}

int launch_mpgemv_x(TokenSource source, const Layout& L, const void* packed, const void* x, void* y, void* workspace,
                    hipStream_t st) {
    KernelArgs<true> a;
    fill_desc_x(a.single, L, packed, x, y, workspace);
    a.n_gemv = 1;
    a.status = device_status_word();
    if (!a.status) return TMAN_ERR_LAUNCH;
    const GemvPlan p = plan_gemv_x(L);
    return launch_x_source<true>(source, L.bits, L.has_zero, L.group, a, p.n_workgroups, p.seg_tiles, st);
}

// The numbered launch of a one-token batch (see order_workgroups_of): at most 8 workgroups per compute unit, and no
// more than 5 of 32 tiles - all of them are resident (LDS 11 KB, at most 66 vector registers), but numbering a
// launch pays while a unit has few of them (1152 workgroups of a layer set with MLP width 14336, uint4 g128: 25.5 us on
// the plain grid, 23.3 us numbered; equal workgroups need none).
static int x_resident_per_unit(int count, const Layout* L) {
    int max_seg_tiles = 1;
    for (int g = 0; g < count; ++g) max_seg_tiles = std::max(max_seg_tiles, plan_gemv_x(L[g]).seg_tiles);
    return std::min(8, 160 / max_seg_tiles);
}
int ordered_workgroups(int count, const Layout* L, int n_units) {
    if (count > 8) return 0;
    std::vector<GemvPlan> plans(count);
    for (int g = 0; g < count; ++g) plans[g] = plan_gemv_x(L[g]);
    return ordered_workgroups_of(count, L, plans.data(), n_units, x_resident_per_unit(count, L));
}
bool order_workgroups(int count, const Layout* L, int n_units, std::vector<uint16_t>* order) {
    if (count > 8) return false;
    std::vector<GemvPlan> plans(count);
    for (int g = 0; g < count; ++g) plans[g] = plan_gemv_x(L[g]);
    return order_workgroups_of(count, L, plans.data(), n_units, x_resident_per_unit(count, L), order);
}

int launch_mpgemv_x_ordered(TokenSource source, int bits, int group, int has_zero, const GemvDesc* descs_dev, int n_gemv,
                            const uint16_t* order_dev, int n_wg, int max_seg_tiles, hipStream_t st) {
    OrderedArgs a;
    a.descs = descs_dev;
    a.order = order_dev;
    a.n_gemv = n_gemv;
    return launch_x_source<false>(source, bits, has_zero, group, a, n_wg, max_seg_tiles, st);
}

int launch_mpgemv_x_batch(TokenSource source, int bits, int group, int has_zero, const GemvDesc* descs_dev, int n_gemv,
                          int max_workgroups, int max_seg_tiles, hipStream_t st) {
    KernelArgs<false> a;
    a.descs = descs_dev;
    a.n_gemv = n_gemv;
    return launch_x_source<false>(source, bits, has_zero, group, a, max_workgroups, max_seg_tiles, st);
}

}  // namespace tman
