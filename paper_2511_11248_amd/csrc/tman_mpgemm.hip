// Prefill mpGEMM: two-level dequantization fused in front of the matrix cores
// (Sec. 4.1 "Unified Layout through Fused LUT-based Dequantization", Sec. 4.2 three-stage pipeline).
//
// The weights stay in the bit-serial layout decoding uses (lane = row, 64 rows x 128 columns per tile
// block).  Per 32-column stage a producer wave turns the bit-plane words of its 64 rows into fp16 weights:
//   level 1  bit-serial -> bit-parallel (Sec. 4.1 "Bit repacking"): two rounds of bit-field inserts
//            transpose a 4 x 32 bit matrix in 16 ALU ops, giving for each 32-weight block four words
//            of eight 4-bit codes, word o holding the codes of weights 4f + o;
//   level 2  code -> fp16 weight with the block's scale and zero baked in (Sec. 4.1 "Integer-to-float
//            conversion", "Applying scales and zero-points").  The 16-entry conversion table of the
//            paper collapses on this hardware to inserting the code into the mantissa of 1024.0
//            (fp16 0x6400 | c == 1024 + c exactly), and the baked affine table entry
//            D[c] = fp16((c - zero) * scale) is produced by one fp32 FMA, (1024 + c) * scale - (1024 + zero) * scale,
//            and one conversion of two results to fp16.  The FMA rounds to fp32 and the conversion to fp16; in three times
//            2^20 random entries, zeros inside the codes' range and far outside it, that gave the bits of the exact result
//            rounded once to fp16 every time.  The per-block constant -(1024 + zero) * scale, computed once per block,
//            is rounded to fp32 before (it has up to 24 significant bits), which moves the result by at most
//            2^-23 * 1040 * scale: about 5 % of the entries come out one fp16 step from fp16((c - zero) * scale).
//            A lookup per weight in LDS would compete with the MFMA operand reads for LDS bandwidth.
// The fp16 weight tile goes to LDS and is shared by the waves of the workgroup (each weight is
// dequantized once per 256 tokens); activations go from global memory straight into LDS.  Pipeline (the
// GPU form of DMA -> vector -> matrix): producer waves keep packed weights four stages ahead in registers
// and fill a ring of LDS stage buffers; consumer waves feed v_mfma_f32_32x32x16_f16
// (fp32 accumulation) from the ring; one barrier per 32-column stage.
// Grids too small for that kernel go to mpgemm_ksplit_kernel, grids whose rounds its tiles fit badly to mpgemm_wide_kernel, both
// below; choose_tile decides.
#include <hip/hip_fp16.h>

#include <mutex>

#include "tman_activation_requests.h"
#include "tman_dequant_device.h"

namespace tman {

typedef _Float16 half8_t __attribute__((ext_vector_type(8)));
typedef _Float16 half2_t __attribute__((ext_vector_type(2)));
typedef float float16_t __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

constexpr int kTN = 256;      // tokens per workgroup
constexpr int kStageK = 32;   // columns per pipeline stage (one 32-weight block of the layout)
constexpr int kRowBytes = kStageK * 2 + 16;  // padded LDS row: 20 dwords, conflict-free 16-byte accesses
constexpr int kRing = 3;      // weight buffers in LDS (a stage each) and activation buffers (a pair of stages each)
constexpr int kSets = 4;      // register sets of the producers = stages of global loads in flight
constexpr int kXcds = 8;      // workgroups are dealt to the chip's 8 XCDs (one L2 each) round robin

// A workgroup covers RB row blocks (64 * RB output features) x 256 tokens; RB = 1 .. 4 is chosen
// per call so that the number of workgroups fills the compute units best.
template <int RB>
struct Tile {
    static constexpr int TM = RB * 64;
    static constexpr int WBytes = TM * kRowBytes;    // fp16 weights of a stage, padded rows
    static constexpr int XBytes = kTN * kStageK * 4; // activations of a pair of stages, 128-byte rows, chunks swizzled
    static constexpr int OutRow = TM * 2 + 16;       // bytes per token of the output tile in LDS
    static constexpr int LdsBytes = kRing * (WBytes + XBytes) > kTN * OutRow ? kRing * (WBytes + XBytes) : kTN * OutRow;
    static_assert(LdsBytes <= 160 * 1024, "tile of the tiled kernel");
};

struct GemmArgs {
    const uint8_t* tiles;
    const _Float16* x;
    _Float16* y;
    int* status;  // the library's status word
    int M, N, K, n_row_blocks;
    int m_tiles, n_tiles;
    int per_xcd;  // workgroups dealt to each XCD
    int whole_row_tiles;
};
// The kernels take the 16 words of their arguments one by one: of scalar arguments the first 14 words are in registers when a wave
// starts (the build asks for it), a structure is read from memory first (44 shapes of 6 to 200 us: 1.006 and 1.018 times as fast in
// two runs).  The last two, per_xcd and whole_row_tiles, are still read from memory ahead of everything else.
template <typename Launch>
static int with_fields(const GemmArgs& a, Launch launch) {
    return launch(a.tiles, a.x, a.y, a.status, a.M, a.N, a.K, a.n_row_blocks, a.m_tiles, a.n_tiles, a.per_xcd, a.whole_row_tiles);
}
// Launches a kernel that takes more LDS than a kernel may without asking (once per kernel instantiation, also when several host
// threads make their first call together).
template <int LDS_BYTES, typename... Fields>
static int launch_with_lds(void (*kernel)(Fields...), std::once_flag& once, hipError_t& attr_rc, unsigned grid, int threads,
                           hipStream_t st, Fields... fields) {
    std::call_once(once, [&] {
        attr_rc = hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, LDS_BYTES);
    });
    if (attr_rc != hipSuccess) return TMAN_ERR_LAUNCH;
    hipLaunchKernelGGL(kernel, dim3(grid), dim3(threads), LDS_BYTES, st, fields...);
    return launch_status();
}

// Tile of this workgroup, token tiles fastest.  Consecutive workgroup ids go to consecutive XCDs, and the token tiles that
// share the weights of one row tile should sit on one XCD and its L2.  Either every XCD gets an equal run of consecutive
// tiles, which cuts up to seven row tiles in two, or row tiles are dealt out whole, which may leave XCDs unequal (see
// deal_tiles).  `mt` may lie past the last row tile.
__device__ __forceinline__ void tile_of_workgroup(const GemmArgs& a, int& mt, int& nt) {
    const int xcd = (int)(blockIdx.x % kXcds), slot = (int)(blockIdx.x / kXcds);
    const int at = a.whole_row_tiles ? slot : xcd * a.per_xcd + slot, row = at / a.n_tiles;
    nt = at - row * a.n_tiles;
    mt = a.whole_row_tiles ? row * kXcds + xcd : row;
}

typedef __amdgpu_buffer_rsrc_t rsrc_t;
// raw buffer resource: loads at or beyond `bytes` return zero
__device__ __forceinline__ rsrc_t make_rsrc(const void* base, uint32_t bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, bytes, 0x00020000);
}

// Loads 32-weight block `kb32` of tile block `tile` of this wave's row block.  `rw` covers the row
// block's tiles or nothing (rows beyond M, stages beyond K), in which case everything reads as zero.
template <int B, int GQ, bool HZ>
__device__ __forceinline__ void load_w(WRegs<B>& r, rsrc_t rw, int tile, int kb32, int lane) {
    constexpr int CH = kKTile / B;
    constexpr int MSZ = HZ ? 4 : 2;
    constexpr int MPL = (kKTile / GQ) * MSZ;
    constexpr int TB = B * 1024 + 64 * MPL;
    const int v = (kb32 * 32) / CH, ksub = ((kb32 * 32) % CH) / 32;
    const int so = tile * TB + v * 1024 + ksub * B * 4;
    if constexpr (B == 4) {
        const u32x4 w = __builtin_amdgcn_raw_buffer_load_b128(rw, lane * 16, so, 0);
        r.plane[0] = w.x; r.plane[1] = w.y; r.plane[2] = w.z; r.plane[3] = w.w;
    } else if constexpr (B == 2) {
        const u32x2 w = __builtin_amdgcn_raw_buffer_load_b64(rw, lane * 16, so, 0);
        r.plane[0] = w.x; r.plane[1] = w.y;
    } else {
        r.plane[0] = __builtin_amdgcn_raw_buffer_load_b32(rw, lane * 16, so, 0);
    }
    const int mo = tile * TB + B * 1024 + ((kb32 * 32) / GQ) * MSZ;
    if constexpr (HZ) r.meta = __builtin_amdgcn_raw_buffer_load_b32(rw, lane * MPL, mo, 0);
    else r.meta = __builtin_amdgcn_raw_buffer_load_b16(rw, lane * MPL, mo, 0);
}

// Activation staging: a token contributes 128 bytes, a whole cache line, to a pair of stages (with 64 bytes per stage every
// line came into the unit's L1 twice: 11008 x 4096 uint4 N = 1024 94.2 -> 92.5 us, 12288 x 4096 uint2 N = 2048 193.5 -> 188.5).  They go
// from global memory straight into LDS (no registers, no LDS store instruction); such a load writes
// the 64 lanes' 16 bytes consecutively, i.e. 8 token rows of 128 bytes per wave instruction.  Rows are
// not padded, so chunk c of token row R is kept at position c ^ ((R >> 1) & 7) of its row: the MFMA
// operand reads of 16 consecutive rows then fall into 16 different 16-byte bank groups.  The
// permutation is applied on the global-address side, where every lane is free to pick its source.

// Workgroup = 12 waves, three per SIMD.  Waves 0..7 are consumers: wave (wm, wn) owns 32 RB rows x 64
// tokens of the tile and does nothing but read MFMA operands from LDS and issue MFMAs.  Waves 8..11
// are producers: wave p < RB turns row block p of each stage into fp16 in LDS, and all four stage the
// activations.  Vector work of the producers and matrix work of the consumers come from different
// waves of a SIMD, so the hardware overlaps them without any help from the instruction schedule.
//
// Ring protocol, one barrier at the end of every stage s: before it the producers have written the weights of stage
// s+2 and the consumers have finished reading stage s.  Hence consumers may prefetch operands of stage
// s+1 during stage s, and the buffer written during stage s (stage s+2) was last read in stage s-1.  The activations
// of pair P+2 are requested in stages 2P and 2P+1, whose buffer was last read in stage 2P-1, and are in by the end of stage
// 2P+2, before the first prefetch from them.
// The producers hold the global loads of four further stages in registers: at the rates of this kernel
// that many bytes in flight are needed to cover the latency of HBM and L2.
constexpr int kConsumerWaves = 8;
constexpr int kThreads = 768;

template <int B, int GQ, bool HZ, int RB, typename... Fields>
__global__ void __launch_bounds__(kThreads, 1) mpgemm_kernel(Fields... fields) {
    const GemmArgs a{fields...};
    const int n_ktiles = (a.K + kKTile - 1) / kKTile;
    using T = Tile<RB>;
    constexpr int MSZ = HZ ? 4 : 2;
    constexpr int TB = B * 1024 + 64 * (kKTile / GQ) * MSZ;

    extern __shared__ __attribute__((aligned(16))) uint8_t smem[];

    int mt, nt;
    tile_of_workgroup(a, mt, nt);
    // A blob packed for another shape or layout: say so and leave y alone.  (The check is folded into the one
    // exit below: a second exit after this load makes the compiler keep the dequantization state in scratch
    // memory.)
    const bool header_ok = header_matches(a.tiles, a.M, a.K, B, GQ, HZ ? 1 : 0);
    if (!header_ok && blockIdx.x == 0 && threadIdx.x == 0) report_header_mismatch(a.status);
    if (mt >= (header_ok ? a.m_tiles : 0)) return;

    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int n0 = nt * kTN;
    // K is a multiple of the quantization group, hence of 32.  The loops run a multiple of four stages
    // (no conditional code between the loads and their use); a stage beyond K holds zero activations.
    // (Eight with one row block, whose producers work in rounds of eight stages.)
    constexpr int kRound = RB == 1 ? 2 * kSets : kSets;
    const int k_stages = a.K / kStageK, n_stages = (k_stages + kRound - 1) & ~(kRound - 1);

    float16_t acc[RB][2];
#pragma unroll
    for (int mb = 0; mb < RB; ++mb)
#pragma unroll
        for (int nb = 0; nb < 2; ++nb)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[mb][nb][v] = 0.f;
    const int wm = (wave >> 2) & 1, wn = wave & 3, r = lane & 31, h = lane >> 5;

    if (wave >= kConsumerWaves) {
        // ---------------------------------------------------------------- producer
        const int p = wave - kConsumerWaves;
        // the row block this wave dequantizes (with one row block per workgroup waves 0 and 1 share it)
        const int pb = RB == 1 ? 0 : p;
        const int rbw = mt * RB + pb;
        // the producers' short vector bursts gate every stage: issue them ahead of the consumers' MFMAs
        __builtin_amdgcn_s_setprio(3);
        const bool wvalid = (RB == 1 ? p < 2 : p < RB) && rbw < a.n_row_blocks;
        const uint8_t* wsrc = a.tiles + (size_t)(wvalid ? rbw : 0) * n_ktiles * TB;
        const int xrows = a.N - n0 < kTN ? a.N - n0 : kTN;
        const _Float16* xsrc = a.x + (size_t)n0 * a.K;
        const uint32_t xbytes = (uint32_t)xrows * (uint32_t)a.K * 2u;
        // Roles.  With four row blocks every producer wave dequantizes one and issues a quarter of the
        // activation loads.  With fewer, wave 3 has no row block: it issues all activation loads (about 40
        // cycles each) and the dequantizing waves none, which shortens the chain that gates a stage. (With one
        // row block wave 2 helps it ahead of the loop.)
        constexpr bool kSplitRoles = RB < 4;
        constexpr int kLoaderWave = 3;
        constexpr int kXAll = kTN / 16;  // activation loads per stage, half of a pair's (8 token rows each)
        const uint32_t xlane = (uint32_t)(lane >> 3) * (uint32_t)a.K * 2u;
        const uint32_t xsrc_chunk[2] = {request_chunk(0, lane), request_chunk(1, lane)};
        const uint32_t x8rows = 8u * (uint32_t)a.K * 2u;  // bytes between the sources of consecutive loads
        uint8_t* const xring = smem + kRing * T::WBytes;
        // load number i of a pair of stages fills token rows 8 i .. 8 i + 7; lane = 8 * row + position; `odd`: `first` is odd.
        // Columns beyond K in the last pair belong to a stage that is not multiplied; those of the last token are not read either
        // (resource_bytes).
        auto load_x = [&](int pair, int first, int count, int odd = 0) {
            // (only with blocks of 32 can K be an odd multiple of 32; the others start every resource at the tile's first token,
            // which takes less scalar work per pair: 4096 x 4096 N = 700 blocks of 64, 192 x 256 tiles 64.1 us, else 64.5; blocks of 32
            // 66.7 -> 66.7, 128 x 256 tiles 58.8 -> 59.7, 256 x 256 82.3 -> 82.0)
            constexpr bool kHalfPair = GQ == 32;
            const rsrc_t rx = kHalfPair ? make_rsrc(reinterpret_cast<const uint8_t*>(xsrc) + (uint32_t)pair * kPairBytes,
                                                    resource_bytes(xbytes, pair, k_stages))
                                        : make_rsrc(xsrc, 2 * pair < k_stages ? xbytes : 0u);
            uint8_t* dst = xring + (uint32_t)pair % kRing * T::XBytes;
#pragma unroll
            for (int i = 0; i < 2 * kXAll; ++i)
                if (i < count)
                    __builtin_amdgcn_raw_ptr_buffer_load_lds(rx, (__attribute__((address_space(3))) void*)(dst + (first + i) * 1024),
                                                             16, xlane + xsrc_chunk[(i + odd) & 1] + (uint32_t)(first + i) * x8rows,
                                                             kHalfPair ? 0 : pair * kPairBytes, 0, 0);
        };
        const int wdst = (pb * 64 + lane) * kRowBytes;  // this lane's 64 bytes in the weight tile

        WRegs<B> wr[kSets];
        // stage t: packed weights global -> register set (a wave without a row block reads nothing)
        auto load_wregs = [&](int set, int t) {
            load_w<B, GQ, HZ>(wr[set], make_rsrc(wsrc, t < k_stages && wvalid ? 0x7fffffffu : 0u), t >> 2, t & 3, lane);
        };
        auto w_to_lds = [&](int set, int t) {
            if (p < RB) dequant_to_lds<B, HZ>(wr[set], smem + (uint32_t)t % kRing * T::WBytes + wdst);
        };
        // Ring timing, any role: during stage s half of the activations of pair s/2 + 2 are requested, the weights of stage s+2
        // go registers -> ring and the weights of stage s+6 global -> the same registers.  Loads complete in order.  Before
        // the barrier of an even stage s the activations of pair s/2 + 1 must have landed; their second half was issued first
        // in stage s-1.
        if (kSplitRoles && p == kLoaderWave) {
            // Ahead of the first barrier: pair 0 and half of pair 1.  Pair 1 is not read before stage 1, and behind all of it the
            // barrier comes later: K <= 512, 128 and 192 rows 0.3 to 1.2 % (one row block 1.2 %, and 1.1 to 2.3 % more with wave 2
            // asking for half of the rows).
            constexpr int kMine = RB == 1 ? kXAll : 2 * kXAll;  // of a pair's requests
            load_x(0, 0, kMine);
            __builtin_amdgcn_sched_barrier(0);  // (the wait below counts the requests behind these)
            load_x(1, 0, kMine / 2);
            asm volatile("s_waitcnt vmcnt(%0)" ::"n"(kMine / 2) : "memory");
            asm volatile("s_barrier" ::: "memory");
            load_x(1, kMine / 2, kMine / 2);
            // The requests of a stage are spread over it (s_sleep: 64 cycles a step): what they write to LDS and read from L2
            // in one go keeps the other waves waiting.  4096 x 4096 N = 700, 192 x 256 tiles, all at once / in fours with
            // 1 / 3 / 5 steps between: 70.6 / 69.1 / 65.7 / 74.0 us (11008 x 4096 N = 1024 92.9 / 91.8 / 90.6 / 94.9).
            constexpr int kPause = RB == 3 ? 3 : RB == 2 ? 2 : 1;
            auto spread_x = [&](int pair, int first) {
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    load_x(pair, first + 4 * q, 4);
                    if (q < 3) __builtin_amdgcn_s_sleep(kPause);
                }
            };
            for (int s = 0; s < n_stages; s += 2) {
                spread_x(s / 2 + 2, 0);
                // younger than the loads of pair s/2 + 1: the sixteen just issued
                asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"(kXAll) : "memory");
                spread_x(s / 2 + 2, kXAll);
                asm volatile("s_barrier" ::: "memory");
            }
        } else if constexpr (RB == 1) {
            if (p < 2) {
                // One row block: a stage is short, and what gates it is the chain load -> dequantize ->
                // write -> barrier of a single wave.  Waves 0 and 1 take the even and the odd stages and
                // spread the work of a stage over two stage slots (codes -> fp16 integers in registers
                // during the first, the FMAs and the LDS writes during the second), in antiphase: in every
                // slot one of them is in its first half and the other in its second.  Stage t is written
                // during stage t-2, like in the other roles.
                const uint32_t wlive = wvalid ? 0x7fffffffu : 0u;
                uint8_t* const wrow = smem + wdst;
                Dequant<B, HZ> dq;
                auto load_own = [&](int set, int t) {  // t: a stage of this wave (p, p + 2, ...)
                    load_w<B, GQ, HZ>(wr[set], make_rsrc(wsrc, t < k_stages ? wlive : 0u), t >> 2, t & 3, lane);
                };
                auto first_half = [&](int set) {
                    dq.start(wr[set]);
                    dq.insert();
                };
                auto second_half = [&](int t) {
                    uint8_t* dst = wrow + (uint32_t)t % kRing * T::WBytes;
#pragma unroll
                    for (int q = 0; q < 4; ++q) dq.emit(q, dst);
                };
                // prologue: this wave's first stage complete in the ring, its next four in the register sets;
                // wave 0 also has the first half of stage 2 done
#pragma unroll
                for (int i = 0; i < kSets; ++i) load_own(i, p + 2 * i);
                first_half(0);
                second_half(p);
                __builtin_amdgcn_sched_barrier(0);
                load_own(0, p + 2 * kSets);
                if (p == 0) {
                    first_half(1);
                    __builtin_amdgcn_sched_barrier(0);
                    load_own(1, 2 + 2 * kSets);
                }
                __builtin_amdgcn_sched_barrier(0);
                asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
                // slots t (even) and t + 1.  Wave 0: second half of stage t+2, then first half of t+4.
                // Wave 1: first half of stage t+3, then its second half.
                if (p == 0) {
                    for (int s = 0; s < n_stages; s += 2 * kSets) {
#pragma unroll
                        for (int u = 0; u < kSets; ++u) {
                            const int t = s + 2 * u;
                            second_half(t + 2);
                            __builtin_amdgcn_sched_barrier(0);
                            asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
                            first_half((u + 2) % kSets);  // stage t + 4, the wave's stage number t / 2 + 2
                            __builtin_amdgcn_sched_barrier(0);
                            load_own((u + 2) % kSets, t + 4 + 2 * kSets);
                            __builtin_amdgcn_sched_barrier(0);
                            asm volatile("s_barrier" ::: "memory");
                        }
                    }
                } else {
                    for (int s = 0; s < n_stages; s += 2 * kSets) {
#pragma unroll
                        for (int u = 0; u < kSets; ++u) {
                            const int t = s + 2 * u;
                            first_half((u + 1) % kSets);  // stage t + 3, the wave's stage number t / 2 + 1
                            __builtin_amdgcn_sched_barrier(0);
                            load_own((u + 1) % kSets, t + 3 + 2 * kSets);
                            __builtin_amdgcn_sched_barrier(0);
                            asm volatile("s_barrier" ::: "memory");
                            second_half(t + 3);
                            __builtin_amdgcn_sched_barrier(0);
                            asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
                        }
                    }
                }
            } else {  // wave 2 asks for the other rows of pairs 0 and 1, then only keeps the barriers
                load_x(0, kXAll, kXAll);
                __builtin_amdgcn_sched_barrier(0);
                load_x(1, kXAll, kXAll);
                asm volatile("s_waitcnt vmcnt(%0)" ::"n"(kXAll) : "memory");
                asm volatile("s_barrier" ::: "memory");
                asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
                for (int s = 0; s < n_stages; ++s) asm volatile("s_barrier" ::: "memory");
            }
        } else if (kSplitRoles) {
            load_wregs(0, 0);
            load_wregs(1, 1);
            load_wregs(2, 2);
            load_wregs(3, 3);
            w_to_lds(0, 0);
            w_to_lds(1, 1);
            __builtin_amdgcn_sched_barrier(0);
            load_wregs(0, 4);
            load_wregs(1, 5);
            __builtin_amdgcn_sched_barrier(0);
            asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
            for (int s = 0; s < n_stages; s += kSets) {
#pragma unroll
                for (int u = 0; u < kSets; ++u) {
                    w_to_lds((u + 2) % kSets, s + u + 2);
                    __builtin_amdgcn_sched_barrier(0);
                    load_wregs((u + 2) % kSets, s + u + 6);
                    __builtin_amdgcn_sched_barrier(0);
                    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
                }
            }
        } else {
            // prologue: stages 0 and 1 complete in the ring, activations of pair 1 on their way, weights
            // of stages 2..5 in the register sets 2, 3, 0, 1.  Of a pair this wave issues loads 8 p .. 8 p + 7.
            load_x(0, 8 * p, 8);
            __builtin_amdgcn_sched_barrier(0);  // (the wait below counts the requests behind these)
            load_wregs(0, 0);
            load_wregs(1, 1);
            load_wregs(2, 2);
            load_wregs(3, 3);
            w_to_lds(0, 0);
            w_to_lds(1, 1);
            __builtin_amdgcn_sched_barrier(0);
            asm volatile("s_waitcnt vmcnt(4)" ::: "memory");  // all but the weights of stages 2 and 3 (two loads each)
            load_x(1, 8 * p, 8);
            __builtin_amdgcn_sched_barrier(0);  // (and so does the loop's first)
            load_wregs(0, 4);
            load_wregs(1, 5);
            __builtin_amdgcn_sched_barrier(0);
            asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
            for (int s = 0; s < n_stages; s += kSets) {
#pragma unroll
                for (int u = 0; u < kSets; ++u) {
                    // a request ahead of each part of the vector work
                    Dequant<B, HZ> dq;
                    uint8_t* const wrow = smem + (uint32_t)(s + u + 2) % kRing * T::WBytes + wdst;
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        load_x((s + u) / 2 + 2, 8 * p + (u & 1) * 4 + j, 1, j & 1);
                        __builtin_amdgcn_sched_barrier(0);
                        if (j == 0) dq.start(wr[(u + 2) % kSets]);
                        else if (j == 1) dq.insert();
                        else dq.emit(2 * j - 4, wrow), dq.emit(2 * j - 3, wrow);
                        __builtin_amdgcn_sched_barrier(0);
                    }
                    load_wregs((u + 2) % kSets, s + u + 6);
                    __builtin_amdgcn_sched_barrier(0);
                    // even stages: younger than the activation loads of pair s/2 + 1: 2 weight loads of stage s-1, 4
                    // activation loads and 2 weight loads of stage s
                    if (u & 1) asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
                    else asm volatile("s_waitcnt vmcnt(8) lgkmcnt(0)\n\ts_barrier" ::: "memory");
                }
            }
        }
        // Loads of stages past the end (zero-sized sources: they write zeros) may still be on their way to
        // LDS, which the epilogue reuses: they must have landed before any wave passes the barrier below.
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    } else {
        // ---------------------------------------------------------------- consumer
        // MFMA operand addresses: lanes with h = 0 / 1 take the two 8-column groups of a 16-column step
        const int wfrag = (wm * RB * 32 + r) * kRowBytes + h * 16;
        // activation operand: token row wn * 64 + nb * 32 + r, chunk 4 (stage % 2) + 2j + h, kept at chunk ^ ((r >> 1) & 7)
        const int xrow = (wn * 64 + r) * (kStageK * 4);
        const int xchunk[2] = {xrow + ((h ^ ((r >> 1) & 7)) * 16), xrow + (((2 + h) ^ ((r >> 1) & 7)) * 16)};
        // Operand registers: one weight operand per 32-row block, reloaded for the next 16-column step
        // as soon as its two MFMAs are issued (so the read has the other blocks' MFMAs to land), and two
        // pairs of activation operands (this step's and the next one's).
        half8_t wf[RB], xf[2][2];
        auto read_w = [&](int mb, const uint8_t* stage, int j) {
            wf[mb] = *reinterpret_cast<const half8_t*>(stage + wfrag + mb * 32 * kRowBytes + j * 32);
        };
        // `pair`: LDS of the pair of stages, `odd`: 64 for its second stage
        auto read_x = [&](int set, const uint8_t* pair, int odd, int j) {
#pragma unroll
            for (int nb = 0; nb < 2; ++nb)
                xf[set][nb] = *reinterpret_cast<const half8_t*>(pair + (xchunk[j] ^ odd) + nb * 32 * (kStageK * 4));
        };
        int w_at = 0, x_at = kRing * T::WBytes;  // LDS of this stage's weights and of its pair's activations
        __syncthreads();
        read_x(0, smem + x_at, 0, 0);
#pragma unroll
        for (int mb = 0; mb < RB; ++mb) read_w(mb, smem + w_at, 0);
        for (int s = 0; s < k_stages; ++s) {
            const int odd = (s & 1) * 64;
            const int w_next = w_at == (kRing - 1) * T::WBytes ? 0 : w_at + T::WBytes;
            const int x_pair = x_at == kRing * T::WBytes + (kRing - 1) * T::XBytes ? kRing * T::WBytes : x_at + T::XBytes;
            const int x_next = odd ? x_pair : x_at;
            const uint8_t *w_cur = smem + w_at, *w_nxt = smem + w_next, *x_cur = smem + x_at, *x_nxt = smem + x_next;
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                // operands after this step: step 1 of this stage, or step 0 of stage s+1, which is complete
                // in the ring (past the last stage this reads stale LDS that is never used)
                read_x(j ^ 1, j == 0 ? x_cur : x_nxt, j == 0 ? odd : odd ^ 64, j ^ 1);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int mb = 0; mb < RB; ++mb) {
#pragma unroll
                    for (int nb = 0; nb < 2; ++nb)
                        acc[mb][nb] = __builtin_amdgcn_mfma_f32_32x32x16_f16(wf[mb], xf[j][nb], acc[mb][nb], 0, 0, 0);
                    __builtin_amdgcn_sched_barrier(0);
                    read_w(mb, j == 0 ? w_cur : w_nxt, j ^ 1);
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
            w_at = w_next;
            x_at = x_next;
            // Plain barrier: this wave has no LDS writes to publish, and its outstanding reads (stage
            // s+1) need not land before it; everything it read from stage s has been consumed.
            asm volatile("s_barrier" ::: "memory");
        }
        // the producers run a multiple of four stages; meet them at the barriers of the padding stages
        for (int s = k_stages; s < n_stages; ++s) asm volatile("s_barrier" ::: "memory");
    }

    // epilogue: accumulators -> fp16 -> LDS as [token][row] -> coalesced 16-byte stores
    // C[i][j] of a 32x32 block: i = row (8 * (v / 4) + 4 * h + v % 4), j = token (lane % 32)
    // One more barrier between the last stage and the epilogue: the consumers leave the last stage barrier
    // while activation loads of the padding stages, issued by the producers, can still be writing to the ring.
    __syncthreads();
    uint8_t* otile = smem;  // the stage buffers are free now
    if (wave < kConsumerWaves) {
#pragma unroll
        for (int mb = 0; mb < RB; ++mb)
#pragma unroll
            for (int nb = 0; nb < 2; ++nb) {
                uint8_t* col = otile + (wn * 64 + nb * 32 + r) * T::OutRow + ((wm * RB + mb) * 32 + 4 * h) * 2;
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    half2_t lo, hi;
                    lo.x = (_Float16)acc[mb][nb][4 * g + 0];
                    lo.y = (_Float16)acc[mb][nb][4 * g + 1];
                    hi.x = (_Float16)acc[mb][nb][4 * g + 2];
                    hi.y = (_Float16)acc[mb][nb][4 * g + 3];
                    u32x2 w = {__builtin_bit_cast(uint32_t, lo), __builtin_bit_cast(uint32_t, hi)};
                    *reinterpret_cast<u32x2*>(col + g * 16) = w;  // rows 8g + 4h + 0..3
                }
            }
    }
    __syncthreads();
    store_tile<T::TM, kTN, T::OutRow, kThreads>(a.y, a.M, a.N, otile, mt * T::TM, n0, tid);
}

// ---------------------------------------------------------------------------------------------
// Grids that would otherwise leave compute units idle: the W waves of a workgroup split K.  Wave w takes the 64-column
// stages w, w + W, ... whole: it dequantizes the stage's weights in registers, brings the stage's activations into its own LDS buffers and multiplies
// them with all tokens of the tile.  So a weight is dequantized once per tile, no weight goes through LDS, a wave reads
// 0.5 KB of LDS per MFMA instead of 1.5 KB, and the waves never wait for one another until the end, where their
// partial tiles meet in LDS (added in wave order: results do not depend on timing).
// Shapes of the tile (RBW row blocks x 32 TT tokens): 64 rows x 64 tokens with four waves (two workgroups share a
// compute unit) or eight, 64 x 128, 128 x 128 (every wave dequantizes two row blocks per stage and needs half the
// activation bytes per MFMA), and 64 x 256 where the tiling asks for it.  What bounds a wave is the sum of its
// dequantization (about 90 vector instructions per row unit and stage, of which about 6 hide behind an MFMA) and its MFMAs
// (four of 32 cycles per row unit, stage and 32 tokens): a narrow tile costs more dequantization per token
// but spreads the work over more units and multiplies less padding.
//
// A stage is 64 columns, 128 bytes of a token: whole cache lines (with 64 bytes of a line per request every line came into the
// unit's L1 twice).  Lane (r, h) of a row unit (32 rows) takes block h of the stage's two 32-column blocks of row r, which it
// loads and dequantizes alone; a product then sums over 8 columns of each block, and the activations are read to match, so no
// lane exchanges anything.  With 32-column stages and the operands made by exchanges: 4096 x 11008 N = 173 32.1 us, now 28.1; 11008 x
// 4096 N = 64 / 128 20.2 / 30.3, now 17.3 / 23.9.
constexpr int kKsStageK = 64;
template <int RBW, int TT, int W>
struct KsTile {
    static constexpr int TN = 32 * TT, TM = 64 * RBW;
    static constexpr int XBytes = TN * kKsStageK * 2;         // activations of a stage
    static constexpr int NBuf = 128 * 1024 / (W * XBytes) < 2 ? 1 : 2;  // activation buffers per wave
    static constexpr int XLoads = TN / 8;                     // requests per stage (8 token rows each)
    static constexpr int PartRow = TM * 4 + 16;               // bytes per token of a wave's partial tile in LDS
    static constexpr int PartBytes = (TN / 2) * PartRow;      // ... of half of its tokens
    static constexpr int LdsBytes = W * NBuf * XBytes > W * PartBytes ? W * NBuf * XBytes : W * PartBytes;
    static_assert(TT % 2 == 0 && RBW * TT <= 8 && LdsBytes <= 160 * 1024, "tile of the K-split kernel");
};

// Loads the lane's block of stage t of 32 rows (see load_w for `rw`); `row` is the lane's row in its row block.
template <int B, int GQ, bool HZ>
__device__ __forceinline__ void load_w_block(WRegs<B>& r, rsrc_t rw, int t, int row, int h) {
    constexpr int MSZ = HZ ? 4 : 2;
    constexpr int MPL = (kKTile / GQ) * MSZ;
    constexpr int TB = B * 1024 + 64 * MPL;
    const int so = (t >> 1) * TB, v = t & 1;  // block 2 v + h of the tile
    if constexpr (B == 4) {
        const u32x4 w = __builtin_amdgcn_raw_buffer_load_b128(rw, row * 16 + h * 1024, so + v * 2048, 0);
        r.plane[0] = w.x; r.plane[1] = w.y; r.plane[2] = w.z; r.plane[3] = w.w;
    } else if constexpr (B == 2) {
        const u32x2 w = __builtin_amdgcn_raw_buffer_load_b64(rw, row * 16 + h * 8, so + v * 1024, 0);
        r.plane[0] = w.x; r.plane[1] = w.y;
    } else {
        r.plane[0] = __builtin_amdgcn_raw_buffer_load_b32(rw, row * 16 + h * 4, so + v * 8, 0);
    }
    const int mv = row * MPL + (GQ == 32 ? h * MSZ : 0), mo = so + B * 1024 + v * 64 / GQ * MSZ;
    if constexpr (HZ) r.meta = __builtin_amdgcn_raw_buffer_load_b32(rw, mv, mo, 0);
    else r.meta = __builtin_amdgcn_raw_buffer_load_b16(rw, mv, mo, 0);
}

template <int B, int GQ, bool HZ, int RBW, int TT, int W, typename... Fields>
__global__ void __launch_bounds__(64 * W, 1) mpgemm_ksplit_kernel(Fields... fields) {
    const GemmArgs a{fields...};
    const int n_ktiles = (a.K + kKTile - 1) / kKTile;
    using T = KsTile<RBW, TT, W>;
    constexpr int kUnits = 2 * RBW;  // row units of the tile
    constexpr int MSZ = HZ ? 4 : 2;
    constexpr int TB = B * 1024 + 64 * (kKTile / GQ) * MSZ;
    extern __shared__ __attribute__((aligned(16))) uint8_t smem[];

    int mt, nt;
    tile_of_workgroup(a, mt, nt);
    const bool header_ok = header_matches(a.tiles, a.M, a.K, B, GQ, HZ ? 1 : 0);
    if (!header_ok && blockIdx.x == 0 && threadIdx.x == 0) report_header_mismatch(a.status);
    if (mt >= (header_ok ? a.m_tiles : 0)) return;

    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int n0 = nt * T::TN;
    const int k_stages = (a.K + kKsStageK - 1) / kKsStageK;
    // own stages of this wave: wave, wave + W, ...; the loop runs an even number of them (a stage past K has empty
    // sources: zero weights, zero activations)
    const int n_own = (k_stages + W - 1) / W, n_own_pad = (n_own + 1) & ~1;
    const int r = lane & 31, h = lane >> 5;

    float16_t acc[RBW][2][TT];
#pragma unroll
    for (int b = 0; b < RBW; ++b)
#pragma unroll
        for (int hb = 0; hb < 2; ++hb)
#pragma unroll
            for (int nb = 0; nb < TT; ++nb)
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[b][hb][nb][v] = 0.f;

    WRegs<B> wr[2][kUnits];
    auto load_unit = [&](int set, int unit, int i) {  // own stage i = stage W i + wave
        const int t = W * i + wave, rb = mt * RBW + unit / 2;
        const bool wvalid = rb < a.n_row_blocks;
        const uint8_t* wsrc = a.tiles + (size_t)(wvalid ? rb : 0) * n_ktiles * TB;
        load_w_block<B, GQ, HZ>(wr[set][unit], make_rsrc(wsrc, t < k_stages && wvalid ? 0x7fffffffu : 0u), t, (unit & 1) * 32 + r, h);
    };
    // Activations of own stage i go to this wave's buffer i % NBuf.  A request brings 8 token rows of 128 bytes; 16-byte chunk c
    // of row R is kept at place c ^ ((R >> 1) & 7): the operand reads of 16 consecutive rows fall on 16 different places.
    // Columns beyond K (blocks of 32 only) have weights of zero and are sent past the end of the resource, where they read as zero.
    const int xrows = a.N - n0 < T::TN ? a.N - n0 : T::TN;
    const _Float16* xsrc = a.x + (size_t)n0 * a.K;
    const uint32_t xbytes = (uint32_t)xrows * (uint32_t)a.K * 2u;
    const uint32_t xlane = (uint32_t)(lane >> 3) * (uint32_t)a.K * 2u, x8rows = 8u * (uint32_t)a.K * 2u;
    const uint32_t xchunk[2] = {(uint32_t)((lane & 7) ^ (lane >> 4)) * 16u, (uint32_t)((lane & 7) ^ (4 + (lane >> 4))) * 16u};
    uint8_t* const xbuf = smem + wave * T::NBuf * T::XBytes;
    auto load_x = [&](int i, int from = 0, int to = T::XLoads) {
        const int t = W * i + wave;
        const rsrc_t rx = make_rsrc(xsrc, t < k_stages ? xbytes : 0u);
        uint8_t* dst = xbuf + (i & (T::NBuf - 1)) * T::XBytes;
#pragma unroll
        for (int q = from; q < to; ++q) {
            uint32_t off = xlane + (uint32_t)q * x8rows + xchunk[q & 1];
            if constexpr (GQ == 32) off = t * kKsStageK + (int)(xchunk[q & 1] / 2) < a.K ? off : 0xFFFFFF00u;
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rx, (__attribute__((address_space(3))) void*)(dst + q * 1024), 16, off,
                                                     t * kKsStageK * 2, 0, 0);
        }
    };
    // operand of step j: columns 8 j .. 8 j + 7 of the lane's block, chunk 4 h + j
    int xoff[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) xoff[j] = r * (kKsStageK * 2) + ((4 * h + j) ^ ((r >> 1) & 7)) * 16;
    half8_t xf[4][TT];
    auto read_x = [&](int j, const uint8_t* stage) {
#pragma unroll
        for (int nb = 0; nb < TT; ++nb)
            xf[j][nb] = *reinterpret_cast<const half8_t*>(stage + xoff[j] + nb * 32 * (kKsStageK * 2));
    };
    half8_t wf[2][4];  // [unit % 2][step]
    Dequant<B, HZ> dq;
    // the vector work of a row unit in four parts, one beside each step of the unit before it
    auto dequant_part = [&](int j, int set, int unit) {
        if (j == 0) {
            dq.start(wr[set][unit]);
        } else if (j == 1) {
            dq.insert();
        } else {
#pragma unroll
            for (int q = 2 * j - 4; q < 2 * j - 2; ++q) wf[unit & 1][q] = __builtin_bit_cast(half8_t, dq.piece(q));
        }
    };

    // prologue: weights of own stages 0 and 1 and activations requested, the first row unit dequantized, the first activations
    // in registers.  The wait below counts the requests, so none may be moved past another group.
#pragma unroll
    for (int u = 0; u < kUnits; ++u) load_unit(0, u, 0);
    __builtin_amdgcn_sched_barrier(0);
    load_x(0);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int u = 0; u < kUnits; ++u) load_unit(1, u, 1);
#pragma unroll
    for (int j = 0; j < 4; ++j) dequant_part(j, 0, 0);
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (T::NBuf == 2) {
        load_x(1);
        __builtin_amdgcn_sched_barrier(0);
    }
    load_unit(0, 0, 2);
    __builtin_amdgcn_sched_barrier(0);
    // activations of own stage 0: younger are the requests of own stage 1 and unit 0 of own stage 2
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(2 * kUnits + (T::NBuf - 1) * T::XLoads + 2) : "memory");
#pragma unroll
    for (int j = 0; j < 4; ++j) read_x(j, xbuf);

    // The activations of an own stage are in registers when unit 0 has used them: the next but one are requested then.  Four units:
    // spread over unit 1 (5367 x 5504 N = 580 52.7 -> 51.6 us).  Two: at once, the wait for the next stage's is close (spread: 2 to
    // 5 % slower).
    constexpr bool kSpread = T::NBuf == 2 && kUnits > 2;
    for (int i0 = 0; i0 < n_own_pad; i0 += 2) {
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            const int i = i0 + s;
            const uint8_t* nxt = xbuf + ((i + 1) & (T::NBuf - 1)) * T::XBytes;
            if constexpr (T::NBuf == 1) {  // the only buffer is free when its activations are in registers
                asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
                load_x(i + 1);
                __builtin_amdgcn_sched_barrier(0);
            }
#pragma unroll
            for (int u = 0; u < kUnits; ++u) {
                constexpr int kLast = kUnits - 1;
                const int nu = u == kLast ? 0 : u + 1, nset = u == kLast ? (s + 1) & 1 : s;
                if (u == kLast) {
                    // The activations of own stage i + 1 must be in.  Younger: NBuf == 2 (requested behind unit 0 of the previous
                    // own stage or beside its unit 1): at least its weights from then on, the weights of this stage and the
                    // activations of stage i + 2; NBuf == 1 (requested above): the weights of this stage.
                    constexpr int kYounger = T::NBuf == 2 ? 2 * kUnits + T::XLoads : 2 * (kUnits - 1);
                    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(kYounger) : "memory");
                }
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    if (kSpread && u == 1) {
                        load_x(i + 2, j * T::XLoads / 4, (j + 1) * T::XLoads / 4);
                        __builtin_amdgcn_sched_barrier(0);
                    }
                    dequant_part(j, nset, nu);
#pragma unroll
                    for (int nb = 0; nb < TT; ++nb)
                        acc[u / 2][u & 1][nb] = __builtin_amdgcn_mfma_f32_32x32x16_f16(wf[u & 1][j], xf[j][nb], acc[u / 2][u & 1][nb], 0, 0, 0);
                    if (u == kLast) read_x(j, nxt);
#pragma unroll
                    for (int q = 0; q < TT; ++q) {
                        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                        __builtin_amdgcn_sched_group_barrier(0x002, 24 / TT, 0);
                        if (u == kLast) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
                    }
                    __builtin_amdgcn_sched_barrier(0);
                }
                // the registers of the row unit just dequantized are free
                load_unit(nset, nu, (u == kLast ? i + 1 : i) + 2);
                __builtin_amdgcn_sched_barrier(0);
                if (T::NBuf == 2 && !kSpread && u == 0) {
                    load_x(i + 2);
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
        }
    }
    // requests of own stages past the end may still be writing zeros to LDS, which the partial tiles reuse
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();

    // The four partial tiles meet in LDS, half of the tokens at a time: wave w writes its fp32 sums as
    // [token][row], then thread -> (token, 8 rows) adds the four in wave order and stores fp16.
    // acc[b][hb][nb][v] is row 64 b + 32 hb + 8 (v / 4) + 4 h + v % 4 for token 32 nb + r.
    const int m0 = mt * T::TM;
    const bool fast = a.M % 8 == 0 && aligned16(a.y);  // 16-byte aligned rows of y
#pragma unroll
    for (int half = 0; half < 2; ++half) {
        uint8_t* mine = smem + wave * T::PartBytes;
#pragma unroll
        for (int nq = 0; nq < TT / 2; ++nq) {
            const int nb = half * (TT / 2) + nq;
#pragma unroll
            for (int b = 0; b < RBW; ++b)
#pragma unroll
                for (int hb = 0; hb < 2; ++hb)
#pragma unroll
                    for (int g = 0; g < 4; ++g) {
                        float* dst = reinterpret_cast<float*>(mine + (nq * 32 + r) * T::PartRow + (64 * b + 32 * hb + 8 * g + 4 * h) * 4);
#pragma unroll
                        for (int e = 0; e < 4; ++e) dst[e] = acc[b][hb][nb][4 * g + e];
                    }
        }
        __syncthreads();
        if (!fast) {  // (rows of y start anywhere: consecutive lanes take consecutive rows; eight of a lane before, 2119 x 2240 2 bits N = 648 17.8 -> 16.1 us)
            const int live = a.N - n0 - half * (T::TN / 2);
#pragma unroll 2
            for (int i = tid; i < (live < T::TN / 2 ? live : T::TN / 2) * T::TM; i += 64 * W) {
                const int n = i / T::TM, row = i % T::TM;
                float sum = 0.f;
#pragma unroll
                for (int w = 0; w < W; ++w) sum += *reinterpret_cast<const float*>(smem + w * T::PartBytes + n * T::PartRow + row * 4);
                if (m0 + row < a.M) a.y[(size_t)(n0 + half * (T::TN / 2) + n) * a.M + m0 + row] = (_Float16)sum;
            }
            __syncthreads();
            continue;
        }
        for (int piece = tid; piece < (T::TN / 2) * (T::TM / 8); piece += 64 * W) {
            const int n = piece / (T::TM / 8), c8 = piece % (T::TM / 8);
            const int gn = n0 + half * (T::TN / 2) + n, gm = m0 + c8 * 8;
            float sum[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) sum[e] = 0.f;
#pragma unroll
            for (int w = 0; w < W; ++w) {
                const float* src = reinterpret_cast<const float*>(smem + w * T::PartBytes + n * T::PartRow + c8 * 32);
#pragma unroll
                for (int e = 0; e < 8; ++e) sum[e] += src[e];
            }
            if (gn >= a.N || gm >= a.M) continue;
            half8_t o;
#pragma unroll
            for (int e = 0; e < 8; ++e) o[e] = (_Float16)sum[e];
            *reinterpret_cast<half8_t*>(a.y + (size_t)gn * a.M + gm) = o;  // (M is a multiple of 8)
        }
        __syncthreads();
    }
}

// ---------------------------------------------------------------------------------------------
// Grids that fill the chip with 256-row workgroups: no weight tile in LDS, no producer waves.  A wave owns 64 rows x 32 TT
// tokens and dequantizes its own weights in registers, block by block per lane as in the K-split kernel; the activations of a
// 64-column stage (whole cache lines) are shared by the four waves through LDS.  Two workgroups share a compute unit.
// 96 tokens: with 128 the accumulators, the activations of a stage and the weights in flight do not fit 256 registers.
// What bounds it: products plus vector work at the clock the chip holds under both (8 vector instructions per product, about 6
// hide behind one).  11008 x 4096 4 bits, N = 1024 / 2048: 101 / 194 us = 0.92 / 0.95 PFLOP/s (tiled, 192 x 256, timed in turn with
// it: 95 / 181); its grain is half as large.
constexpr int kWideRing = 4;   // stage buffers
constexpr int kWideRows = 256;
template <int TT>
struct WideTile {
    static_assert(TT <= 4, "a request a step");
    static constexpr int TN = 32 * TT;
    static constexpr int XBytes = TN * kKsStageK * 2;
    static constexpr int XLoads = TT;                  // requests of a stage per wave (8 token rows each)
    static constexpr int OutRow = kWideRows * 2 + 16;  // bytes per token of the output tile in LDS
    static constexpr int LdsBytes = kWideRing * XBytes > TN * OutRow ? kWideRing * XBytes : TN * OutRow;
};

template <int B, int GQ, bool HZ, int TT, typename... Fields>
__global__ void __launch_bounds__(256, 2) mpgemm_wide_kernel(Fields... fields) {
    const GemmArgs a{fields...};
    const int n_ktiles = (a.K + kKTile - 1) / kKTile;
    using T = WideTile<TT>;
    constexpr int MSZ = HZ ? 4 : 2;
    constexpr int TB = B * 1024 + 64 * (kKTile / GQ) * MSZ;
    extern __shared__ __attribute__((aligned(16))) uint8_t smem[];

    int mt, nt;
    tile_of_workgroup(a, mt, nt);
    const bool header_ok = header_matches(a.tiles, a.M, a.K, B, GQ, HZ ? 1 : 0);
    if (!header_ok && blockIdx.x == 0 && threadIdx.x == 0) report_header_mismatch(a.status);
    if (mt >= (header_ok ? a.m_tiles : 0)) return;

    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int n0 = nt * T::TN;
    // the loop runs an even number of stages (a stage past K has empty sources: zero weights, zero activations)
    const int k_stages = (a.K + kKsStageK - 1) / kKsStageK, n_stages = (k_stages + 1) & ~1;
    const int r = lane & 31, h = lane >> 5;

    float16_t acc[2][TT];
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int nb = 0; nb < TT; ++nb)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[u][nb][v] = 0.f;

    const int rb = mt * 4 + wave;
    const bool wvalid = rb < a.n_row_blocks;
    const uint8_t* wsrc = a.tiles + (size_t)(wvalid ? rb : 0) * n_ktiles * TB;
    WRegs<B> wr[2][2];  // [set][row unit]
    auto load_unit = [&](int set, int unit, int t) {
        load_w_block<B, GQ, HZ>(wr[set][unit], make_rsrc(wsrc, t < k_stages && wvalid ? 0x7fffffffu : 0u), t, unit * 32 + r, h);
    };
    // activations: wave w issues requests w, w + 4, ... of a stage; chunks placed as in the K-split kernel
    const int xrows = a.N - n0 < T::TN ? a.N - n0 : T::TN;
    const _Float16* xsrc = a.x + (size_t)n0 * a.K;
    const uint32_t xbytes = (uint32_t)xrows * (uint32_t)a.K * 2u;
    const uint32_t xchunk = (uint32_t)((lane & 7) ^ ((wave & 1) * 4 + (lane >> 4))) * 16u;
    const uint32_t xlane = (uint32_t)(wave * 8 + (lane >> 3)) * (uint32_t)a.K * 2u + xchunk, x32rows = 32u * (uint32_t)a.K * 2u;
    auto load_x = [&](int t, int from = 0, int to = T::XLoads) {
        const rsrc_t rx = make_rsrc(xsrc, t < k_stages ? xbytes : 0u);
        uint8_t* dst = smem + (t & (kWideRing - 1)) * T::XBytes;
#pragma unroll
        for (int i = from; i < to; ++i) {
            uint32_t off = xlane + (uint32_t)i * x32rows;
            if constexpr (GQ == 32) off = t * kKsStageK + (int)(xchunk / 2) < a.K ? off : 0xFFFFFF00u;
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rx, (__attribute__((address_space(3))) void*)(dst + (wave + 4 * i) * 1024), 16, off,
                                                     t * kKsStageK * 2, 0, 0);
        }
    };
    int xoff[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) xoff[j] = r * (kKsStageK * 2) + ((4 * h + j) ^ ((r >> 1) & 7)) * 16;
    half8_t xf[4][TT];
    auto read_x = [&](int j, const uint8_t* stage) {
#pragma unroll
        for (int nb = 0; nb < TT; ++nb)
            xf[j][nb] = *reinterpret_cast<const half8_t*>(stage + xoff[j] + nb * 32 * (kKsStageK * 2));
    };
    half8_t wf[2][4];  // [row unit][step]
    Dequant<B, HZ> dq;
    auto dequant_part = [&](int j, int set, int unit) {
        if (j == 0) {
            dq.start(wr[set][unit]);
        } else if (j == 1) {
            dq.insert();
        } else {
#pragma unroll
            for (int q = 2 * j - 4; q < 2 * j - 2; ++q) wf[unit][q] = __builtin_bit_cast(half8_t, dq.piece(q));
        }
    };

    // Requests in the order of the loop, whose waits count them: per stage the activations of stage s + 3, the weights of row
    // unit 1 of stage s + 2 and of unit 0 of stage s + 3.
    load_unit(0, 0, 0);
    load_unit(0, 1, 0);
    load_unit(1, 0, 1);
    __builtin_amdgcn_sched_barrier(0);
    load_x(0);
    load_x(1);
    __builtin_amdgcn_sched_barrier(0);
    load_x(2);
    __builtin_amdgcn_sched_barrier(0);
    load_unit(1, 1, 1);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int j = 0; j < 4; ++j) dequant_part(j, 0, 0);
    __builtin_amdgcn_sched_barrier(0);
    load_unit(0, 0, 2);
    __builtin_amdgcn_sched_barrier(0);
    // the activations of stages 0 and 1 are in
    asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"(T::XLoads + 4) : "memory");
#pragma unroll
    for (int j = 0; j < 4; ++j) read_x(j, smem);

    for (int s0 = 0; s0 < n_stages; s0 += 2) {
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            const int t = s0 + s;
            const uint8_t* nxt = smem + ((t + 1) & (kWideRing - 1)) * T::XBytes;
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                // the products of row unit u; meanwhile the vector work of the next unit, and beside the last one the activations
                // of stage t + 1, each as soon as its registers are used
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    if (u == 0 && j < T::XLoads) {  // (one request a step: in one go they keep the other waves waiting)
                        load_x(t + 3, j, j + 1);
                        __builtin_amdgcn_sched_barrier(0);
                    }
                    dequant_part(j, u ? (s + 1) & 1 : s, u ^ 1);
#pragma unroll
                    for (int nb = 0; nb < TT; ++nb)
                        acc[u][nb] = __builtin_amdgcn_mfma_f32_32x32x16_f16(wf[u][j], xf[j][nb], acc[u][nb], 0, 0, 0);
                    if (u == 1) read_x(j, nxt);
#pragma unroll
                    for (int q = 0; q < TT; ++q) {
                        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                        __builtin_amdgcn_sched_group_barrier(0x002, (24 + TT - 1) / TT, 0);
                        if (u == 1) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
                    }
                    __builtin_amdgcn_sched_barrier(0);
                }
                if (u == 0) load_unit(s, 1, t + 2);
                else load_unit((s + 1) & 1, 0, t + 3);
                __builtin_amdgcn_sched_barrier(0);
            }
            // the activations of stage t + 2 (requested one stage ago) are in before any wave goes on: younger are the weights
            // requested then and what this stage requested
            asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"(T::XLoads + 8) : "memory");
        }
    }
    // requests of stages past the end may still be writing zeros to the ring, which the output tile reuses
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();

    // epilogue: C[i][j] of a 32 x 32 tile: i = row 8 (v / 4) + 4 h + v % 4, j = token lane % 32
    uint8_t* otile = smem;
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int nb = 0; nb < TT; ++nb) {
            uint8_t* col = otile + (nb * 32 + r) * T::OutRow + (wave * 64 + u * 32 + 4 * h) * 2;
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                half2_t lo, hi;
                lo.x = (_Float16)acc[u][nb][4 * g + 0];
                lo.y = (_Float16)acc[u][nb][4 * g + 1];
                hi.x = (_Float16)acc[u][nb][4 * g + 2];
                hi.y = (_Float16)acc[u][nb][4 * g + 3];
                u32x2 w = {__builtin_bit_cast(uint32_t, lo), __builtin_bit_cast(uint32_t, hi)};
                *reinterpret_cast<u32x2*>(col + g * 16) = w;  // rows 8g + 4h + 0..3
            }
        }
    __syncthreads();
    store_tile<kWideRows, T::TN, T::OutRow, 256>(a.y, a.M, a.N, otile, mt * kWideRows, n0, tid);
}

static int compute_units() {
    static std::once_flag once;
    static int n_cu = 256;  // assumed when no device answers
    std::call_once(once, [] {
        int dev = 0, n = 0;
        if (hipGetDevice(&dev) == hipSuccess &&
            hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && n > 0)
            n_cu = n;
    });
    return n_cu;
}

// Equal runs of tiles per XCD (K-split kernel: always).  Tiled kernel: whole row tiles where that costs an XCD no further round
// of workgroups over its units, and leaves it at most 5 % more of them, or there are so few row tiles that the cuts are what
// costs.  11008 x 4096, 58 row tiles x 4 token tiles, 32 or 29 per XCD: 98.9 us whole, 96.8 in runs (N = 2048, 64 or 58:
// 192.9 / 189.4); 2112 x 4096, N = 2048, 17 x 8, weights in cache: 60.9 / 63.0; 6912 x 2560, N = 777, 54 x 4, 28 or 27: 46.4 /
// 47.8; 24 x 8 (3072 x 8192, N = 2048), 24 per XCD in both: 129.5 / 131.5; 2112 x 4096, N = 3072, 17 x 12, 36 or 26 for 32
// units: 70 / 38.
static unsigned deal_tiles(GemmArgs& a, bool may_be_whole) {
    const long long whole = (long long)((a.m_tiles + kXcds - 1) / kXcds) * a.n_tiles;
    const long long even = ((long long)a.m_tiles * a.n_tiles + kXcds - 1) / kXcds;
    const int units = compute_units() / kXcds > 0 ? compute_units() / kXcds : 1;
    const bool same_rounds = (whole + units - 1) / units == (even + units - 1) / units;
    a.whole_row_tiles = may_be_whole && same_rounds && (whole * 20 <= even * 21 || (a.m_tiles >= kXcds && a.m_tiles < 18));
    a.per_xcd = (int)(a.whole_row_tiles ? whole : even);
    return (unsigned)a.per_xcd * kXcds;
}

template <int B, int GQ, bool HZ, int RBW, int TT, int W>
static int launch_ksplit(GemmArgs a, hipStream_t st) {
    using T = KsTile<RBW, TT, W>;
    static std::once_flag once;
    static hipError_t attr_rc = hipSuccess;
    a.m_tiles = (a.n_row_blocks + RBW - 1) / RBW;
    a.n_tiles = (a.N + T::TN - 1) / T::TN;
    const unsigned grid = deal_tiles(a, false);
    return with_fields(a, [&](auto... f) {
        return launch_with_lds<T::LdsBytes>(&mpgemm_ksplit_kernel<B, GQ, HZ, RBW, TT, W, decltype(f)...>, once, attr_rc, grid, 64 * W, st, f...);
    });
}

template <int B, int GQ, bool HZ, int TT>
static int launch_wide(GemmArgs a, hipStream_t st) {
    using T = WideTile<TT>;
    static std::once_flag once;
    static hipError_t attr_rc = hipSuccess;
    a.m_tiles = (a.n_row_blocks + 3) / 4;
    a.n_tiles = (a.N + T::TN - 1) / T::TN;
    const unsigned grid = deal_tiles(a, false);
    return with_fields(a, [&](auto... f) {
        return launch_with_lds<T::LdsBytes>(&mpgemm_wide_kernel<B, GQ, HZ, TT, decltype(f)...>, once, attr_rc, grid, 256, st, f...);
    });
}

template <int B, int GQ, bool HZ, int RB>
static int launch_tile(GemmArgs a, hipStream_t st) {
    static std::once_flag once;
    static hipError_t attr_rc = hipSuccess;
    a.m_tiles = (a.n_row_blocks + RB - 1) / RB;
    a.n_tiles = (a.N + kTN - 1) / kTN;
    const unsigned grid = deal_tiles(a, true);
    return with_fields(a, [&](auto... f) {
        return launch_with_lds<Tile<RB>::LdsBytes>(&mpgemm_kernel<B, GQ, HZ, RB, decltype(f)...>, once, attr_rc, grid, kThreads, st, f...);
    });
}

// Which kernel and tile: 1 .. 4 = the tiled kernel with that many row blocks per workgroup; kWide = the kernel without a weight
// tile, 256 rows x 96 tokens; the others = the K-split kernel with 64 rows x 256 tokens, 128 x 128, 64 x 128, and 64 x 64
// (four or eight waves).
//
// The choice models the time of the grid each of them gives, in microseconds on 256 units: rounds of workgroups over the units,
// each a fixed part (prologue, exchange of the partial sums) and a part in proportion to K.  A last round that leaves units
// idle takes less, because the clock is higher then: a share `alone` with few workgroups, the whole with all units busy.
// Measured (64 / 128 / 192 / 256 / 320 / 512 / 768 workgroups, K = 4096, 4 bits, blocks of 64):
//   tiled, 256 x 256   90 / 93 / 110
//   tiled, 192 x 256   73 / 79 / 90 / 106 / 175 / 214        K-split, 128 x 128   30 / 33 / 37 / 43 / 68 / 83 / 122
//   tiled, 128 x 256   61 / 61 / 68 / 83 / 139 / 162 / 242   K-split, 64 x 128    19 / 20 / 22 / 26 / 41 / 51 / 74
//   tiled, 64 x 256    38 / 40 / 42 / 49 / 85 / 100 / 146    K-split, 64 x 64     14 / 15 / 15 / 16 / 24 / 30 / 43
//   wide, 256 x 96     50 / 52 / 55 / 64 / 92 / 115 / 173    ... eight waves      14 / 15 / 15 / 18 / 29 / 36 / 52
// So short prompts, whose 256-token tiles are mostly padding, and grids that leave units idle go to the narrow tiles, large grids
// to 192 x 256 or, where its rounds fit better, to the wide kernel (12288 x 4096, N = 1500: 175 us tiled, 161 wide; 9000 x 2048
// 2 bits, N = 1300: 80 and 54; 256 x 256 tiles 58).  64 x 256 of the K-split kernel is only taken where the tiling asks for it.  Eight waves for 64 x 64 pay from a K of 8192 on (11008: 29.1 / 29.7 / 32.0 / 37.9 us
// against 30.4 / 32.0 / 33.4 / 38.3).
constexpr int kSplitWide = 5, kSplitTall = 6, kSplit128 = 7, kSplit64 = 8, kSplit64x8 = 9, kWide = 10;
static int choose_tile(int n_row_blocks, int N, int K) {
    const int n_cu = compute_units();
    const tman_tiling_t t = current_tiling();
    if (t.prefill_k_split == 2) return kSplitWide;
    if (t.prefill_k_split == 3) return kSplitTall;
    const int forced = t.prefill_row_blocks;
    if (forced >= 1 && forced <= 4) return forced;
    const double k = K / 4096.0;
    int best = 3;
    double best_cost = 1e30;
    auto consider = [&](int choice, int rows, int tokens, double fixed, double per_k, double alone) {
        const long long wgs = (long long)((n_row_blocks + rows - 1) / rows) * ((N + tokens - 1) / tokens);
        const double full = (double)(wgs / n_cu), rest = (double)(wgs % n_cu) / n_cu;
        const double part = rest > 0 ? alone + (1.0 - alone) * rest * rest : 0.0;
        const double cost = (full + (rest > 0)) * fixed + (full + part) * per_k * k;
        if (cost < best_cost) best_cost = cost, best = choice;
    };
    consider(3, 3, kTN, 4.5, 99.0, 0.67);
    consider(4, 4, kTN, 5.0, 130.0, 0.64);
    consider(2, 2, kTN, 3.5, 75.0, 0.71);
    consider(1, 1, kTN, 2.0, 45.0, 0.73);
    consider(kWide, 4, 96, 3.0, 54.0, 0.72);
    // (Short K has little to split, but the 64 x 64 kernel would still be the fastest for most short prompts from about 128 columns on:
    // forced, 832 x 224 N = 145 6.0 -> 5.1 us, 64 x 512 N = 614 7.8 -> 5.0; 22388 x 32 N = 52 7.8 -> 9.0.)
    if (t.prefill_k_split == 1 || K <= 512) return best;
    consider(kSplitTall, 2, 128, 5.5, 34.6, 0.64);
    consider(kSplit128, 1, 128, 5.0, 18.7, 0.68);
    consider(kSplit64, 1, 64, 2.0, 11.8, 0.75);
    const long long wgs64 = (long long)n_row_blocks * ((N + 63) / 64);
    return best == kSplit64 && wgs64 <= n_cu && K >= 8192 ? kSplit64x8 : best;
}

template <int B, int GQ, bool HZ>
static int launch_cfg(const GemmArgs& a, hipStream_t st) {
    switch (choose_tile(a.n_row_blocks, a.N, a.K)) {
        case kSplitWide: return launch_ksplit<B, GQ, HZ, 1, 8, 4>(a, st);
        case kSplitTall: return launch_ksplit<B, GQ, HZ, 2, 4, 4>(a, st);
        case kSplit128: return launch_ksplit<B, GQ, HZ, 1, 4, 4>(a, st);
        case kSplit64: return launch_ksplit<B, GQ, HZ, 1, 2, 4>(a, st);
        case kSplit64x8: return launch_ksplit<B, GQ, HZ, 1, 2, 8>(a, st);
        case kWide: return launch_wide<B, GQ, HZ, 3>(a, st);
        case 1: return launch_tile<B, GQ, HZ, 1>(a, st);
        case 2: return launch_tile<B, GQ, HZ, 2>(a, st);
        case 3: return launch_tile<B, GQ, HZ, 3>(a, st);
        default: return launch_tile<B, GQ, HZ, 4>(a, st);
    }
}

template <int B, bool HZ>
static int launch_group(int group, const GemmArgs& a, hipStream_t st) {
    switch (group) {
        case 32: return launch_cfg<B, 32, HZ>(a, st);
        case 64: return launch_cfg<B, 64, HZ>(a, st);
        default: return launch_cfg<B, 128, HZ>(a, st);
    }
}

int mpgemm_row_blocks_per_workgroup(const Layout& L, int N) {
    const int c = choose_tile(L.n_row_blocks, N, L.K);
    return c == kWide ? 4 : c == kSplitTall ? 2 : c >= kSplitWide ? 1 : c;
}
int mpgemm_splits_k(const Layout& L, int N) {
    const int c = choose_tile(L.n_row_blocks, N, L.K);
    return c >= kSplitWide && c != kWide;
}

int launch_mpgemm(const Layout& L, const void* packed, const void* x, int N, void* y, void* workspace,
                  hipStream_t st) {
    (void)workspace;
    GemmArgs a;
    a.tiles = static_cast<const uint8_t*>(packed) + kHeaderBytes;
    a.x = static_cast<const _Float16*>(x);
    a.y = static_cast<_Float16*>(y);
    a.M = L.M;
    a.N = N;
    a.K = L.K;
    a.n_row_blocks = L.n_row_blocks;
    a.m_tiles = a.n_tiles = a.per_xcd = a.whole_row_tiles = 0;
    a.status = device_status_word();
    if (!a.status) return TMAN_ERR_LAUNCH;
    if (L.bits == 1) return L.has_zero ? launch_group<1, true>(L.group, a, st) : launch_group<1, false>(L.group, a, st);
    if (L.bits == 2) return launch_group<2, true>(L.group, a, st);
    return launch_group<4, true>(L.group, a, st);
}

}  // namespace tman
