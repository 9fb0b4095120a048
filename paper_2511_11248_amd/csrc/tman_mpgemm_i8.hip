// mpGEMM on the integer matrix cores for formats with ONE scale and zero per row of W -- per-channel, or
// per-tensor such as BitNet's ternary weights (Sec. 6.1: "per-tensor quantization ... treated as 2-bit";
// Sec. 6.2 mpGEMM: such models are dequantized to INT8 and computed as W_INT8 x A_INT8).
//
//   xq[n][k]  = rint(x[n][k] * 127 / max_k |x[n][k]|)                      int8, per token (tman_quantize_act_i8)
//   acc[n][m] = sum_k c[m][k] * xq[n][k]                                     int32, exact (v_mfma_i32_32x32x32_i8)
//   y[n][m]   = scale[m] * (max_n / 127) * (acc[n][m] - zero[m] * sum_k xq[n][k])      fp32, rounded once to fp16
//
// Level 1 of the paper's dequantization (bit-serial -> bit-parallel) is all the weights need here: the matrix
// unit multiplies the unsigned codes themselves, the zero point moves to the epilogue through the token's sum of
// integer activations.  The codes of a 32-weight block come out of the bit-field transposition as four words
// of eight nibbles, word o nibble f = weight 4 f + o; two masks per word turn them into bytes in the order
//   position p = 8 o + 4 h + b  <->  column 8 b + 4 h + o          (o < 4, h < 2, b < 4)
// and instead of sorting the weights the ACTIVATIONS are stored in that order: the quantizer writes every
// 32-column group of a token permuted accordingly, so both MFMA operands are plain 16-byte LDS reads.
//
// Three kernels, chosen per call from the grids they give (choose_i8_token_blocks).  The first:
// workgroup = 4 waves = 128 rows x 128 tokens; wave (wm, wn) accumulates 64 x 64 as four 32 x 32 tiles.  Per
// 64-column stage every wave transposes one 32-weight block of one of the two row blocks into LDS (lane = row),
// the 128 x 64 bytes of activations go through registers into LDS, one barrier, eight MFMAs per wave.  Two stage
// buffers: a wave writes stage s + 1 while others still read stage s.
// The second (mpgemm_i8_wide_kernel, below) keeps the weights out of LDS altogether; in the third
// (mpgemm_i8_ksplit_kernel) the waves of a workgroup also split K, for grids too small for the other two.
#include <hip/hip_fp16.h>

#include <mutex>
#include <type_traits>

#include "tman_dequant_device.h"

namespace tman {

typedef _Float16 half8_t __attribute__((ext_vector_type(8)));
typedef int32_t i32x4 __attribute__((ext_vector_type(4)));
typedef int32_t i32x16 __attribute__((ext_vector_type(16)));
typedef __amdgpu_buffer_rsrc_t rsrc_t;

constexpr int kI8Rows = 128, kI8Tokens = 128, kI8StageK = 64;
constexpr int kI8Ahead = 4;  // stages of global loads in flight per wave
constexpr int kI8RowBytes = kI8StageK + 16;  // padded LDS row: 20 dwords, conflict-free 16-byte accesses
constexpr int kI8StageBytes = (kI8Rows + kI8Tokens) * kI8RowBytes;
constexpr int kI8OutRow = kI8Rows * 2 + 16;  // bytes per token of the fp16 output tile in LDS
constexpr int kI8LdsBytes = 2 * kI8StageBytes > kI8Tokens * kI8OutRow ? 2 * kI8StageBytes : kI8Tokens * kI8OutRow;

__device__ __forceinline__ rsrc_t rsrc_of(const void* base, uint32_t bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, bytes, 0x00020000);
}

// ---------------------------------------------------------------------------------------------
// activation quantizer: one workgroup per token

// byte position p of a 32-column group holds column sigma(p) (see above)
__host__ __device__ constexpr int sigma(int p) { return 8 * (p & 3) + 4 * ((p >> 2) & 1) + (p >> 3); }

struct ActI8Layout {
    size_t q_bytes;     // int8 [N][K], every 32-column group permuted
    size_t absmax_off;  // float [N]
    size_t sum_off;     // int32 [N]
    size_t total;
};
static ActI8Layout act_i8_layout(int N, int K) {
    ActI8Layout l;
    l.q_bytes = ((size_t)N * K + 255) / 256 * 256;
    l.absmax_off = l.q_bytes;
    l.sum_off = l.absmax_off + (((size_t)N * 4 + 255) / 256 * 256);
    l.total = l.sum_off + (((size_t)N * 4 + 255) / 256 * 256);
    return l;
}
size_t act_i8_bytes(int N, int K) { return act_i8_layout(N, K).total; }

__global__ void __launch_bounds__(256) quantize_act_i8_kernel(const uint16_t* __restrict__ x, int K, int8_t* __restrict__ q,
                                                              float* __restrict__ absmax, int32_t* __restrict__ sums) {
    __shared__ unsigned wave_max[4];
    __shared__ int wave_sum[4];
    const int n = blockIdx.x, tid = threadIdx.x;
    const uint16_t* xb = x + (size_t)n * K;
    unsigned mx = 0;  // magnitudes compare like their bit patterns
    for (int k = tid; k < K; k += 256) mx = max(mx, (unsigned)(xb[k] & 0x7fffu));
    for (int d = 1; d < 64; d <<= 1) mx = max(mx, (unsigned)__shfl_xor((int)mx, d, 64));
    if ((tid & 63) == 0) wave_max[tid >> 6] = mx;
    __syncthreads();
    mx = max(max(wave_max[0], wave_max[1]), max(wave_max[2], wave_max[3]));
    const float amax = (float)__builtin_bit_cast(_Float16, (uint16_t)mx);
    // the decision is taken in binary32: one correctly rounded division, one product, round to nearest even
    const float inv = amax > 0.f ? __fdiv_rn(127.0f, amax) : 0.f;
    int s = 0;
    for (int g = tid; g < K / 32; g += 256) {
        int v[32];
#pragma unroll
        for (int c = 0; c < 32; ++c) {
            v[c] = (int)rintf(__fmul_rn((float)__builtin_bit_cast(_Float16, xb[g * 32 + c]), inv));
            s += v[c];
        }
        uint32_t w[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            w[i] = 0;
#pragma unroll
            for (int b = 0; b < 4; ++b) w[i] |= (uint32_t)(v[sigma(4 * i + b)] & 0xff) << (8 * b);
        }
        uint32_t* dst = reinterpret_cast<uint32_t*>(q + (size_t)n * K + (size_t)g * 32);
#pragma unroll
        for (int i = 0; i < 8; ++i) dst[i] = w[i];
    }
    for (int d = 1; d < 64; d <<= 1) s += __shfl_xor(s, d, 64);
    if ((tid & 63) == 0) wave_sum[tid >> 6] = s;
    __syncthreads();
    if (tid == 0) {
        absmax[n] = amax;
        sums[n] = (wave_sum[0] + wave_sum[1]) + (wave_sum[2] + wave_sum[3]);
    }
}

// The same for activations that start on a 16-byte boundary (every row then does: K is a multiple of 32): thread t
// reads group t of the token (32 columns, 64 bytes) once, with four 16-byte loads, and keeps it in registers from
// the search for the maximum to the rounding; only tokens longer than 8192 columns read their further groups twice.
__global__ void __launch_bounds__(256) quantize_act_i8_aligned_kernel(const uint16_t* __restrict__ x, int K,
                                                                      int8_t* __restrict__ q, float* __restrict__ absmax,
                                                                      int32_t* __restrict__ sums) {
    __shared__ unsigned wave_max[4];
    __shared__ int wave_sum[4];
    const int n = blockIdx.x, tid = threadIdx.x;
    const uint16_t* xb = x + (size_t)n * K;
    const int n_groups = K / 32;
    auto load_group = [&](u32x4 (&c)[4], int g) {
        const u32x4* src = reinterpret_cast<const u32x4*>(xb + (size_t)g * 32);
#pragma unroll
        for (int i = 0; i < 4; ++i) c[i] = src[i];
    };
    auto group_max = [&](const u32x4 (&c)[4], unsigned mx) {
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int e = 0; e < 4; ++e) mx = max(mx, max(c[i][e] & 0x7fffu, (c[i][e] >> 16) & 0x7fffu));
        return mx;
    };
    u32x4 mine[4] = {};
    const bool have = tid < n_groups;
    if (have) load_group(mine, tid);
    unsigned mx = group_max(mine, 0u);  // magnitudes compare like their bit patterns
    for (int g = tid + 256; g < n_groups; g += 256) {
        u32x4 c[4];
        load_group(c, g);
        mx = group_max(c, mx);
    }
    for (int d = 1; d < 64; d <<= 1) mx = max(mx, (unsigned)__shfl_xor((int)mx, d, 64));
    if ((tid & 63) == 0) wave_max[tid >> 6] = mx;
    __syncthreads();
    mx = max(max(wave_max[0], wave_max[1]), max(wave_max[2], wave_max[3]));
    const float amax = (float)__builtin_bit_cast(_Float16, (uint16_t)mx);
    // the decision is taken in binary32: one correctly rounded division, one product, round to nearest even
    const float inv = amax > 0.f ? __fdiv_rn(127.0f, amax) : 0.f;
    int s = 0;
    auto quantize_group = [&](const u32x4 (&c)[4], int g) {
        int v[32];
#pragma unroll
        for (int col = 0; col < 32; ++col) {
            const uint32_t word = c[col >> 3][(col >> 1) & 3];
            const uint16_t bits = (uint16_t)((col & 1) ? word >> 16 : word);
            v[col] = (int)rintf(__fmul_rn((float)__builtin_bit_cast(_Float16, bits), inv));
            s += v[col];
        }
        u32x4 out[2];
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            uint32_t w = 0;
#pragma unroll
            for (int b = 0; b < 4; ++b) w |= (uint32_t)(v[sigma(4 * i + b)] & 0xff) << (8 * b);
            out[i >> 2][i & 3] = w;
        }
        u32x4* dst = reinterpret_cast<u32x4*>(q + (size_t)n * K + (size_t)g * 32);
        dst[0] = out[0];
        dst[1] = out[1];
    };
    if (have) quantize_group(mine, tid);
    for (int g = tid + 256; g < n_groups; g += 256) {
        u32x4 c[4];
        load_group(c, g);
        quantize_group(c, g);
    }
    for (int d = 1; d < 64; d <<= 1) s += __shfl_xor(s, d, 64);
    if ((tid & 63) == 0) wave_sum[tid >> 6] = s;
    __syncthreads();
    if (tid == 0) {
        absmax[n] = amax;
        sums[n] = (wave_sum[0] + wave_sum[1]) + (wave_sum[2] + wave_sum[3]);
    }
}

int launch_quantize_act_i8(const void* x, int N, int K, void* out, hipStream_t st) {
    const ActI8Layout l = act_i8_layout(N, K);
    uint8_t* o = static_cast<uint8_t*>(out);
    const auto kernel = (reinterpret_cast<uintptr_t>(x) & 15u) == 0 ? quantize_act_i8_aligned_kernel : quantize_act_i8_kernel;
    hipLaunchKernelGGL(kernel, dim3((unsigned)N), dim3(256), 0, st, static_cast<const uint16_t*>(x), K,
                       reinterpret_cast<int8_t*>(o), reinterpret_cast<float*>(o + l.absmax_off),
                       reinterpret_cast<int32_t*>(o + l.sum_off));
    return launch_status();
}

// ---------------------------------------------------------------------------------------------
// the product

struct GemmI8Args {
    const uint8_t* tiles;
    const int8_t* xq;
    const float* absmax;
    const int32_t* sums;
    _Float16* y;
    int32_t* acc_out;  // optional: the integer accumulators [N][M]
    int M, N, K, n_row_blocks, n_ktiles;
    int m_tiles, n_tiles;
    int* status;
};

// Scale and sum of token n0 + tid, zero beyond the tokens: requested at the start of a kernel for its end.
struct TokenScales {
    float absmax;
    int32_t sum;
};
__device__ __forceinline__ TokenScales request_token_scales(const GemmI8Args& a, int n0, int tid) {
    const uint32_t off = (uint32_t)(n0 + tid) * 4u;
    TokenScales t;
    t.absmax = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rsrc_of(a.absmax, (uint32_t)a.N * 4u), off, 0, 0));
    t.sum = (int32_t)__builtin_amdgcn_raw_buffer_load_b32(rsrc_of(a.sums, (uint32_t)a.N * 4u), off, 0, 0);
    return t;
}

// The codes of one 32-weight block as 32 bytes in sigma order.
template <int B>
__device__ __forceinline__ void codes_to_bytes(const uint32_t (&plane)[B], u32x4& lo, u32x4& hi) {
    uint32_t codes[4];
    planes_to_codes<B>(plane, codes);
    constexpr uint32_t kMask = ((1u << B) - 1u) * 0x01010101u;
    // word o: even nibbles -> bytes 8 o .. 8 o + 3, odd nibbles -> bytes 8 o + 4 .. 8 o + 7
    lo = u32x4{codes[0] & kMask, (codes[0] >> 4) & kMask, codes[1] & kMask, (codes[1] >> 4) & kMask};
    hi = u32x4{codes[2] & kMask, (codes[2] >> 4) & kMask, codes[3] & kMask, (codes[3] >> 4) & kMask};
}

template <int B, int GQ, bool HZ>
__global__ void __launch_bounds__(256) mpgemm_i8_kernel(GemmI8Args a) {
    constexpr int MSZ = HZ ? 4 : 2;
    constexpr int MPL = (kKTile / GQ) * MSZ;
    constexpr int TB = B * 1024 + 64 * MPL;
    constexpr int CH = kKTile / B;
    extern __shared__ __attribute__((aligned(16))) uint8_t smem[];
    __shared__ float row_scale[kI8Rows], row_zs[kI8Rows];  // scale[m] and zero[m] * scale[m]

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int mt = blockIdx.x / a.n_tiles, nt = blockIdx.x % a.n_tiles;
    // a blob packed for another shape or layout: say so and leave y alone (one exit)
    const bool header_ok = header_matches(a.tiles, a.M, a.K, B, GQ, HZ ? 1 : 0);
    if (!header_ok && blockIdx.x == 0 && tid == 0) report_header_mismatch(a.status);
    if (mt >= (header_ok ? a.m_tiles : 0)) return;
    const int n0 = nt * kI8Tokens;
    const int k_stages = (a.K + kI8StageK - 1) / kI8StageK;  // K is a multiple of 32; a last half stage reads zeros

    // roles in the weight transposition: wave w -> row block w / 2 of the tile, 32-weight block w % 2 of the stage
    const int wrb = mt * 2 + (wave >> 1), wblk = wave & 1;
    const bool wvalid = wrb < a.n_row_blocks;
    const uint8_t* wsrc = a.tiles + (size_t)(wvalid ? wrb : 0) * a.n_ktiles * TB;
    const uint32_t wbytes = wvalid ? (uint32_t)(a.n_ktiles * TB) : 0u;
    const int k32_total = a.K / 32;
    auto load_planes = [&](uint32_t (&plane)[B], int stage) {
        const int k32 = stage * 2 + wblk;  // 32-weight block along K
        const rsrc_t rw = rsrc_of(wsrc, k32 < k32_total ? wbytes : 0u);
        const int tile = k32 >> 2, kb32 = k32 & 3;
        const int v = (kb32 * 32) / CH, ksub = ((kb32 * 32) % CH) / 32;
        const int so = tile * TB + v * 1024 + ksub * B * 4;
        if constexpr (B == 4) {
            const u32x4 w = __builtin_amdgcn_raw_buffer_load_b128(rw, lane * 16, so, 0);
            plane[0] = w.x; plane[1] = w.y; plane[2] = w.z; plane[3] = w.w;
        } else if constexpr (B == 2) {
            const u32x2 w = __builtin_amdgcn_raw_buffer_load_b64(rw, lane * 16, so, 0);
            plane[0] = w.x; plane[1] = w.y;
        } else {
            plane[0] = __builtin_amdgcn_raw_buffer_load_b32(rw, lane * 16, so, 0);
        }
    };
    // activations of a stage: thread -> token tid / 2, 32 bytes at column half tid % 2; tokens beyond N and columns
    // beyond K lie outside the resource and read as zero
    const int xtok = tid >> 1, xhalf = tid & 1;
    const rsrc_t rx = rsrc_of(a.xq, (uint32_t)a.N * (uint32_t)a.K);
    auto load_x = [&](u32x4 (&xv)[2], int stage) {
        const int col = stage * kI8StageK + xhalf * 32;
        const bool in = (n0 + xtok) < a.N && col < a.K;
        const uint32_t off = in ? (uint32_t)(n0 + xtok) * (uint32_t)a.K + (uint32_t)col : 0xFFFFFFF0u;
        xv[0] = __builtin_amdgcn_raw_buffer_load_b128(rx, off, 0, 0);
        xv[1] = __builtin_amdgcn_raw_buffer_load_b128(rx, in ? off + 16u : 0xFFFFFFF0u, 0, 0);
    };

    i32x16 acc[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = 0;
    const int wm = wave >> 1, wn = wave & 1, r = lane & 31, h = lane >> 5;

    // Global loads run kI8Ahead stages ahead of their use, in a ring of register sets (a stage of MFMAs is far
    // shorter than the latency of a load); stages past K read zeros, so the loop runs whole rings.
    uint32_t plane[kI8Ahead][B];
    u32x4 xv[kI8Ahead][2];
#pragma unroll
    for (int u = 0; u < kI8Ahead; ++u) {
        load_planes(plane[u], u);
        load_x(xv[u], u);
    }
    // scale and zero of the tile's rows (the first quantization block of a row stands for the whole row)
    if (tid < kI8Rows) {
        const int rb = mt * 2 + (tid >> 6), l = tid & 63;
        float sc = 0.f, zs = 0.f;
        if (rb < a.n_row_blocks) {
            const uint8_t* meta = a.tiles + (size_t)rb * a.n_ktiles * TB + B * 1024 + l * MPL;
            sc = (float)*reinterpret_cast<const _Float16*>(meta);
            zs = HZ ? (float)*reinterpret_cast<const _Float16*>(meta + 2) * sc : 0.f;
        }
        row_scale[tid] = sc;
        row_zs[tid] = zs;
    }
    const int n_stages = (k_stages + kI8Ahead - 1) / kI8Ahead * kI8Ahead;
    for (int s0 = 0; s0 < n_stages; s0 += kI8Ahead) {
#pragma unroll
        for (int u = 0; u < kI8Ahead; ++u) {
            const int s = s0 + u;
            uint8_t* buf = smem + (s & 1) * kI8StageBytes;
            {
                u32x4 lo, hi;
                codes_to_bytes<B>(plane[u], lo, hi);
                uint8_t* wrow = buf + ((wave >> 1) * 64 + lane) * kI8RowBytes + wblk * 32;
                *reinterpret_cast<u32x4*>(wrow) = lo;
                *reinterpret_cast<u32x4*>(wrow + 16) = hi;
                uint8_t* xrow = buf + (kI8Rows + xtok) * kI8RowBytes + xhalf * 32;
                *reinterpret_cast<u32x4*>(xrow) = xv[u][0];
                *reinterpret_cast<u32x4*>(xrow + 16) = xv[u][1];
            }
            load_planes(plane[u], s + kI8Ahead);
            load_x(xv[u], s + kI8Ahead);
            __syncthreads();
            const uint8_t* wbase = buf + (wm * 64 + r) * kI8RowBytes + h * 16;
            const uint8_t* xbase = buf + (kI8Rows + wn * 64 + r) * kI8RowBytes + h * 16;
#pragma unroll
            for (int ks = 0; ks < 2; ++ks) {
                i32x4 wf[2], xf[2];
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    wf[i] = *reinterpret_cast<const i32x4*>(wbase + i * 32 * kI8RowBytes + ks * 32);
                    xf[i] = *reinterpret_cast<const i32x4*>(xbase + i * 32 * kI8RowBytes + ks * 32);
                }
#pragma unroll
                for (int i = 0; i < 2; ++i)
#pragma unroll
                    for (int j = 0; j < 2; ++j)
                        acc[i][j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(wf[i], xf[j], acc[i][j], 0, 0, 0);
            }
        }
    }
    __syncthreads();  // every wave is done with the stage buffers, which the output tile reuses

    // epilogue: C[i][j] of a 32 x 32 tile: i = row 8 (v / 4) + 4 h + v % 4, j = token lane % 32
    uint8_t* otile = smem;
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        const int tok = wn * 64 + j * 32 + r, gn = n0 + tok;
        const bool live = gn < a.N;
        const float delta = live ? a.absmax[gn] * (1.0f / 127.0f) : 0.f;
        const float sx = live ? (float)a.sums[gn] : 0.f;
#pragma unroll
        for (int i = 0; i < 2; ++i) {
#pragma unroll
            for (int g4 = 0; g4 < 4; ++g4) {
                const int row = wm * 64 + i * 32 + 8 * g4 + 4 * h;
                float v[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float av = (float)acc[i][j][4 * g4 + e];
                    // (c - z) s summed: s acc - (z s) sum(xq); sign form (2 c - 1) s: 2 s acc - s sum(xq)
                    v[e] = HZ ? delta * fmaf(row_scale[row + e], av, -row_zs[row + e] * sx)
                              : delta * row_scale[row + e] * fmaf(2.f, av, -sx);
                }
                half2_t p0, p1;
                p0.x = (_Float16)v[0]; p0.y = (_Float16)v[1];
                p1.x = (_Float16)v[2]; p1.y = (_Float16)v[3];
                u32x2 w = {__builtin_bit_cast(uint32_t, p0), __builtin_bit_cast(uint32_t, p1)};
                *reinterpret_cast<u32x2*>(otile + tok * kI8OutRow + row * 2) = w;
                if (a.acc_out && live) {
                    const int gm = mt * kI8Rows + row;
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        if (gm + e < a.M) a.acc_out[(size_t)gn * a.M + gm + e] = acc[i][j][4 * g4 + e];
                }
            }
        }
    }
    __syncthreads();
    store_tile<kI8Rows, kI8Tokens, kI8OutRow, 256>(a.y, a.M, a.N, otile, mt * kI8Rows, n0, tid);
}

// The two 32-column blocks of a lane in a tile block of 32 rows (lane half h: blocks 2 h and 2 h + 1); `off`: of the lane's
// first chunk, r * 16 + h * (bytes of two blocks' chunks, within a chunk for 1 bit).
template <int B>
__device__ __forceinline__ void load_unit_planes(uint32_t (&pl)[2][B], rsrc_t rw, int off, int tile_off) {
    if constexpr (B == 4) {
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const u32x4 w = __builtin_amdgcn_raw_buffer_load_b128(rw, off + i * 1024, tile_off, 0);
#pragma unroll
            for (int e = 0; e < 4; ++e) pl[i][e] = w[e];
        }
    } else if constexpr (B == 2) {
        const u32x4 w = __builtin_amdgcn_raw_buffer_load_b128(rw, off, tile_off, 0);
        pl[0][0] = w.x; pl[0][1] = w.y; pl[1][0] = w.z; pl[1][1] = w.w;
    } else {
        const u32x2 w = __builtin_amdgcn_raw_buffer_load_b64(rw, off, tile_off, 0);
        pl[0][0] = w.x; pl[1][0] = w.y;
    }
}

// ---------------------------------------------------------------------------------------------
// Wide variant for long token ranges: no weight tile in LDS.  A wave owns 64 rows x 32 TT tokens.  Lane (r, h) of a row unit
// (32 rows) takes the 32-column blocks 2 h and 2 h + 1 of row r of a 128-column tile, which it loads and turns into bytes
// alone: a product sums over 16 columns of a block of the first and of one of the second half of the tile, and the
// activations are read to match, so no lane exchanges anything.  Only the activations go through LDS, straight from memory,
// shared by the four waves (256 rows) of the workgroup, a tile (128 bytes of a token, a whole cache line) at a time
// (by 32-column stages, with exchanges: 11008 x 4096 4 bits N = 2048 124 us, now 88; 6912 x 2560 2 bits N = 1024 28.6, now 23.3).  Per MFMA
// this reads half the LDS bytes of the 128 x 128 kernel and dequantizes each weight once per 32 TT tokens instead of once per 128.
constexpr int kI8WRing = 4;   // tile buffers of activations in LDS
constexpr int kI8WRows = 256;

template <int TT>
struct I8Wide {
    static constexpr int TN = TT * 32;
    static constexpr int XBytes = TN * kKTile;         // activations of a tile
    static constexpr int XLoads = TT;                  // requests of a tile per wave (8 token rows each)
    static constexpr int OutRow = kI8WRows * 2 + 16;   // bytes per token of the fp16 output tile in LDS
    static constexpr int LdsBytes = kI8WRing * XBytes > TN * OutRow ? kI8WRing * XBytes : TN * OutRow;
};

template <int B, bool HZ, int TT>
__global__ void __launch_bounds__(256, (TT <= 4 ? 2 : 1)) mpgemm_i8_wide_kernel(GemmI8Args a, int group) {
    using T = I8Wide<TT>;
    constexpr int MSZ = HZ ? 4 : 2;
    constexpr int kSets = 2;  // register sets of bit planes = tiles of weights in flight
    extern __shared__ __attribute__((aligned(16))) uint8_t smem[];
    __shared__ float row_scale[kI8WRows], row_zs[kI8WRows], token_step[T::TN], token_sum[T::TN];

    const int MPL = (kKTile / group) * MSZ, TB = B * 1024 + 64 * MPL;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int mt = blockIdx.x / a.n_tiles, nt = blockIdx.x % a.n_tiles;
    const bool header_ok = header_matches(a.tiles, a.M, a.K, B, group, HZ ? 1 : 0);
    if (!header_ok && blockIdx.x == 0 && threadIdx.x == 0) report_header_mismatch(a.status);
    if (mt >= (header_ok ? a.m_tiles : 0)) return;
    const int n0 = nt * T::TN;
    const int r = lane & 31, h = lane >> 5;

    i32x16 acc[2][TT];
#pragma unroll
    for (int ru = 0; ru < 2; ++ru)
#pragma unroll
        for (int nb = 0; nb < TT; ++nb)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[ru][nb][v] = 0;

    // bit planes of this wave's row block: of each row unit the lane's two blocks of a tile; a tile past K reads as zero
    const int wrb = mt * 4 + wave;
    const bool wvalid = wrb < a.n_row_blocks;
    const uint8_t* wsrc = a.tiles + (size_t)(wvalid ? wrb : 0) * a.n_ktiles * TB;
    const uint32_t wbytes = wvalid ? (uint32_t)(a.n_ktiles * TB) : 0u;
    uint32_t plane[kSets][2][2][B];  // [set][row unit][block][plane]
    const int woff = r * 16 + (B == 1 ? h * 8 : h * (B / 2) * 1024);
    constexpr int kPlaneLoads = 2 * (B == 4 ? 2 : 1);
    auto load_planes = [&](uint32_t (&pl)[2][2][B], int t) {
        const rsrc_t rw = rsrc_of(wsrc, t < a.n_ktiles ? wbytes : 0u);
#pragma unroll
        for (int ru = 0; ru < 2; ++ru) load_unit_planes<B>(pl[ru], rw, woff + ru * 512, t * TB);
    };
    // Activations: a request brings 8 token rows x 128 bytes straight into LDS; wave w issues requests w, w + 4, ...  16-byte
    // chunk c of row R is kept at place c ^ ((R >> 1) & 7), so that the operand reads of 16 consecutive rows fall on 16
    // different places.  Rows beyond the tile's tokens lie outside the resource (zeros).  Columns beyond K are those of the
    // next token, behind the last one what the buffer keeps there (at least 512 bytes: scales and sums): their codes are zero.
    const int xrows = a.N - n0 < T::TN ? a.N - n0 : T::TN;
    const int8_t* xsrc = a.xq + (size_t)n0 * a.K;
    const uint32_t xbytes = (uint32_t)xrows * (uint32_t)a.K;
    const uint32_t xlane = (uint32_t)(wave * 8 + (lane >> 3)) * (uint32_t)a.K + (uint32_t)((lane & 7) ^ ((wave & 1) * 4 + (lane >> 4))) * 16u;
    const uint32_t x32rows = 32u * (uint32_t)a.K;
    auto load_x = [&](int t, int from = 0, int to = T::XLoads) {
        const rsrc_t rx = rsrc_of(xsrc, t < a.n_ktiles ? xbytes : 0u);
        uint8_t* dst = smem + (t & (kI8WRing - 1)) * T::XBytes;
#pragma unroll
        for (int i = from; i < to; ++i)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rx, (__attribute__((address_space(3))) void*)(dst + (wave + 4 * i) * 1024), 16,
                                                     xlane + (uint32_t)i * x32rows, t * kKTile, 0, 0);
    };
    // operand of step j (block j / 2 of the lane's two, its bytes 16 (j % 2) ..): chunk 4 h + j
    int xoff[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) xoff[j] = r * kKTile + ((4 * h + j) ^ ((r >> 1) & 7)) * 16;
    i32x4 xf[2][TT];
    auto read_x = [&](int j, const uint8_t* tile) {
#pragma unroll
        for (int nb = 0; nb < TT; ++nb) xf[j & 1][nb] = *reinterpret_cast<const i32x4*>(tile + xoff[j] + nb * 32 * kKTile);
    };
    i32x4 wf[2][2][2];  // [block][row unit][step of the block]
    auto operands = [&](int block, int ru, const uint32_t (&pl)[2][2][B]) {
        u32x4 lo, hi;
        codes_to_bytes<B>(pl[ru][block], lo, hi);
        wf[block][ru][0] = __builtin_bit_cast(i32x4, lo);
        wf[block][ru][1] = __builtin_bit_cast(i32x4, hi);
    };

    // Requests in the order of the loop, whose waits count them.
    // scale and zero of the tile's rows (the first quantization block of a row stands for the whole row)
    const rsrc_t rmeta = rsrc_of(wsrc, wbytes);
    const uint32_t meta_s = __builtin_amdgcn_raw_buffer_load_b16(rmeta, lane * MPL, B * 1024, 0);
    const uint32_t meta_z = HZ ? __builtin_amdgcn_raw_buffer_load_b16(rmeta, lane * MPL + 2, B * 1024, 0) : 0u;
    const TokenScales scales = request_token_scales(a, n0, tid);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int t = 0; t < kSets - 1; ++t) {
        load_planes(plane[t], t);
        __builtin_amdgcn_sched_barrier(0);
    }
    load_x(0);
    load_x(1);
    __builtin_amdgcn_sched_barrier(0);
    load_x(2);
    __builtin_amdgcn_sched_barrier(0);
    load_planes(plane[kSets - 1], kSets - 1);
    __builtin_amdgcn_sched_barrier(0);
    {
        const float sc = (float)__builtin_bit_cast(_Float16, (uint16_t)meta_s);
        row_scale[tid] = sc;
        row_zs[tid] = HZ ? (float)__builtin_bit_cast(_Float16, (uint16_t)meta_z) * sc : 0.f;
        if (tid < T::TN) {
            token_step[tid] = scales.absmax * (1.0f / 127.0f);
            token_sum[tid] = (float)scales.sum;
        }
    }
    operands(0, 0, plane[0]);
    operands(0, 1, plane[0]);
    __builtin_amdgcn_sched_barrier(0);
    // the activations of tiles 0 and 1 are in
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(T::XLoads + kPlaneLoads) : "memory");
    read_x(0, smem);

    const int n_tiles_k = (a.n_ktiles + kSets - 1) & ~(kSets - 1);  // (a tile past K is zeros)
    for (int t0 = 0; t0 < n_tiles_k; t0 += kSets) {
#pragma unroll
        for (int u = 0; u < kSets; ++u) {
            const int t = t0 + u;
            const uint8_t* cur = smem + (t & (kI8WRing - 1)) * T::XBytes;
            const uint8_t* nxt = smem + ((t + 1) & (kI8WRing - 1)) * T::XBytes;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                if (j < 2) {  // (half of the requests a step, ahead of the planes')
                    load_x(t + 3, j ? (T::XLoads + 1) / 2 : 0, j ? T::XLoads : (T::XLoads + 1) / 2);
                    __builtin_amdgcn_sched_barrier(0);
                }
                // the products of step j; meanwhile the activations of the next step and one row unit of the next block
                read_x((j + 1) & 3, j == 3 ? nxt : cur);
                operands(j < 2 ? 1 : 0, j & 1, plane[(j < 2 ? u : u + 1) % kSets]);
#pragma unroll
                for (int nb = 0; nb < TT; ++nb)
#pragma unroll
                    for (int ru = 0; ru < 2; ++ru)
                        acc[ru][nb] = __builtin_amdgcn_mfma_i32_32x32x32_i8(wf[j >> 1][ru][j & 1], xf[j & 1][nb], acc[ru][nb], 0, 0, 0);
#pragma unroll
                for (int i = 0; i < 2 * TT; ++i) {
                    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                    __builtin_amdgcn_sched_group_barrier(0x002, 3, 0);
                    if (i < TT) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
                }
                __builtin_amdgcn_sched_barrier(0);
                if (j == 1) {  // both blocks of the tile's planes are used
                    load_planes(plane[u % kSets], t + kSets);
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
            // the activations of tile t + 2 (requested one tile ago) are in before any wave goes on: younger are the planes
            // requested then and what this tile requested
            asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"(T::XLoads + 2 * kPlaneLoads) : "memory");
        }
    }
    // requests of tiles past the end may still be writing to the ring, which the output tile reuses
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();

    // epilogue: C[i][j] of a 32 x 32 tile: i = row 8 (v / 4) + 4 h + v % 4, j = token lane % 32.  Scales come from LDS (read from
    // memory here, one token block after the other, they took 3 of a call's 25 us), stores of whole tiles are unrolled.
    if (a.acc_out) {  // (uniform)
#pragma unroll 1
        for (int nb = 0; nb < TT; ++nb) {
            const int gn = n0 + nb * 32 + r;
#pragma unroll
            for (int hb = 0; hb < 2; ++hb)
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const int gm = mt * kI8WRows + wave * 64 + hb * 32 + 8 * (v / 4) + 4 * h + v % 4;
                    int32_t av = acc[hb][0][v];
#pragma unroll
                    for (int q = 1; q < TT; ++q) av = nb == q ? acc[hb][q][v] : av;
                    if (gn < a.N && gm < a.M) a.acc_out[(size_t)gn * a.M + gm] = av;
                }
        }
    }
    uint8_t* otile = smem;
#pragma unroll
    for (int nb = 0; nb < TT; ++nb) {
        const int tok = nb * 32 + r;
        const float delta = token_step[tok], sx = token_sum[tok];
#pragma unroll
        for (int hb = 0; hb < 2; ++hb) {
#pragma unroll
            for (int g4 = 0; g4 < 4; ++g4) {
                const int row = wave * 64 + hb * 32 + 8 * g4 + 4 * h;
                float v[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float av = (float)acc[hb][nb][4 * g4 + e];
                    v[e] = HZ ? delta * fmaf(row_scale[row + e], av, -row_zs[row + e] * sx)
                              : delta * row_scale[row + e] * fmaf(2.f, av, -sx);
                }
                half2_t p0, p1;
                p0.x = (_Float16)v[0]; p0.y = (_Float16)v[1];
                p1.x = (_Float16)v[2]; p1.y = (_Float16)v[3];
                u32x2 w = {__builtin_bit_cast(uint32_t, p0), __builtin_bit_cast(uint32_t, p1)};
                *reinterpret_cast<u32x2*>(otile + tok * T::OutRow + row * 2) = w;
            }
        }
    }
    __syncthreads();
    store_tile<kI8WRows, T::TN, T::OutRow, 256>(a.y, a.M, a.N, otile, mt * kI8WRows, n0, tid);
}

template <int B, bool HZ, int TT>
static int launch_i8_wide(GemmI8Args a, int group, hipStream_t st) {
    static std::once_flag once;
    static hipError_t attr_rc = hipSuccess;
    std::call_once(once, [] {
        attr_rc = hipFuncSetAttribute(reinterpret_cast<const void*>(&mpgemm_i8_wide_kernel<B, HZ, TT>),
                                      hipFuncAttributeMaxDynamicSharedMemorySize, I8Wide<TT>::LdsBytes);
    });
    if (attr_rc != hipSuccess) return TMAN_ERR_LAUNCH;
    a.m_tiles = (a.n_row_blocks + 3) / 4;
    a.n_tiles = (a.N + I8Wide<TT>::TN - 1) / I8Wide<TT>::TN;
    hipLaunchKernelGGL((mpgemm_i8_wide_kernel<B, HZ, TT>), dim3((unsigned)(a.m_tiles * a.n_tiles)), dim3(256),
                       I8Wide<TT>::LdsBytes, st, a, group);
    return launch_status();
}

// ---------------------------------------------------------------------------------------------
// Third kernel, for grids that leave compute units idle even with 64-row workgroups: the four waves of a workgroup
// split K.  Wave w takes the 128-column tiles w, w + 4, ... whole: bit planes -> bytes in registers, the tile's int8
// activations into LDS buffers of its own (whole cache lines, as in the wide kernel), MFMAs with all tokens of the workgroup's
// tile; no wave waits for another until the end, where the four partial integer tiles are added in LDS (integers: the result
// does not depend on the grouping, so every kernel of this file gives the same bits).
// Tile: 128 rows x 128 tokens (two row blocks per wave).  A wave's share was 32-column stages before, 32 bytes of each of 32 cache
// lines per request: 2560 x 6912 2 bits N = 1024 35.8 us, now 27.2; 4096 x 4096 4 bits N = 700 27.1 / 21.6; 1024 x 8192 N = 2048
// 39.1 / 29.7; 11008 x 4096 4 bits N = 256 26.4 / 21.3.
template <int RBW, int TT>
struct I8KsTile {
    static constexpr int TN = 32 * TT, TM = 64 * RBW;
    static constexpr int XBytes = TN * kKTile;                // activations of a tile, 128 bytes per token
    static constexpr int NBuf = 2;                             // activation buffers per wave
    static constexpr int XLoads = TN / 8;                     // requests per tile (8 token rows each)
    static constexpr int PartRow = TM * 4 + 16;                // bytes per token of a wave's partial tile in LDS
    static constexpr int PartBytes = (TN / 2) * PartRow;       // ... of half of its tokens
    static constexpr int LdsBytes = 4 * NBuf * XBytes > 4 * PartBytes ? 4 * NBuf * XBytes : 4 * PartBytes;
    static_assert(RBW * TT == 8 && LdsBytes + 2 * TM * 4 <= 160 * 1024, "tile of the K-split kernel");
};

template <int B, bool HZ, int RBW, int TT>
__global__ void __launch_bounds__(256, 1) mpgemm_i8_ksplit_kernel(GemmI8Args a, int group) {
    using T = I8KsTile<RBW, TT>;
    constexpr int kUnits = 2 * RBW;  // row units of 32 rows
    constexpr int MSZ = HZ ? 4 : 2;
    extern __shared__ __attribute__((aligned(16))) uint8_t smem[];
    __shared__ float row_scale[T::TM], row_zs[T::TM], token_step[T::TN], token_sum[T::TN];

    const int MPL = (kKTile / group) * MSZ, TB = B * 1024 + 64 * MPL;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int mt = blockIdx.x / a.n_tiles, nt = blockIdx.x % a.n_tiles;
    const bool header_ok = header_matches(a.tiles, a.M, a.K, B, group, HZ ? 1 : 0);
    if (!header_ok && blockIdx.x == 0 && tid == 0) report_header_mismatch(a.status);
    if (mt >= (header_ok ? a.m_tiles : 0)) return;
    const int n0 = nt * T::TN;
    const int n_own = (a.n_ktiles + 3) / 4;  // own tiles of this wave
    const int r = lane & 31, h = lane >> 5;

    i32x16 acc[RBW][2][TT];
#pragma unroll
    for (int b = 0; b < RBW; ++b)
#pragma unroll
        for (int hb = 0; hb < 2; ++hb)
#pragma unroll
            for (int nb = 0; nb < TT; ++nb)
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[b][hb][nb][v] = 0;

    uint32_t plane[2][kUnits][2][B];  // [set][row unit][block][plane]
    constexpr int kUnitLoads = B == 4 ? 2 : 1;
    const int woff = r * 16 + (B == 1 ? h * 8 : h * (B / 2) * 1024);
    auto load_unit = [&](int set, int unit, int i) {  // own tile i = tile 4 i + wave
        const int t = 4 * i + wave, rb = mt * RBW + unit / 2;
        const bool wvalid = rb < a.n_row_blocks;
        const uint8_t* wsrc = a.tiles + (size_t)(wvalid ? rb : 0) * a.n_ktiles * TB;
        const rsrc_t rw = rsrc_of(wsrc, t < a.n_ktiles && wvalid ? (uint32_t)(a.n_ktiles * TB) : 0u);
        load_unit_planes<B>(plane[set][unit], rw, woff + (unit & 1) * 512, t * TB);
    };
    // activations of own tile i go to this wave's buffer i % NBuf, chunks placed as in the wide kernel
    const int xrows = a.N - n0 < T::TN ? a.N - n0 : T::TN;
    const int8_t* xsrc = a.xq + (size_t)n0 * a.K;
    const uint32_t xbytes = (uint32_t)xrows * (uint32_t)a.K;
    const uint32_t xlane = (uint32_t)(lane >> 3) * (uint32_t)a.K, x8rows = 8u * (uint32_t)a.K;
    const uint32_t xchunk[2] = {(uint32_t)((lane & 7) ^ (lane >> 4)) * 16u, (uint32_t)((lane & 7) ^ (4 + (lane >> 4))) * 16u};
    uint8_t* const xbuf = smem + wave * T::NBuf * T::XBytes;
    auto load_x = [&](int i, int from = 0, int to = T::XLoads) {
        const int t = 4 * i + wave;
        const rsrc_t rx = rsrc_of(xsrc, t < a.n_ktiles ? xbytes : 0u);
        uint8_t* dst = xbuf + (i & (T::NBuf - 1)) * T::XBytes;
#pragma unroll
        for (int q = from; q < to; ++q)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rx, (__attribute__((address_space(3))) void*)(dst + q * 1024), 16,
                                                     xlane + (uint32_t)q * x8rows + xchunk[q & 1], t * kKTile, 0, 0);
    };
    int xoff[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) xoff[j] = r * kKTile + ((4 * h + j) ^ ((r >> 1) & 7)) * 16;
    i32x4 xf[4][TT];
    auto read_x = [&](int j, const uint8_t* tile) {
#pragma unroll
        for (int nb = 0; nb < TT; ++nb) xf[j][nb] = *reinterpret_cast<const i32x4*>(tile + xoff[j] + nb * 32 * kKTile);
    };
    i32x4 wf[2][4];  // [unit % 2][step]
    auto operands = [&](int block, int set, int unit) {
        u32x4 lo, hi;
        codes_to_bytes<B>(plane[set][unit][block], lo, hi);
        wf[unit & 1][2 * block] = __builtin_bit_cast(i32x4, lo);
        wf[unit & 1][2 * block + 1] = __builtin_bit_cast(i32x4, hi);
    };

    // scale and zero of the tile's rows (the first quantization block of a row stands for the whole row)
    const int mrb = mt * RBW + wave;
    const rsrc_t rmeta = rsrc_of(a.tiles + (size_t)(mrb < a.n_row_blocks ? mrb : 0) * a.n_ktiles * TB,
                                 wave < RBW && mrb < a.n_row_blocks ? (uint32_t)TB : 0u);
    const uint32_t meta_s = __builtin_amdgcn_raw_buffer_load_b16(rmeta, lane * MPL, B * 1024, 0);
    const uint32_t meta_z = HZ ? __builtin_amdgcn_raw_buffer_load_b16(rmeta, lane * MPL + 2, B * 1024, 0) : 0u;
    const TokenScales scales = request_token_scales(a, n0, tid);
    __builtin_amdgcn_sched_barrier(0);
    // The waits below and in the loop count the requests, so none may be moved past another group.  The activations of own tile 1
    // go ahead of its weights: 4096 x 4096 4 bits N = 700 20.8 us, behind them 21.2.
#pragma unroll
    for (int u = 0; u < kUnits; ++u) load_unit(0, u, 0);
    __builtin_amdgcn_sched_barrier(0);
    load_x(0);
    __builtin_amdgcn_sched_barrier(0);
    load_x(1);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int u = 0; u < kUnits; ++u) load_unit(1, u, 1);
    __builtin_amdgcn_sched_barrier(0);
    if (tid < T::TM) {
        const float sc = (float)__builtin_bit_cast(_Float16, (uint16_t)meta_s);
        row_scale[tid] = sc;
        row_zs[tid] = HZ ? (float)__builtin_bit_cast(_Float16, (uint16_t)meta_z) * sc : 0.f;
    }
    if (tid < T::TN) {
        token_step[tid] = scales.absmax * (1.0f / 127.0f);
        token_sum[tid] = (float)scales.sum;
    }
    operands(0, 0, 0);
    operands(1, 0, 0);
    __builtin_amdgcn_sched_barrier(0);
    load_unit(0, 0, 2);
    __builtin_amdgcn_sched_barrier(0);
    // activations of own tile 0: younger are the requests of own tile 1 and unit 0 of own tile 2
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"((kUnits + 1) * kUnitLoads + T::XLoads) : "memory");
#pragma unroll
    for (int j = 0; j < 4; ++j) read_x(j, xbuf);

    auto own_tile = [&](int i, auto parity) {
        constexpr int s = decltype(parity)::value;  // i % 2
        const uint8_t* nxt = xbuf + ((i + 1) & (T::NBuf - 1)) * T::XBytes;
#pragma unroll
        for (int u = 0; u < kUnits; ++u) {
            constexpr int kLast = kUnits - 1;
            const int nu = u == kLast ? 0 : u + 1, nset = u == kLast ? (s + 1) & 1 : s;
            // The activations of own tile i + 1 must be in (requested behind unit 0 of the previous own tile).  Younger: at
            // least its weights from then on, as many of this tile, and the activations of own tile i + 2.
            if (u == kLast) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(kUnits * kUnitLoads + T::XLoads) : "memory");
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                if (j % 2 == 0) {
                    if (u == 1) {  // the activations of this own tile are in registers (unit 0 used them all)
                        load_x(i + 2, j * T::XLoads / 4, (j + 2) * T::XLoads / 4);
                        __builtin_amdgcn_sched_barrier(0);
                    }
                    operands(j / 2, nset, nu);
                }
#pragma unroll
                for (int nb = 0; nb < TT; ++nb)
                    acc[u / 2][u & 1][nb] = __builtin_amdgcn_mfma_i32_32x32x32_i8(wf[u & 1][j], xf[j][nb], acc[u / 2][u & 1][nb], 0, 0, 0);
                if (u == kLast) read_x(j, nxt);
                if (j % 2 == 1) {
#pragma unroll
                    for (int q = 0; q < 2 * TT; ++q) {
                        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                        __builtin_amdgcn_sched_group_barrier(0x002, 32 / (2 * TT), 0);
                        if (u == kLast) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
                    }
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
            load_unit(nset, nu, (u == kLast ? i + 1 : i) + 2);  // the registers of the row unit just turned into bytes are free
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    // (the registers alternate by the parity of i, so the body is there for both; an odd number of own tiles rounded up to an even one
    // cost a tile of zeros: 18818 x 2304 4 bits N = 56 17.5 -> 16.0 us, 1600 x 2496 N = 548 14.7 -> 13.2, K > 7000 3 %)
    int i0 = 0;
    for (; i0 + 2 <= n_own; i0 += 2) {
        own_tile(i0, std::integral_constant<int, 0>{});
        own_tile(i0 + 1, std::integral_constant<int, 1>{});
    }
    if (i0 < n_own) own_tile(i0, std::integral_constant<int, 0>{});
    // requests of own stages past the end may still be writing zeros to LDS, which the partial tiles reuse
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();

    // The four partial tiles meet in LDS, half of the tokens at a time: wave w writes its int32 sums as
    // [token][row], then thread -> (token, 8 rows) adds the four, scales and stores fp16.
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
                        int32_t* dst = reinterpret_cast<int32_t*>(mine + (nq * 32 + r) * T::PartRow + (64 * b + 32 * hb + 8 * g + 4 * h) * 4);
#pragma unroll
                        for (int e = 0; e < 4; ++e) dst[e] = acc[b][hb][nb][4 * g + e];
                    }
        }
        __syncthreads();
        if (!fast) {  // (rows of y start anywhere: consecutive lanes take consecutive rows; eight of a lane before, 141 x 2048 N = 1202 21.2 -> 17.8 us)
            const int first = half * (T::TN / 2), live = a.N - n0 - first;
            for (int i = tid; i < (live < T::TN / 2 ? live : T::TN / 2) * T::TM; i += 256) {
                const int n = i / T::TM, row = i % T::TM;
                int32_t sum = 0;
#pragma unroll
                for (int w = 0; w < 4; ++w) sum += *reinterpret_cast<const int32_t*>(smem + w * T::PartBytes + n * T::PartRow + row * 4);
                if (m0 + row >= a.M) continue;
                const float av = (float)sum, delta = token_step[first + n], sx = token_sum[first + n];
                const size_t at = (size_t)(n0 + first + n) * a.M + m0 + row;
                float v = HZ ? delta * fmaf(row_scale[row], av, -row_zs[row] * sx) : delta * row_scale[row] * fmaf(2.f, av, -sx);
                asm("" : "+v"(v));  // (rounded to fp32 first, as everywhere else: one conversion of the product would give other bits)
                a.y[at] = (_Float16)v;
                if (a.acc_out) a.acc_out[at] = sum;
            }
            __syncthreads();
            continue;
        }
        for (int piece = tid; piece < (T::TN / 2) * (T::TM / 8); piece += 256) {
            const int n = piece / (T::TM / 8), c8 = piece % (T::TM / 8);
            const int gn = n0 + half * (T::TN / 2) + n, gm = m0 + c8 * 8;
            int32_t sum[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) sum[e] = 0;
#pragma unroll
            for (int w = 0; w < 4; ++w) {
                const int32_t* src = reinterpret_cast<const int32_t*>(smem + w * T::PartBytes + n * T::PartRow + c8 * 32);
#pragma unroll
                for (int e = 0; e < 8; ++e) sum[e] += src[e];
            }
            if (gn >= a.N || gm >= a.M) continue;
            const float delta = token_step[gn - n0], sx = token_sum[gn - n0];
            half8_t o;
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const float av = (float)sum[e];
                const int row = c8 * 8 + e;
                o[e] = (_Float16)(HZ ? delta * fmaf(row_scale[row], av, -row_zs[row] * sx)
                                     : delta * row_scale[row] * fmaf(2.f, av, -sx));
            }
            *reinterpret_cast<half8_t*>(a.y + (size_t)gn * a.M + gm) = o;  // (M is a multiple of 8)
            if (a.acc_out) {
#pragma unroll
                for (int t = 0; t < 8; ++t) a.acc_out[(size_t)gn * a.M + gm + t] = sum[t];
            }
        }
        __syncthreads();
    }
}

template <int B, bool HZ, int RBW, int TT>
static int launch_i8_ksplit(GemmI8Args a, int group, hipStream_t st) {
    using T = I8KsTile<RBW, TT>;
    static std::once_flag once;
    static hipError_t attr_rc = hipSuccess;
    std::call_once(once, [] {
        attr_rc = hipFuncSetAttribute(reinterpret_cast<const void*>(&mpgemm_i8_ksplit_kernel<B, HZ, RBW, TT>),
                                      hipFuncAttributeMaxDynamicSharedMemorySize, T::LdsBytes);
    });
    if (attr_rc != hipSuccess) return TMAN_ERR_LAUNCH;
    a.m_tiles = (a.n_row_blocks + RBW - 1) / RBW;
    a.n_tiles = (a.N + T::TN - 1) / T::TN;
    hipLaunchKernelGGL((mpgemm_i8_ksplit_kernel<B, HZ, RBW, TT>), dim3((unsigned)(a.m_tiles * a.n_tiles)), dim3(256),
                       T::LdsBytes, st, a, group);
    return launch_status();
}

template <int B, int GQ, bool HZ>
static int launch_i8_cfg(GemmI8Args a, hipStream_t st) {
    static std::once_flag once;
    static hipError_t attr_rc = hipSuccess;
    std::call_once(once, [] {
        attr_rc = hipFuncSetAttribute(reinterpret_cast<const void*>(&mpgemm_i8_kernel<B, GQ, HZ>),
                                      hipFuncAttributeMaxDynamicSharedMemorySize, kI8LdsBytes);
    });
    if (attr_rc != hipSuccess) return TMAN_ERR_LAUNCH;
    a.m_tiles = (a.n_row_blocks + 1) / 2;
    a.n_tiles = (a.N + kI8Tokens - 1) / kI8Tokens;
    hipLaunchKernelGGL((mpgemm_i8_kernel<B, GQ, HZ>), dim3((unsigned)(a.m_tiles * a.n_tiles)), dim3(256), kI8LdsBytes, st, a);
    return launch_status();
}

template <int B, bool HZ>
static int launch_i8_group(int group, const GemmI8Args& a, hipStream_t st) {
    switch (group) {
        case 32: return launch_i8_cfg<B, 32, HZ>(a, st);
        case 64: return launch_i8_cfg<B, 64, HZ>(a, st);
        default: return launch_i8_cfg<B, 128, HZ>(a, st);
    }
}

template <int B, bool HZ>
static int launch_i8_wide_tokens(int tt, const GemmI8Args& a, int group, hipStream_t st) {
    switch (tt) {
        case 3: return launch_i8_wide<B, HZ, 3>(a, group, st);
        case 4: return launch_i8_wide<B, HZ, 4>(a, group, st);
        case 9: return launch_i8_ksplit<B, HZ, 2, 4>(a, group, st);
        default: return launch_i8_wide<B, HZ, 7>(a, group, st);
    }
}

// Which kernel, and for the wide one how many 32-token blocks per workgroup: the choice with the least modelled
// time.  The model counts rounds of workgroups over the compute units with the time of one workgroup (alone on its unit /
// sharing it with a second one, which the 96- and 128-token tiles allow), scaled by K; the 128 x 128 kernel's time grows
// linearly with its workgroups.  1 = that kernel, 3 / 4 / 7 = the wide kernel with that many 32-token blocks, 9 = the kernel
// whose waves split K.  Its constants weigh the candidates against each other; they are larger than the times of the present
// kernels.  Calls of 64 / 128 / 256 / 384 / 512 workgroups take, at K = 4096 and 4 bits, in microseconds:
//   3 (96 tokens)  23 / 25 / 32 / 46 / 53    9 (K split)    18 / 19 / 24 / 40 / 46
//   4 (128)        27 / 29 / 38 / 55 / 64    1 (128 x 128)  27 / 28 / 29 / 40 / 46
//   7 (224)        42 / 44 / 57 / 99 / 115
// From K = 2048 on the rule picks the fastest or one within 1 % of it at 33 of 33 shapes (random ones of 256 .. 12288 rows and 33 ..
// 2048 tokens).  Below it does not: the 128 x 128 kernel has no fixed part here and the K-split kernel is not asked, so at 22 of 27
// shapes the 96-token or the K-split kernel takes 3 to 19 % less (640 x 1792 N = 56: 14.1 us, K split 11.5; 4096 x 1024 N = 512 12.0,
// 96 tokens 10.3).
int choose_i8_token_blocks(int n_row_blocks, int N, int K) {
    static std::once_flag once;
    static int n_cu = 256;  // assumed when no device answers
    std::call_once(once, [] {
        int dev = 0, n = 0;
        if (hipGetDevice(&dev) == hipSuccess &&
            hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && n > 0)
            n_cu = n;
    });
    const int forced = current_tiling().i8_token_blocks;
    if (forced == 1 || forced == 3 || forced == 4 || forced == 7 || forced == 9) return forced;
    const double k = (double)K / 4096.0;
    const long long old_wgs = (long long)((n_row_blocks + 1) / 2) * ((N + kI8Tokens - 1) / kI8Tokens);
    double best_cost = (17.0 + 0.08 * (double)old_wgs * 256.0 / n_cu) * k;
    int best = 1;
    const int tts[3] = {7, 4, 3};
    const double alone[3] = {59.0, 40.0, 35.0}, shared[3] = {0.0, 58.0, 52.0};
    for (int i = 0; i < 3; ++i) {
        const long long wgs = (long long)((n_row_blocks + 3) / 4) * ((N + 32 * tts[i] - 1) / (32 * tts[i]));
        double cost;
        if (tts[i] > 4) {
            cost = (double)((wgs + n_cu - 1) / n_cu) * alone[i];
        } else {
            const long long full = wgs / (2 * n_cu), rem = wgs % (2 * n_cu);
            cost = (double)full * shared[i] + (rem == 0 ? 0.0 : rem > n_cu ? shared[i] : alone[i]);
        }
        cost *= k;
        if (cost < best_cost) {
            best_cost = cost;
            best = tts[i];
        }
    }
    // the kernel whose waves split K (128 rows x 128 tokens, one workgroup per unit): 17 us per round on an almost
    // empty chip, 22.5 when every unit streams activations
    if (K >= 2048) {
        const long long wgs = (long long)((n_row_blocks + 1) / 2) * ((N + 127) / 128);
        const double fill = wgs >= n_cu ? 1.0 : (double)wgs / n_cu;
        const double cost = (double)((wgs + n_cu - 1) / n_cu) * (16.5 + 6.0 * fill) * k;
        if (cost < best_cost) {
            best_cost = cost;
            best = 9;
        }
    }
    return best;
}

int launch_mpgemm_i8(const Layout& L, const void* packed, const void* xq_buf, int N, void* y, void* acc_out, hipStream_t st) {
    const ActI8Layout al = act_i8_layout(N, L.K);
    const uint8_t* xb = static_cast<const uint8_t*>(xq_buf);
    GemmI8Args a;
    a.tiles = static_cast<const uint8_t*>(packed) + kHeaderBytes;
    a.xq = reinterpret_cast<const int8_t*>(xb);
    a.absmax = reinterpret_cast<const float*>(xb + al.absmax_off);
    a.sums = reinterpret_cast<const int32_t*>(xb + al.sum_off);
    a.y = static_cast<_Float16*>(y);
    a.acc_out = static_cast<int32_t*>(acc_out);
    a.M = L.M;
    a.N = N;
    a.K = L.K;
    a.n_row_blocks = L.n_row_blocks;
    a.n_ktiles = L.n_ktiles;
    a.m_tiles = a.n_tiles = 0;
    a.status = device_status_word();
    if (!a.status) return TMAN_ERR_LAUNCH;
    const int tt = choose_i8_token_blocks(L.n_row_blocks, N, L.K);
    if (tt > 1) {
        if (L.bits == 1)
            return L.has_zero ? launch_i8_wide_tokens<1, true>(tt, a, L.group, st) : launch_i8_wide_tokens<1, false>(tt, a, L.group, st);
        if (L.bits == 2) return launch_i8_wide_tokens<2, true>(tt, a, L.group, st);
        return launch_i8_wide_tokens<4, true>(tt, a, L.group, st);
    }
    if (L.bits == 1) return L.has_zero ? launch_i8_group<1, true>(L.group, a, st) : launch_i8_group<1, false>(L.group, a, st);
    if (L.bits == 2) return launch_i8_group<2, true>(L.group, a, st);
    return launch_i8_group<4, true>(L.group, a, st);
}

}  // namespace tman
