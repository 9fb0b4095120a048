// Lookup-table precompute for decoding (Sec. 2.2 "Bit-serial table lookup"; Sec. 5 "Graph
// optimization" makes it a kernel of its own so several GEMVs share one table).
//
// For every group j of 4 consecutive activations and every 4-bit pattern p the table holds
//   T[n][j][p] = sum_{t<4, bit t of p} x[n][4j+t]
// as a 16-bit entry (Sec. 5: 16-entry tables with 16-bit entries), here fp16 rounded once from an
// fp32 sum taken in ascending t.  The fp32 sums S[n][G] of x over each quantization block follow;
// the GEMV needs them for the zero-point term.
//
// Buffer layout (tokens padded to NP = 1, 2, 4 or 8; K padded to a multiple of 128 with zeros):
//   fp16 element (j * 16 + p) * NP + n          for j < n_ktiles * 32
//   fp32 element  G * NP + n                    at byte offset n_ktiles * 1024 * NP, G < n_ktiles * 128 / group
// so the slice of one K tile is contiguous and can be copied to LDS as it is.
//
// One launch serves up to 8 activations (the distinct inputs of a decode step): the second grid dimension is the activation.
// One fp16 token: a thread builds one table; several tokens and integer tables: four threads share a table of all tokens.
#include <hip/hip_fp16.h>

#include "tman_internal.h"

namespace tman {

struct LutJob {
    const _Float16* x;
    _Float16* T;
    float* S;
    int K, n_tables;
};
constexpr int kLutJobsPerLaunch = 8;  // kernel arguments stay small
struct LutJobs {
    LutJob job[kLutJobsPerLaunch];
    int count, N, group;
};

typedef _Float16 half8_t __attribute__((ext_vector_type(8)));

// One token: one thread per table j.  Consecutive lanes own consecutive tables, so the group sum of a quantization block
// (group / 4 tables) is a butterfly over adjacent lanes.
__global__ void __launch_bounds__(256) build_lut_kernel(LutJobs a) {
    // grid = (blocks of the longest activation) x (activations): no search for the job
    const LutJob& jb = a.job[blockIdx.y];
    const int K = jb.K;
    if ((int)blockIdx.x * 256 >= jb.n_tables) return;
    const int j = (int)blockIdx.x * 256 + threadIdx.x;  // n_tables is a multiple of 32
    const bool live = j < jb.n_tables;
    float v[4] = {0.f, 0.f, 0.f, 0.f};
    if (live) {
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const int k = 4 * j + t;
            if (k < K) v[t] = (float)jb.x[k];
        }
    }
    _Float16 e[16];
#pragma unroll
    for (int p = 0; p < 16; ++p) {
        float s = 0.f;
#pragma unroll
        for (int t = 0; t < 4; ++t)
            if ((p >> t) & 1) s += v[t];
        e[p] = (_Float16)s;  // round to nearest even
    }
    if (live) {
        half8_t lo, hi;
#pragma unroll
        for (int p = 0; p < 8; ++p) {
            lo[p] = e[p];
            hi[p] = e[p + 8];
        }
        half8_t* dst = reinterpret_cast<half8_t*>(jb.T + (size_t)j * 16);
        dst[0] = lo;
        dst[1] = hi;
    }
    // group sums: add the four activations, then the group / 4 tables of the block
    float s = (v[0] + v[1]) + (v[2] + v[3]);
    const int tables_per_group = a.group / kLutGroup;  // 8, 16 or 32: within one wave
    for (int d = 1; d < tables_per_group; d <<= 1) s += __shfl_xor(s, d, 64);
    if (live && (j % tables_per_group) == 0) jb.S[j / tables_per_group] = s;
}

// Several tokens: four threads per table j, thread q makes entries 4 q .. 4 q + 3 (activations 2 and 3 as the bits of q say, 0 and 1
// in all four combinations) of all NP tokens, 8 NP bytes, so that a wave stores whole lines and four times as many waves
// share the wait for the activations.  Same sums, same roundings.  The four activations of a 7B layer, NP = 4, take
// 3.2 us, NP = 8 3.5 us (one thread per table: 3.8 and 5.8).
template <int NP>
__global__ void __launch_bounds__(256) build_lut_tokens_kernel(LutJobs a) {
    const LutJob& jb = a.job[blockIdx.y];
    const int N = a.N, K = jb.K;
    const int j = (int)blockIdx.x * 64 + ((int)threadIdx.x >> 2), q = threadIdx.x & 3;  // n_tables is a multiple of 32
    if ((int)blockIdx.x * 64 >= jb.n_tables) return;
    const bool live = j < jb.n_tables, inside = live && 4 * j < K;  // K is a multiple of 32
    const bool wide = (reinterpret_cast<uintptr_t>(jb.x) & 7u) == 0;  // (a row is K * 2 bytes, a multiple of 64)
    typedef _Float16 half4_t __attribute__((ext_vector_type(4)));
    half4_t h[NP];
#pragma unroll
    for (int n = 0; n < NP; ++n) {
        h[n] = half4_t{(_Float16)0.f, (_Float16)0.f, (_Float16)0.f, (_Float16)0.f};
        if (inside && n < N) {
            const _Float16* src = jb.x + (size_t)n * K + 4 * j;
            if (wide) {
                h[n] = *reinterpret_cast<const half4_t*>(src);
            } else {
#pragma unroll
                for (int t = 0; t < 4; ++t) h[n][t] = src[t];
            }
        }
    }
    _Float16 e[4][NP];
    float gs[NP];
#pragma unroll
    for (int n = 0; n < NP; ++n) {
        const float v[4] = {(float)h[n][0], (float)h[n][1], (float)h[n][2], (float)h[n][3]};
#pragma unroll
        for (int p = 0; p < 4; ++p) {
            float s = 0.f;
            if (p & 1) s += v[0];
            if (p & 2) s += v[1];
            s = q & 1 ? s + v[2] : s;
            s = q & 2 ? s + v[3] : s;
            e[p][n] = (_Float16)s;  // round to nearest even
        }
        gs[n] = (v[0] + v[1]) + (v[2] + v[3]);
    }
    if (live) {
        constexpr int PER = 8 / NP;  // entry rows per 16-byte store
        half8_t* dst = reinterpret_cast<half8_t*>(jb.T + ((size_t)j * 16 + 4 * q) * NP);
#pragma unroll
        for (int o = 0; o < 4 / PER; ++o) {
            half8_t w;
#pragma unroll
            for (int i = 0; i < 8; ++i) w[i] = e[o * PER + i / NP][i % NP];
            dst[o] = w;
        }
    }
    // group sums: lanes 4 i of a wave hold 16 tables, a quantization block is 8, 16 or 32 tables
    __shared__ float sums[64][NP];
    if (q == 0) {
#pragma unroll
        for (int n = 0; n < NP; ++n) sums[threadIdx.x >> 2][n] = gs[n];
    }
    __syncthreads();
    const int tables_per_group = a.group / kLutGroup, groups = 64 / tables_per_group;
    const int gi = (int)threadIdx.x / NP, n = (int)threadIdx.x % NP;
    const int j0 = (int)blockIdx.x * 64 + gi * tables_per_group;
    if (gi < groups && j0 < jb.n_tables) {
        // the tables of the block in pairs, pairs of pairs, ...: the order of the butterfly over one lane per table
        float s[32];
#pragma unroll
        for (int i = 0; i < 32; ++i) s[i] = i < tables_per_group ? sums[gi * tables_per_group + i][n] : 0.f;
#pragma unroll
        for (int d = 1; d < 32; d <<= 1)
#pragma unroll
            for (int i = 0; i + d < 32; i += 2 * d) s[i] += s[i + d];
        jb.S[(size_t)(j0 / tables_per_group) * NP + n] = s[0];
    }
}

int launch_build_lut_batch(int count, const void* const* x, int N, const int* K, int group, void* const* lut,
                           hipStream_t st) {
    const int NP = padded_tokens(N);
    for (int i0 = 0; i0 < count; i0 += kLutJobsPerLaunch) {
        LutJobs a;
        a.count = count - i0 < kLutJobsPerLaunch ? count - i0 : kLutJobsPerLaunch;
        a.N = N;
        a.group = group;
        int blocks = 0;  // of the longest activation
        for (int i = 0; i < kLutJobsPerLaunch; ++i) {
            const int src = i0 + (i < a.count ? i : 0);
            const int nkt = (K[src] + kKTile - 1) / kKTile;
            LutJob& jb = a.job[i];
            jb.x = static_cast<const _Float16*>(x[src]);
            jb.T = static_cast<_Float16*>(lut[src]);
            jb.S = reinterpret_cast<float*>(static_cast<uint8_t*>(lut[src]) + (size_t)nkt * kTableBytesPerKTile * NP);
            jb.K = K[src];
            jb.n_tables = nkt * kTablesPerKTile;
            const int b = NP == 1 ? (jb.n_tables + 255) / 256 : (jb.n_tables + 63) / 64;
            if (i < a.count && b > blocks) blocks = b;
        }
        const dim3 grid((unsigned)blocks, (unsigned)a.count);
        if (NP == 1) hipLaunchKernelGGL(build_lut_kernel, grid, dim3(256), 0, st, a);
        else if (NP == 2) hipLaunchKernelGGL(build_lut_tokens_kernel<2>, grid, dim3(256), 0, st, a);
        else if (NP == 4) hipLaunchKernelGGL(build_lut_tokens_kernel<4>, grid, dim3(256), 0, st, a);
        else hipLaunchKernelGGL(build_lut_tokens_kernel<8>, grid, dim3(256), 0, st, a);
    }
    return launch_status();
}

// ---------------------------------------------------------------------------------------------
// Integer tables (Sec. 6.1 "A_INT16"; Sec. 5: 16-bit table entries).
//
// Every token gets a power-of-two step 2^e, the smallest for which all |x| / 2^e <= 8191, and integer
// activations xq = round_to_nearest_even(x / 2^e); four of them always sum to a 16-bit integer, so the table
//   Tq[n][j][p] = sum_{t<4, bit t of p} xq[n][4j+t]
// is exact.  Dividing an fp16 number by a power of two is exact in fp32, so xq does not depend on the precision
// it is computed in.  With the largest |x| = m * 2^E (0.5 <= m < 1), e = E - 13; a token of zeros gets e = 0.
// The activations must be finite.
//
// Buffer layout: as the fp16 tables (int16 element (j * 16 + p) * NP + n, then the int32 block sums, element
// G * NP + n), followed by the int32 exponents e[n], n < NP.
//
// Every block first finds the largest magnitude of its tokens, T of the block's threads to a token.
template <int T>
__device__ __forceinline__ unsigned largest_of_token(const uint16_t* xb, int K, int t) {
    unsigned mx = 0;  // magnitudes compare like their bit patterns
    // 16 bytes per thread and step where the row allows it (K is a multiple of 32; the row start is 16-byte
    // aligned when x is and K * 2 is a multiple of 16, which it is)
    if ((reinterpret_cast<uintptr_t>(xb) & 15u) == 0) {
        // (six requests at once, past the row they read as zero: one after the other they were half of the launch)
        const __amdgpu_buffer_rsrc_t rx = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(xb), 0, (uint32_t)K * 2u, 0x00020000);
        for (uint32_t c = t; c < (uint32_t)K / 8u; c += 6 * T) {
            typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
            u32x4_t w[6];
#pragma unroll
            for (int u = 0; u < 6; ++u) w[u] = __builtin_amdgcn_raw_buffer_load_b128(rx, (c + u * T) * 16u, 0, 0);
#pragma unroll
            for (int u = 0; u < 6; ++u)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const uint32_t d = w[u][i] & 0x7fff7fffu;
                    mx = max(mx, max(d & 0xffffu, d >> 16));
                }
        }
    } else {
        for (int k = t; k < K; k += T) mx = max(mx, (unsigned)(xb[k] & 0x7fffu));
    }
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) mx = max(mx, (unsigned)__shfl_xor((int)mx, d, 64));
    return mx;
}
// Exponent of the step for a largest magnitude with this bit pattern.
__device__ __forceinline__ int step_exponent(unsigned mx) {
    if (mx == 0) return 0;
    const int eb = (int)(mx >> 10), f = (int)(mx & 0x3ffu);
    // normal: (1024 + f) * 2^(eb - 25) lies in [2^(eb - 15), 2^(eb - 14)); subnormal: f * 2^-24
    const int E = eb != 0 ? eb - 14 : (32 - __builtin_clz((unsigned)f)) - 24;
    return E - 13;
}

// As for fp16 entries: four threads per table, thread q makes entries 4 q .. 4 q + 3 of the block's tokens, all or half of 8.  At
// least 128 threads search a token, because every block searches all of its tokens, six requests at a time.  The launch for four
// activations of a 7B layer takes 3.5 / 4.0 / 5.0 / 5.5 us for NP = 1 / 2 / 4 / 8, for one activation of 4096 3.5 / 3.6 / 4.4 / 4.6 (a
// block per token, whose threads stored two bytes at a time: 5.3 / 5.7 / 6.5 / 10.7 and 4.5 / 4.8 / 5.1 / 5.1; all 8 tokens in a block
// of 1024 threads: 8.2 and 7.0).
constexpr int i16_tokens(int np) { return np < 4 ? np : 4; }  // per block
constexpr int i16_threads(int np) { return np <= 2 ? 256 : 512; }
template <int NP>
__global__ void __launch_bounds__(i16_threads(NP)) build_lut_i16_kernel(LutJobs a) {
    constexpr int kThreads = i16_threads(NP), kTables = kThreads / 4, TB = i16_tokens(NP);
    __shared__ unsigned largest[TB][4];
    __shared__ int sums[kTables][TB];
    const LutJob& jb = a.job[blockIdx.y];
    const int n0 = (int)blockIdx.z * TB;  // the block's first token
    const int N = a.N - n0, K = jb.K, tid = threadIdx.x;
    const int j = (int)blockIdx.x * kTables + (tid >> 2), q = tid & 3;  // n_tables is a multiple of 32
    if ((int)blockIdx.x * kTables >= jb.n_tables) return;
    const bool live = j < jb.n_tables, inside = live && 4 * j < K;  // K is a multiple of 32
    const uint16_t* const x = reinterpret_cast<const uint16_t*>(jb.x) + (size_t)n0 * K;
    const bool wide = (reinterpret_cast<uintptr_t>(x) & 7u) == 0;  // (a row is K * 2 bytes, a multiple of 64)
    typedef uint16_t u16x4_t __attribute__((ext_vector_type(4)));
    u16x4_t own[TB];  // requested before the search
#pragma unroll
    for (int n = 0; n < TB; ++n) {
        own[n] = u16x4_t{0, 0, 0, 0};
        if (inside && n < N) {
            const uint16_t* src = x + (size_t)n * K + 4 * j;
            if (wide) {
                own[n] = *reinterpret_cast<const u16x4_t*>(src);
            } else {
#pragma unroll
                for (int t = 0; t < 4; ++t) own[n][t] = src[t];
            }
        }
    }
    constexpr int T = kThreads / TB;        // threads per token
    constexpr int W = T / 64;               // waves per token
    {
        const int n = tid / T, t = tid % T;
        const unsigned mx = n < N ? largest_of_token<T>(x + (size_t)n * K, K, t) : 0u;
        if (t % 64 == 0) largest[n][t / 64] = mx;
    }
    __syncthreads();
    int* const S = reinterpret_cast<int*>(jb.S);
    int* const ex = S + (size_t)(jb.n_tables / kTablesPerKTile) * (kKTile / a.group) * NP;
    int16_t e[4][TB];
#pragma unroll
    for (int n = 0; n < TB; ++n) {
        unsigned mx = largest[n][0];
#pragma unroll
        for (int w = 1; w < W; ++w) mx = max(mx, largest[n][w]);
        const int exponent = step_exponent(mx);
        if (blockIdx.x == 0 && tid == 0) ex[n0 + n] = exponent;
        int v[4];
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const uint16_t bits = own[n][t];  // (copied out before the cast)
            v[t] = (int)rintf(ldexpf((float)__builtin_bit_cast(_Float16, bits), -exponent));
        }
        const int high = (q & 1 ? v[2] : 0) + (q & 2 ? v[3] : 0);
#pragma unroll
        for (int p = 0; p < 4; ++p) e[p][n] = (int16_t)((p & 1 ? v[0] : 0) + (p & 2 ? v[1] : 0) + high);
        if (q == 0) sums[tid >> 2][n] = (v[0] + v[1]) + (v[2] + v[3]);
    }
    if (live) {
        int16_t* const dst = reinterpret_cast<int16_t*>(jb.T) + ((size_t)j * 16 + 4 * q) * NP + n0;
        if constexpr (NP == 8) {  // half of each entry row
            typedef int16_t i16x4_t __attribute__((ext_vector_type(4)));
#pragma unroll
            for (int p = 0; p < 4; ++p) *reinterpret_cast<i16x4_t*>(dst + p * NP) = i16x4_t{e[p][0], e[p][1], e[p][2], e[p][3]};
        } else if constexpr (NP == 1) {
            typedef int16_t i16x4_t __attribute__((ext_vector_type(4)));
            *reinterpret_cast<i16x4_t*>(dst) = i16x4_t{e[0][0], e[1][0], e[2][0], e[3][0]};
        } else {
            typedef int16_t i16x8_t __attribute__((ext_vector_type(8)));
            constexpr int PER = 8 / NP;  // entry rows per 16-byte store
#pragma unroll
            for (int o = 0; o < 4 / PER; ++o) {
                i16x8_t w;
#pragma unroll
                for (int i = 0; i < 8; ++i) w[i] = e[o * PER + i / NP][i % NP];
                reinterpret_cast<i16x8_t*>(dst)[o] = w;
            }
        }
    }
    __syncthreads();
    const int tables_per_group = a.group / kLutGroup, groups = kTables / tables_per_group;
    const int gi = tid / TB, n = tid % TB, j0 = (int)blockIdx.x * kTables + gi * tables_per_group;
    if (gi < groups && j0 < jb.n_tables) {
        int s = 0;
#pragma unroll 8
        for (int i = 0; i < tables_per_group; ++i) s += sums[gi * tables_per_group + i][n];  // (8, 16 or 32)
        S[(size_t)(j0 / tables_per_group) * NP + n0 + n] = s;
    }
}

int launch_build_lut_i16_batch(int count, const void* const* x, int N, const int* K, int group, void* const* lut,
                               hipStream_t st) {
    const int NP = padded_tokens(N);
    for (int i0 = 0; i0 < count; i0 += kLutJobsPerLaunch) {
        LutJobs a;
        a.count = count - i0 < kLutJobsPerLaunch ? count - i0 : kLutJobsPerLaunch;
        a.N = N;
        a.group = group;
        int blocks = 0;  // of the longest activation
        for (int i = 0; i < kLutJobsPerLaunch; ++i) {
            const int src = i0 + (i < a.count ? i : 0);
            const int nkt = (K[src] + kKTile - 1) / kKTile;
            LutJob& jb = a.job[i];
            jb.x = static_cast<const _Float16*>(x[src]);
            jb.T = static_cast<_Float16*>(lut[src]);
            jb.S = reinterpret_cast<float*>(static_cast<uint8_t*>(lut[src]) + (size_t)nkt * kTableBytesPerKTile * NP);
            jb.K = K[src];
            jb.n_tables = nkt * kTablesPerKTile;
            const int per = i16_threads(NP) / 4, b = (jb.n_tables + per - 1) / per;
            if (i < a.count && b > blocks) blocks = b;
        }
        const dim3 grid((unsigned)blocks, (unsigned)a.count, (unsigned)(NP / i16_tokens(NP)));
        if (NP == 1) hipLaunchKernelGGL(build_lut_i16_kernel<1>, grid, dim3(256), 0, st, a);
        else if (NP == 2) hipLaunchKernelGGL(build_lut_i16_kernel<2>, grid, dim3(256), 0, st, a);
        else if (NP == 4) hipLaunchKernelGGL(build_lut_i16_kernel<4>, grid, dim3(i16_threads(4)), 0, st, a);
        else hipLaunchKernelGGL(build_lut_i16_kernel<8>, grid, dim3(i16_threads(8)), 0, st, a);
    }
    return launch_status();
}

int launch_build_lut(const void* x, int N, int K, int group, void* lut, hipStream_t st) {
    return launch_build_lut_batch(1, &x, N, &K, group, &lut, st);
}

}  // namespace tman
