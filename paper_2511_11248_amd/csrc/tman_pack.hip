// Offline weight repacking into the unified bit-serial layout, and its inverse.
//
// Sec. 4.1 ("Unified Layout through Fused LUT-based Dequantization") stores the weights bit-serially,
// the form decoding needs, and pre-permutes them so both kernels fetch contiguous blocks.  One thread turns 32
// consecutive codes of one row into `bits` one-bit planes (Sec. 2.2 one-bit decomposition) and writes their words
// at the position the layout function assigns; one launch writes the whole blob, header, planes and group
// parameters.  The padded domain (rows up to a multiple of 64, columns up to a multiple of 128) is covered too, so
// the blob is completely defined.
//
// Bound by memory: 45 MB of codes in, 25 MB out (11008 x 4096, uint4 g64) in 20 us = 3.6 TB/s (a large copy reaches 4.85);
// with a thread per 32 codes reading byte by byte along a row, and launches of their own for header and parameters,
// it took 108 us.  With one tile per workgroup it takes 22.6 us.
#include "tman_internal.h"

namespace tman {

struct PackGeom {
    int M, K, bits, group, has_zero;
    int n_ktiles, n_row_blocks, tile_bytes, meta_per_lane, meta_entry;
};

static PackGeom geom_of(const Layout& L) {
    return PackGeom{L.M, L.K, L.bits, L.group, L.has_zero, L.n_ktiles, L.n_row_blocks, L.tile_bytes, L.meta_per_lane,
                    L.meta_entry};
}

// byte offset (from the blob start) of the 32-bit word holding plane i of weights k32*32 .. +31 of row m
__device__ __forceinline__ size_t word_offset(const PackGeom& g, int m, int k32, int i) {
    int rb = m / kRows, lane = m % kRows;
    int k = k32 << 5;
    int kt = k / kKTile, kk = k % kKTile;
    int chunk = kKTile / g.bits;  // weights per 16-byte chunk
    int v = kk / chunk, kc = kk % chunk;
    int ksub = kc >> 5;
    return (size_t)kHeaderBytes + ((size_t)rb * g.n_ktiles + kt) * g.tile_bytes + v * 1024 + lane * 16 +
           (ksub * g.bits + i) * 4;
}

// byte offset of the scale of (row m, quantization group G); the zero follows at +2
__device__ __forceinline__ size_t meta_offset(const PackGeom& g, int m, int G) {
    int rb = m / kRows, lane = m % kRows;
    int k0 = G * g.group;
    int kt = k0 / kKTile, gi = (k0 % kKTile) / g.group;
    return (size_t)kHeaderBytes + ((size_t)rb * g.n_ktiles + kt) * g.tile_bytes + g.bits * 1024 +
           lane * g.meta_per_lane + gi * g.meta_entry;
}

__device__ __forceinline__ int32_t header_word(const PackGeom& g, int t) {
    switch (t) {
        case 0: return 0x4e414d54;  // "TMAN"
        case 1: return 0x00314b50;  // "PK1\0"
        case 2: return g.M;
        case 3: return g.K;
        case 4: return g.bits;
        case 5: return g.group;
        case 6: return g.has_zero;
        case 7: return kRows;
        case 8: return kKTile;
        case 9: return g.n_row_blocks;
        case 10: return g.n_ktiles;
        case 11: return g.tile_bytes;
        case 12: return kHeaderBytes;
        case 13: return kLayoutVersion;
        default: return 0;
    }
}

typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));

// A workgroup writes `tiles` consecutive tile blocks of one row block: four threads share a row of a tile (32 codes
// each: together the 128 bytes of a cache line), so a wave reads 16 such lines and writes runs of 256 bytes.  Several
// tiles per workgroup let it read the scales of a row in one piece.  WIDE: the codes are 16-byte aligned (a row is,
// because K is a multiple of 32, when the first one is); otherwise they are read byte by byte.
template <int B, bool WIDE>
__global__ void __launch_bounds__(256) pack_kernel(PackGeom g, const uint8_t* __restrict__ codes,
                                                   const uint16_t* __restrict__ scales, const uint16_t* __restrict__ zeros,
                                                   uint8_t* __restrict__ packed, int tiles, int chunks) {
    const int rb = (int)(blockIdx.x / (unsigned)chunks);
    const int kt0 = (int)(blockIdx.x % (unsigned)chunks) * tiles, kt1 = min(kt0 + tiles, g.n_ktiles);
    const int tid = threadIdx.x;
    if (blockIdx.x == 0 && tid < kHeaderBytes / 4) reinterpret_cast<int32_t*>(packed)[tid] = header_word(g, tid);

    // codes -> planes
    const int row = tid >> 2, kb = tid & 3, m = rb * kRows + row;
    for (int kt = kt0; kt < kt1; ++kt) {
        const int k = kt * kKTile + kb * 32;
        uint32_t w[8] = {0u, 0u, 0u, 0u, 0u, 0u, 0u, 0u};
        if (m < g.M && k < g.K) {  // K is a multiple of 32, so a block is entirely inside or outside
            const uint8_t* src = codes + (size_t)m * g.K + k;
            if constexpr (WIDE) {
                const u32x4_t lo = __builtin_nontemporal_load(reinterpret_cast<const u32x4_t*>(src));
                const u32x4_t hi = __builtin_nontemporal_load(reinterpret_cast<const u32x4_t*>(src) + 1);
#pragma unroll
                for (int i = 0; i < 4; ++i) w[i] = lo[i], w[4 + i] = hi[i];
            } else {
#pragma unroll
                for (int t = 0; t < 32; ++t) w[t / 4] |= (uint32_t)src[t] << (8 * (t % 4));
            }
        }
        // bit i of the four codes of a word, times 1, 2, 4, 8 (16 ..): a dot product of bytes; the sum of eight codes is
        // 2^i times a byte of the plane
        uint32_t plane[B];
#pragma unroll
        for (int i = 0; i < B; ++i) {
            plane[i] = 0u;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                uint32_t s = __builtin_amdgcn_udot4(w[2 * q] & (0x01010101u << i), 0x08040201u, 0u, false);
                s = __builtin_amdgcn_udot4(w[2 * q + 1] & (0x01010101u << i), 0x80402010u, s, false);
                plane[i] |= (s >> i) << (8 * q);
            }
        }
        uint32_t* dst = reinterpret_cast<uint32_t*>(packed + word_offset(g, m, kt * (kKTile / 32) + kb, 0));
        if constexpr (B == 4) {
            *reinterpret_cast<u32x4_t*>(dst) = u32x4_t{plane[0], plane[1], plane[2], plane[3]};
        } else if constexpr (B == 2) {
            *reinterpret_cast<uint64_t*>(dst) = (uint64_t)plane[1] << 32 | plane[0];
        } else {
            *dst = plane[0];
        }
    }

    // scales and zeros: thread -> (row, quantization group of the chunk), groups fastest
    const int gpt = kKTile / g.group, G_real = g.K / g.group, n_groups = (kt1 - kt0) * gpt;
    for (int i = tid; i < kRows * n_groups; i += 256) {
        const int r = i / n_groups, G = kt0 * gpt + i % n_groups, mm = rb * kRows + r;
        uint32_t s = 0, z = 0;
        if (mm < g.M && G < G_real) {
            s = scales[(size_t)mm * G_real + G];
            if (g.has_zero) z = zeros[(size_t)mm * G_real + G];
        }
        uint8_t* dst = packed + meta_offset(g, mm, G);
        if (g.has_zero) *reinterpret_cast<uint32_t*>(dst) = z << 16 | s;
        else *reinterpret_cast<uint16_t*>(dst) = (uint16_t)s;
    }
}

__global__ void __launch_bounds__(256) unpack_codes_kernel(PackGeom g, const uint8_t* __restrict__ packed,
                                                           uint8_t* __restrict__ codes) {
    int k32_n = g.K / 32;
    long long tid = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    long long total = (long long)g.M * k32_n;
    if (tid >= total) return;
    int m = (int)(tid / k32_n), k32 = (int)(tid % k32_n);
    uint32_t plane[4] = {0u, 0u, 0u, 0u};
    for (int i = 0; i < g.bits; ++i) plane[i] = *reinterpret_cast<const uint32_t*>(packed + word_offset(g, m, k32, i));
    uint8_t* dst = codes + (size_t)m * g.K + (size_t)k32 * 32;
    for (int t = 0; t < 32; ++t) {
        uint32_t c = 0;
        for (int i = 0; i < g.bits; ++i) c |= ((plane[i] >> t) & 1u) << i;
        dst[t] = (uint8_t)c;
    }
}

__global__ void __launch_bounds__(256) unpack_meta_kernel(PackGeom g, const uint8_t* __restrict__ packed,
                                                          uint16_t* __restrict__ scales, uint16_t* __restrict__ zeros) {
    int G_real = g.K / g.group;
    long long tid = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    long long total = (long long)g.M * G_real;
    if (tid >= total) return;
    int m = (int)(tid / G_real), G = (int)(tid % G_real);
    const uint16_t* src = reinterpret_cast<const uint16_t*>(packed + meta_offset(g, m, G));
    if (scales) scales[(size_t)m * G_real + G] = src[0];
    if (zeros && g.has_zero) zeros[(size_t)m * G_real + G] = src[1];
}

static unsigned blocks_for(long long total) { return (unsigned)((total + 255) / 256); }

template <int B>
static void launch_pack_bits(const PackGeom& g, const uint8_t* codes, const uint16_t* scales, const uint16_t* zeros,
                             uint8_t* out, int tiles, hipStream_t st) {
    const int chunks = (g.n_ktiles + tiles - 1) / tiles;
    const dim3 grid((unsigned)((long long)g.n_row_blocks * chunks)), block(256);
    if (aligned16(codes))
        hipLaunchKernelGGL((pack_kernel<B, true>), grid, block, 0, st, g, codes, scales, zeros, out, tiles, chunks);
    else
        hipLaunchKernelGGL((pack_kernel<B, false>), grid, block, 0, st, g, codes, scales, zeros, out, tiles, chunks);
}

int launch_pack(const Layout& L, const uint8_t* codes, const void* scales, const void* zeros, void* packed,
                hipStream_t st) {
    const PackGeom g = geom_of(L);
    const uint16_t *s = static_cast<const uint16_t*>(scales), *z = static_cast<const uint16_t*>(zeros);
    uint8_t* out = static_cast<uint8_t*>(packed);
    // up to 8 tiles per workgroup, fewer when that would leave fewer than 8 workgroups per compute unit
    int tiles = 8;
    while (tiles > 1 && (long long)L.n_row_blocks * ((L.n_ktiles + tiles - 1) / tiles) < 2048) tiles >>= 1;
    if (L.bits == 4) launch_pack_bits<4>(g, codes, s, z, out, tiles, st);
    else if (L.bits == 2) launch_pack_bits<2>(g, codes, s, z, out, tiles, st);
    else launch_pack_bits<1>(g, codes, s, z, out, tiles, st);
    return launch_status();
}

int launch_unpack(const Layout& L, const void* packed, uint8_t* codes, void* scales, void* zeros, hipStream_t st) {
    PackGeom g = geom_of(L);
    const uint8_t* in = static_cast<const uint8_t*>(packed);
    long long n_words = (long long)L.M * (L.K / 32);
    hipLaunchKernelGGL(unpack_codes_kernel, dim3(blocks_for(n_words)), dim3(256), 0, st, g, in, codes);
    if (scales || zeros) {
        long long n_meta = (long long)L.M * (L.K / L.group);
        hipLaunchKernelGGL(unpack_meta_kernel, dim3(blocks_for(n_meta)), dim3(256), 0, st, g, in,
                           static_cast<uint16_t*>(scales), static_cast<uint16_t*>(zeros));
    }
    return launch_status();
}

}  // namespace tman
