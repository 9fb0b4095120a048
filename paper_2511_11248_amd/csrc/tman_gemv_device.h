// Device-side building blocks shared by the kernels that stream tile blocks (decoding, Sec. 2.2 and Sec. 4.3, and the
// small-batch mpGEMM): descriptors and workgroup numbers, requests of tile blocks through buffer loads, LDS access with
// explicit address spaces, the output of a row block and the exchange between K segments.
#pragma once
#include <hip/hip_fp16.h>

#include <type_traits>

#include "tman_internal.h"

namespace tman {

typedef _Float16 half2_t __attribute__((ext_vector_type(2)));
typedef _Float16 half4_t __attribute__((ext_vector_type(4)));
typedef _Float16 half8_t __attribute__((ext_vector_type(8)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

constexpr int kWaves = 4;  // waves per workgroup

template <int B, int NP, int GQ, bool HZ>
struct GemvCfg {
    static constexpr int CH = kKTile / B;    // weights per 16-byte chunk
    static constexpr int GPT = kKTile / GQ;  // quantization groups per tile
    static constexpr int MSZ = HZ ? 4 : 2;
    static constexpr int MPL = GPT * MSZ;    // group-parameter bytes per lane and tile
    static constexpr int TB = B * 1024 + 64 * MPL;
    static constexpr int T_BYTES = kTableBytesPerKTile * NP;
    static constexpr int S_FLOATS = GPT * NP;
    static constexpr int SLOT = T_BYTES + 256;  // table slice + group sums, per wave (multiple of 256)
    // tile blocks in flight per wave.  Measured: more do not help (the waves of a compute unit together
    // keep enough requests in flight) and cost time.
    static constexpr int D = NP >= 4 ? 1 : (B == 2 ? 2 : 3);
};

template <int B, int NP, int MPL>
struct Stage {
    u32x4 c[B];                    // bit-plane chunks
    uint32_t meta[(MPL + 3) / 4];  // scales / zeros of the lane's groups
    u32x4 tt[NP];                  // this lane's 16 bytes of each 1 KB of the table slice
    float sv;                      // one group sum (lanes < S_FLOATS)
};


__device__ __forceinline__ uint32_t word_of(const u32x4& v, int w) {
    return w == 0 ? v.x : w == 1 ? v.y : w == 2 ? v.z : v.w;
}

// Lanes of one wave exchange data through the wave's private LDS slot.  The hardware executes the
// LDS operations of a wave in order; this keeps the compiler from moving them across the exchange.
__device__ __forceinline__ void wave_lds_sync() {
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
}

__device__ __forceinline__ float half_bits_to_float(uint32_t bits16) {
    return (float)__builtin_bit_cast(_Float16, (uint16_t)bits16);
}

// values every lane agrees on, made visibly scalar for the compiler
__device__ __forceinline__ int uniform(int v) { return __builtin_amdgcn_readfirstlane(v); }
template <typename T>
__device__ __forceinline__ T* uniform(T* p) {
    const uint64_t v = reinterpret_cast<uint64_t>(p);
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v), hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
    return reinterpret_cast<T*>(((uint64_t)hi << 32) | lo);
}

// explicit address spaces: descriptor pointers come out of memory as generic pointers, which would
// turn every access into a flat instruction
template <typename T>
using global_ptr = const T __attribute__((address_space(1)))*;
template <typename T>
using lds_ptr = T __attribute__((address_space(3)))*;

// wave-uniform base pointer + 32-bit per-lane byte offset: the form that needs no per-lane
// 64-bit address arithmetic
template <typename T>
__device__ __forceinline__ T load_global(const uint8_t* base, uint32_t off) {
    global_ptr<uint8_t> b = reinterpret_cast<global_ptr<uint8_t>>(reinterpret_cast<uintptr_t>(base));
    return *reinterpret_cast<global_ptr<T>>(b + off);
}
template <typename T>
__device__ __forceinline__ T load_lds(uint32_t addr) {
    return *reinterpret_cast<lds_ptr<const T>>(static_cast<uintptr_t>(addr));
}
template <typename T>
__device__ __forceinline__ void store_lds(uint32_t addr, T v) {
    *reinterpret_cast<lds_ptr<T>>(static_cast<uintptr_t>(addr)) = v;
}

// byte K of x, zero extended, in one full-rate VALU instruction
template <int K>
__device__ __forceinline__ uint32_t byte_of(uint32_t x) {
    uint32_t r;
    if constexpr (K == 0)
        asm("v_and_b32 %0, 0xff, %1" : "=v"(r) : "v"(x));
    else if constexpr (K == 3)
        asm("v_lshrrev_b32 %0, 24, %1" : "=v"(r) : "v"(x));
    else if constexpr (K == 1)
        asm("v_bfe_u32 %0, %1, 8, 8" : "=v"(r) : "v"(x));
    else
        asm("v_bfe_u32 %0, %1, 16, 8" : "=v"(r) : "v"(x));
    return r;
}

// a uniform float the compiler cannot constant-fold, so x * w + acc with fp16 x stays one
// mixed-precision FMA also for w == 1
__device__ __forceinline__ float opaque(float v) {
    asm("" : "+s"(v));
    return v;
}

// Buffer resource over a wave-uniform base: loads then take a 32-bit per-lane offset (constant for
// the whole kernel) plus a scalar offset (the tile), so streaming costs no address arithmetic.
typedef __amdgpu_buffer_rsrc_t rsrc_t;
constexpr int kStreamAux = 2;  // non-temporal: weights are read once, keep them from evicting the tables in L2
__device__ __forceinline__ rsrc_t make_rsrc(const uint8_t* base, uint32_t bytes = 0xFFFFFFFFu) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t*>(base), 0, bytes, 0x00020000);
}

// The three streams a wave reads: its row block's tile blocks, the table slices and the group sums.
struct Streams {
    const uint8_t *w, *t, *s;
    uint32_t w_bytes, t_bytes, s_bytes;
};

// Requests the weights of tile kt: bit-plane chunks and group parameters of the lane's row.  With `live`
// false nothing is fetched and the stage reads as zeros: the caller needs no branch around the request, so
// a tile's lookups and the next request stay one basic block.
template <int B, int NP, int GQ, bool HZ>
__device__ __forceinline__ void issue_weights(Stage<B, NP, GemvCfg<B, NP, GQ, HZ>::MPL>& s, const Streams& src, bool live,
                                              int kt, int lane) {
    using Cfg = GemvCfg<B, NP, GQ, HZ>;
    const rsrc_t rw = make_rsrc(src.w, live ? src.w_bytes : 0u);
    const int so = kt * Cfg::TB;  // scalar offset of the tile block inside the row block
#pragma unroll
    for (int v = 0; v < B; ++v) s.c[v] = __builtin_amdgcn_raw_buffer_load_b128(rw, v * 1024 + lane * 16, so, kStreamAux);
    const int mo = B * 1024 + lane * Cfg::MPL;
    if constexpr (Cfg::MPL == 2) {
        s.meta[0] = __builtin_amdgcn_raw_buffer_load_b16(rw, mo, so, kStreamAux);
    } else if constexpr (Cfg::MPL == 4) {
        s.meta[0] = __builtin_amdgcn_raw_buffer_load_b32(rw, mo, so, kStreamAux);
    } else if constexpr (Cfg::MPL == 8) {
        u32x2 v = __builtin_amdgcn_raw_buffer_load_b64(rw, mo, so, kStreamAux);
        s.meta[0] = v.x;
        s.meta[1] = v.y;
    } else {
        u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(rw, mo, so, kStreamAux);
        s.meta[0] = v.x;
        s.meta[1] = v.y;
        s.meta[2] = v.z;
        s.meta[3] = v.w;
    }
}


// kernel arguments: the descriptor itself for a single GEMV, the device table for a batch
template <bool SINGLE>
struct KernelArgs;
template <>
struct KernelArgs<true> {
    GemvDesc single;
    int n_gemv;   // 1
    int* status;  // the library's status word
};
template <>
struct KernelArgs<false> {
    const GemvDesc* descs;
    int n_gemv;
    int row_blocks;  // one-token kernel, 1 bit: row blocks per workgroup
};

// A batch launch whose workgroups are numbered by the host: workgroup id -> (GEMV, workgroup within the GEMV).
// When all workgroups of a launch are resident at once, this chip's dispatcher hands workgroup i to compute unit
// i mod 256 (measured: ids 8, 264, 520, 776 share a unit), so the numbering decides which workgroups share a
// unit, and the host numbers them so that every unit gets the same amount of work (order_workgroups).
struct OrderedArgs {
    const GemvDesc* descs;
    const uint16_t* order;  // per workgroup id: GEMV in bits 13..15, workgroup within the GEMV in bits 0..12
    int n_gemv;
};

// The batch kernels take the fields of their arguments one by one: scalar arguments are in registers when a wave starts (the
// build asks for it), a structure is read from memory first (0.25 us of a launch).
template <typename Launch>
static void with_fields(const KernelArgs<true>& a, Launch launch) { launch(a); }
template <typename Launch>
static void with_fields(const KernelArgs<false>& a, Launch launch) { launch(a.descs, a.n_gemv, a.row_blocks); }
template <typename Launch>
static void with_fields(const OrderedArgs& a, Launch launch) { launch(a.descs, a.order, a.n_gemv); }

// wave-uniform loads from constant memory (scalar loads)
template <typename T>
using const_ptr = const T __attribute__((address_space(4)))*;

// The descriptor of this workgroup's GEMV, as a value, and the workgroup's index in it: from the numbering, or from the
// 2-D grid.  The descriptor is fetched whole by scalar loads: one memory round trip instead of one per group of fields.
// (Requesting all descriptors of a numbered launch along with the entry that says which one it is, three to a register by
// vector loads, and picking one out of the lanes cost 0.25 us more than the second round trip.)
template <typename Args>
__device__ __forceinline__ GemvDesc desc_of_workgroup(const Args& a, int& wg_local) {
    if constexpr (__is_same(Args, KernelArgs<true>)) {
        wg_local = (int)blockIdx.x;
        return a.single;
    } else {
        int g = (int)blockIdx.y;
        wg_local = (int)blockIdx.x;
        if constexpr (__is_same(Args, OrderedArgs)) {
            // entries in pairs, one scalar load (the numbering has room for an even number)
            const uint32_t pair = reinterpret_cast<const_ptr<uint32_t>>(reinterpret_cast<uintptr_t>(a.order))[blockIdx.x >> 1];
            const uint32_t e = (blockIdx.x & 1) ? pair >> 16 : pair & 0xffffu;
            g = (int)(e >> 13);
            wg_local = (int)(e & 0x1fffu);
        }
        typedef uint32_t u32x16 __attribute__((ext_vector_type(16), aligned(16)));  // (a table is, and its entries of 80 bytes)
        struct alignas(8) Words {
            uint32_t w[20];
        } raw;
        static_assert(sizeof(GemvDesc) == sizeof(Words) && sizeof(GemvDesc) % 16 == 0, "descriptor size");
        const uintptr_t p = reinterpret_cast<uintptr_t>(a.descs + g);
        const u32x16 lo = *reinterpret_cast<const_ptr<u32x16>>(p);
        const u32x4 hi = *reinterpret_cast<const_ptr<u32x4>>(p + 64);
#pragma unroll
        for (int i = 0; i < 16; ++i) raw.w[i] = lo[i];
#pragma unroll
        for (int i = 0; i < 4; ++i) raw.w[16 + i] = hi[i];
        return __builtin_bit_cast(GemvDesc, raw);
    }
}

// Output of one row block by its first wave: y holds the sums of the workgroup's K segment for the lane's
// row; `step` is a factor per token applied to the final sum (1, or the power-of-two step of integer tables).  With one segment they are the result; otherwise the segments meet through memory (see above).
template <int NP>
__device__ __forceinline__ void finish_rows(const GemvDesc& d, int rb, int seg, int n_seg, int lane, float (&y)[NP],
                                            const float (&step)[NP]) {
    const int m = rb * kRows + lane;
    const int M = d.M, N = d.N;
    _Float16* out = static_cast<_Float16*>(d.y);
    if (n_seg == 1) {
        if (m < M) {
#pragma unroll
            for (int n = 0; n < NP; ++n)
                if (n < N) out[(size_t)n * M + m] = (_Float16)(y[n] * step[n]);
        }
        return;
    }

    // K longer than one segment: publish this segment's partial sums and take a ticket
    float* base_p = d.partial + (size_t)rb * n_seg * NP * kRows;
    float* mine = base_p + (size_t)seg * NP * kRows;
#pragma unroll
    for (int n = 0; n < NP; ++n)
        __hip_atomic_store(mine + n * kRows + lane, y[n], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // the partials have reached device-coherent memory
    int32_t* ticket = d.tickets + rb;
    int prev = 0;
    if (lane == 0) prev = __hip_atomic_fetch_add(ticket, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    prev = __builtin_amdgcn_readfirstlane(prev);
    if (prev != n_seg - 1) return;
    // last ticket: every segment of this row block has been published; add them in segment order
    float acc[NP];
#pragma unroll
    for (int n = 0; n < NP; ++n) acc[n] = 0.f;
    for (int p0 = 0; p0 < n_seg; p0 += 4) {
        float v[4][NP];
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int n = 0; n < NP; ++n)
                v[q][n] = (p0 + q < n_seg) ? __hip_atomic_load(base_p + ((size_t)(p0 + q) * NP + n) * kRows + lane,
                                                               __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)
                                           : 0.f;
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int n = 0; n < NP; ++n) acc[n] += v[q][n];
    }
    if (m < M) {
#pragma unroll
        for (int n = 0; n < NP; ++n)
            if (n < N) out[(size_t)n * M + m] = (_Float16)(acc[n] * step[n]);
    }
    if (lane == 0) __hip_atomic_store(ticket, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

}  // namespace tman
