// What the implicit-GEMM kernels of conv_igemm.hip and conv_split.hip share: tile numbering, guarded loads, buffer descriptors, division by
// host constants, and the host-side work split.  Everything is local to the including file.
#pragma once

#include <stdlib.h>

#include "internal.h"

namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
constexpr unsigned kBufferWords3 = 0x00020000u;       // raw buffer, 32-bit data format
constexpr unsigned kBufferBytes = 0x80000000u;        // buffer size given to the hardware; offsets with bit 31 set read zeros


// Blocks are dealt round-robin to the 8 XCDs, each with its own L2.  Re-number them so that every
// XCD works on one contiguous run of tiles (neighbouring tiles share A rows and the whole filter).
__device__ __forceinline__ int xcd_tile(int bid, int total) {
    const int per = (total + 7) >> 3, rem = total & 7;
    const int xcd = bid & 7, idx = bid >> 3;
    if (rem == 0 || xcd < rem) return xcd * per + idx;
    return rem * per + (xcd - rem) * (per - 1) + idx;
}

__device__ __attribute__((aligned(16))) const float g_zero_chunk[4] = {0.f, 0.f, 0.f, 0.f};


// ok ? a : b on pointers by bit masking: never a branch, whatever the cost of computing a
__device__ __forceinline__ const void* pick(bool ok, const void* a, const void* b) {
    const uintptr_t m = (uintptr_t)0 - (uintptr_t)ok;
    return reinterpret_cast<const void*>((reinterpret_cast<uintptr_t>(a) & m) | (reinterpret_cast<uintptr_t>(b) & ~m));
}
// 16-byte load through the global (not flat) path: a flat load would also count as an LDS operation
__device__ __forceinline__ float4 load_global16(const void* ptr) {
    typedef float gf4 __attribute__((ext_vector_type(4)));
    const gf4 v = *(const __attribute__((address_space(1))) gf4*)(uintptr_t)ptr;
    return make_float4(v.x, v.y, v.z, v.w);
}
// This wave's LDS writes and reads are complete, then the workgroup barrier.  Global loads stay in flight
// (__syncthreads() would wait for them too).
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" : : : "memory"); }

__device__ __forceinline__ int div_by(int n, unsigned mul, unsigned shift) {       // n / d for 0 <= n < 2^31, see magic_for()
    return mul ? (int)(__umulhi((unsigned)n, mul) >> shift) : n;
}

__host__ __device__ inline bool aligned16(const void* ptr) { return (reinterpret_cast<uintptr_t>(ptr) & 15) == 0; }

// Split of the output tiles into whole-tile blocks and stream-K blocks for a BM x BN tiling.
struct SkPlan {
    int dp_tiles, sk_blocks;
    long long sk_iters;
};

inline int device_cu_count() {
    static const int n = [] {
        int dev = 0, cus = 0;
        if (hipGetDevice(&dev) != hipSuccess || hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
            cus <= 0)
            cus = 256;
        (void)hipGetLastError();
        return cus;
    }();
    return n;
}

// min_steps: k-steps a stream-K block takes at least
inline SkPlan sk_plan(long long tiles, int nkt, int resident_blocks, bool allow_split = true, int min_steps = 8) {
    SkPlan pl;
    const long long rounds = tiles / resident_blocks;
    long long dp = rounds * resident_blocks;
    long long rest = tiles - dp;
    pl.dp_tiles = (int)dp;
    pl.sk_blocks = 0;
    pl.sk_iters = 0;
    if (rest == 0 || !allow_split || getenv("LARSCONV_NO_STREAMK")) {   // every round is full, or splitting tiles is not wanted
        pl.dp_tiles = (int)tiles;
        return pl;
    }
    pl.sk_iters = rest * nkt;
    long long blocks = pl.sk_iters / min_steps;
    if (blocks > resident_blocks) blocks = resident_blocks;
    if (blocks < 1) blocks = 1;
    pl.sk_blocks = (int)blocks;
    return pl;
}

// Constants for div_by(): n / d == umulhi(n, mul) >> shift for 0 <= n < 2^31 (mul == 0 stands for d == 1).
// With L = ceil(log2 d) and mul = ceil(2^(31+L) / d) the error term n * (mul*d - 2^(31+L)) stays below 2^(31+L).
inline void magic_for(int d, unsigned* mul, unsigned* shift) {
    if (d <= 1) {
        *mul = 0;
        *shift = 0;
        return;
    }
    int L = 0;
    while ((1ll << L) < d) ++L;
    *mul = (unsigned)((((unsigned long long)1 << (31 + L)) + (unsigned)d - 1) / (unsigned)d);
    *shift = (unsigned)(L - 1);
}

}  // namespace
