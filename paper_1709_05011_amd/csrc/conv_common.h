// What the implicit-GEMM kernels of conv_igemm.hip, conv_split.hip and conv_dma.hip share: tile numbering, guarded loads, buffer descriptors, division by
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
constexpr int kNonTemporal = 2;                       // policy operand of the buffer instructions: the nt bit
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

inline SkPlan sk_plan(long long tiles, int nkt, int resident_blocks, bool allow_split = true) {
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
    long long blocks = pl.sk_iters / 8;                      // at least 8 k-steps per stream-K block
    if (blocks > resident_blocks) blocks = resident_blocks;
    if (blocks < 1) blocks = 1;
    pl.sk_blocks = (int)blocks;
    return pl;
}

// The same with the number of blocks for the tiles beyond the whole rounds chosen by what they cost.  Candidates: every such tile to S blocks in
// equal parts -- S = 1 needs no fix-up at all -- or the k-steps end to end over the resident blocks.  For fp32 backward-data (conv_split.hip) and what bf16 leaves the main
// kernel; conv_dma.hip has a model of its own.  In us, fitted to layers of 1 to 512 images on a chip that does nothing else (beside a second stream `alone` is too short; whole training steps with
// their filter gradients on one are 2 to 18 % faster than with the plain form all the same): a k-step takes `alone` where a block has its compute unit
// to itself, `shared` per block where blocks take turns, see the callers; tiles that several blocks share cost 5 for the fix-up launch and
// 0.018 per 128x128 part written and read again.  Before, every problem took
// the last form with 8 k-steps per block or more, which splits tiles that the idle chip could take whole and joins tiles while compute units
// stand idle (fp32 backward-data, 3x3 over 128 channels, 32 images of 28x28 87 -> 60 us).
struct StepCost {
    double alone, shared, tile;      // us, us, what a part costs in parts of 128x128
    int min_steps;                   // k-steps a block takes of a shared tile at least
};
inline SkPlan sk_plan_by_cost(long long tiles, int nkt, int resident_blocks, const StepCost& k) {
    SkPlan pl = sk_plan(tiles, nkt, resident_blocks);
    if (pl.sk_blocks == 0) return pl;
    const long long rest = tiles - pl.dp_tiles, cus = device_cu_count();
    auto cost = [&](long long blocks, long long steps, bool split) {
        const double one = (double)steps * k.alone, many = (double)((blocks + cus - 1) / cus) * (double)steps * k.shared;
        return (one > many ? one : many) + (split ? 5.0 + 0.018 * k.tile * (double)blocks : 0.0);
    };
    long long even = pl.sk_iters / k.min_steps;
    if (even > resident_blocks) even = resident_blocks;
    if (even < 1) even = 1;
    pl.sk_blocks = (int)even;
    double best = cost(even, (pl.sk_iters + even - 1) / even, pl.sk_iters != even * nkt);
    for (int s = 1; rest * s <= resident_blocks && (s == 1 || nkt >= k.min_steps * s); ++s) {
        const double c = cost(rest * s, (nkt + s - 1) / s, s > 1);
        if (c < best) {
            best = c;
            pl.sk_blocks = (int)(rest * s);
        }
    }
    return pl;
}

// First k-step of stream-K block j (j <= sk_blocks), in 32-bit arithmetic: a 64-bit division is some hundred instructions, and every block of
// the product and of its fix-up starts with several.
__device__ __forceinline__ int sk_begin(const GemmConv& p, int j) { return j * p.sk_q + div_by(j * p.sk_rem, p.sk_mul, p.sk_shift); }
// The stream-K blocks [*j0, *j1) with a part of the k-steps [tb, te).
__device__ __forceinline__ void sk_blocks_of(const GemmConv& p, int tb, int te, int* j0, int* j1) {
    int a = min(p.sk_blocks - 1, (int)((float)tb * p.sk_per_step)), b = min(p.sk_blocks, (int)((float)te * p.sk_per_step));      // within one of them
    while (a > 0 && sk_begin(p, a) > tb) --a;
    while (sk_begin(p, a + 1) <= tb) ++a;
    while (b > 0 && sk_begin(p, b - 1) >= te) --b;
    while (b < p.sk_blocks && sk_begin(p, b) < te) ++b;
    *j0 = a;
    *j1 = b;
}

// The shared tile that row x of a fix-up's grid adds up: the tile (counted from the first stream-K tile) and the blocks
// [*j0, *j1) with parts of it; false: the tile that row x stands for was stored whole.  Ranges of a tile's k-steps and more meet in at most one point
// inside a tile: a row per meeting point (MEET).  Shorter ones share nearly every tile: a row per tile.  (1x1 over 32 channels, two k-steps per tile, 17 images
// of 44x44 in fp32: a row per tile and its search for the blocks made 8,352 blocks of which most had nothing to do, 19 us; this way 4.)
template <bool MEET>
__device__ __forceinline__ bool sk_shared_tile(const GemmConv& p, int nkt, int x, int* tile, int* j0, int* j1) {
    if constexpr (MEET) {
        const int b = sk_begin(p, x + 1);
        *tile = b / nkt;
        *j0 = x;
        *j1 = x + 2;
        return b != *tile * nkt;
    } else {
        *tile = x;
        sk_blocks_of(p, x * nkt, x * nkt + nkt, j0, j1);
        return *j1 - *j0 > 1;
    }
}
inline bool sk_ranges_meet(const GemmConv& p, int nkt) { return p.sk_q >= nkt; }
// The segments of one block of a persistent product kernel: its whole tiles, one per round, then its stream-K range cut at the tile boundaries.
struct SkWalk {
    int G, bid, nkt, dp_tiles, rounds, it, len, tile0, k00;
    __device__ __forceinline__ SkWalk(const GemmConv& p, int k_steps) : G(gridDim.x), bid(blockIdx.x), nkt(k_steps), dp_tiles(p.dp_tiles) {
        rounds = dp_tiles / G;                             // the launcher makes dp_tiles a multiple of the grid
        it = len = 0;
        if (bid < p.sk_blocks) {
            it = sk_begin(p, bid);
            len = sk_begin(p, bid + 1) - it;
        }
        tile0 = it / nkt;
        k00 = it - tile0 * nkt;
    }
    __device__ __forceinline__ int steps() const { return rounds * nkt + len; }      // k-steps this block runs
    __device__ __forceinline__ void segment(int s, int& tile, int& k0, int& k1) const {
        if (s < rounds) {
            tile = xcd_tile(s * G + bid, dp_tiles);
            k0 = 0;
            k1 = nkt;
        } else {                                           // piece s - rounds of the stream-K range
            const int t = tile0 + (s - rounds);
            tile = dp_tiles + t;
            k0 = s == rounds ? k00 : 0;
            k1 = min(nkt, it + len - t * nkt);
        }
    }
};

// The taps of an R x S window (at most 32) as bits r * S + s, and which of them lie outside an H x W image for a window whose first tap is at
// (h0, w0): all bits set where none lies inside.
struct WindowTaps {
    unsigned full, rep;                                    // every tap; bit r * S of every r, which spreads a mask over s to all rows
    __device__ __forceinline__ WindowTaps(int R, int S) {
        full = R * S >= 32 ? ~0u : (1u << (R * S)) - 1u;
        rep = 0;
        for (int r = 0; r < R; ++r) rep |= 1u << (r * S);
    }
    __device__ __forceinline__ unsigned outside(int h0, int w0, int H, int W, int R, int S) const {
        int rlo = max(0, -h0), rhi = min(R - 1, H - 1 - h0);      // rows and columns of the window inside the image
        int slo = max(0, -w0), shi = min(S - 1, W - 1 - w0);
        const bool some = (rlo <= rhi) & (slo <= shi);
        rlo = min(rlo, R - 1);                                    // keep the shifts in range when no tap is inside
        rhi = max(rhi, 0);
        slo = min(slo, S - 1);
        const unsigned rows = (full << (rlo * S)) & (full >> ((R - 1 - rhi) * S));
        const unsigned cols = rep * (((2u << max(shi - slo, 0)) - 1u) << slo);
        return some ? ~(rows & cols) : ~0u;
    }
};

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

// The launcher's part of sk_begin(); sk_blocks and sk_iters are set.
inline void sk_constants(GemmConv* p) {
    p->sk_q = p->sk_blocks > 0 ? (int)(p->sk_iters / p->sk_blocks) : 0;
    p->sk_rem = p->sk_blocks > 0 ? (int)(p->sk_iters % p->sk_blocks) : 0;
    magic_for(p->sk_blocks, &p->sk_mul, &p->sk_shift);
    p->sk_per_step = p->sk_iters > 0 ? (float)p->sk_blocks / (float)p->sk_iters : 0.f;
}

}  // namespace
