// bf16 products of gfx950 whose operands go from memory straight into LDS (buffer loads with the lds modifier): no staging registers, no LDS store
// instructions, and several k-steps in flight per compute unit.
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <algorithm>
#include <cmath>
#include <type_traits>

#include "conv_common.h"

namespace {

typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef short s16x8 __attribute__((ext_vector_type(8)));

// 64 lanes x 16 bytes from base + voff + soff to LDS bytes lds .. lds + 1023 in lane order; lanes past the declared size of the buffer fetch zeros.
// (Inline assembly: behind the builtin the compiler waits for all of a wave's loads before each LDS read that might meet them.  No register is
// written, so nothing can be reused too early; whoever reads the bytes waits with wait_loads() and a barrier first.)
__device__ __forceinline__ void load_to_lds(const u32x4& rsrc, unsigned voff, int soff, unsigned lds) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds" : : "s"(lds), "v"(voff), "s"(rsrc), "s"(soff) : "memory");
}
__device__ __forceinline__ void load_to_lds_nt(const u32x4& rsrc, unsigned voff, int soff, unsigned lds) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen nt lds" : : "s"(lds), "v"(voff), "s"(rsrc), "s"(soff) : "memory");
}
__device__ __forceinline__ u32x4 buffer_words(const void* base, unsigned bytes) {
    const uintptr_t a = reinterpret_cast<uintptr_t>(base);
    return u32x4{(unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)a), (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)(a >> 32)),
                 (unsigned)__builtin_amdgcn_readfirstlane((int)bytes), kBufferWords3};
}
// At most N of this wave's loads are still under way (they arrive in order), its LDS reads are complete; then the workgroup barrier.
template <int N>
__device__ __forceinline__ void wait_loads_and_barrier() {
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" : : "n"(N) : "memory");
}
__device__ __forceinline__ unsigned lds_address(const void* ptr) {
    return (unsigned)(uintptr_t)(const __attribute__((address_space(3))) unsigned char*)(uintptr_t)ptr;
}

// ------------------------------------------------------------------------------------------------
// Forward and backward-data.  A k-step is 64 values of the reduction: 128 bytes of a row, so that a load of 64 lanes covers eight whole lines.  LDS holds a
// stage as [row][128 bytes] with the 16-byte pieces of a row at piece ^ (row / 2 % 8) -- the lanes fetch them in that order -- and a fragment of sixteen rows then
// meets every bank once.  Two stages; while one is multiplied the other arrives, across tile boundaries (persistent blocks, segments as in SkWalk).
//
// A wave owns 16 TM x 16 TN of the tile in 16x16 pieces, the filter being the matrix instruction's first operand: a lane holds four neighbouring columns of a
// pixel.  TMA and TMB: rows of pieces of the first and the second row of waves; each SIMD runs one wave of either kind, so a tile may have any
// multiple of 16 rows.
//
// Bound: windows of many columns by power (3x3 over 256 channels, 512 images of 14x14: 98 to 106 us by the card's temperature, 1,110 to 1,200 TFLOP/s where a large
// product reaches 1,377; the pipe is busy in 57 % of the cycles at 1.87 to 1.97 GHz), 1x1 layers of few or of 256 and more columns on large images by memory (512 to 128 at 28x28
// 131 -> 108 us, 4.8 TB/s; 64 to 256 at 56x56 225 -> 197, 5.2).  The 1x1 layers between (128 to 512, 256 to 1024) by neither: 3.0 to 3.5 TB/s and 30 to 40 % of the pipe.
//  With staging registers and k-steps of 32, half
// a line of a row per load, the same layers took 147, 131 and 225.  Measured and left out: the loads spread over the following step, wave priorities around
// the matrix instructions (both equal or slower).
//
// kChunks: the channels are a multiple of 64, a k-step is 64 channels of one tap of the window and its place is scalar.  (The taps run fastest: the rows of a tile are read
// again soon.)  kPadded: the same with the last 64 channels filled up with zeros.  kPieces: the reduction as it lies in the filter, a lane's piece of it has a tap
// of its own.  Which taps of a row's window lie outside the image is a 32-bit mask.  Windows of more than 32 taps, and images so large that two of them span 2 GiB: kRuns is kPadded in
// runs of at most 32 taps (whole rows of the window, or parts of one that is wider), the masks set up anew for each; kTaps is kPieces with a piece's row and column compared with the
// image's size, two 16-bit numbers at a time; both count a tile's offsets from its first row, the others from its first image.  us, staging registers with half lines / here, forward, then backward-data: 7x7 over 256 channels, 256 images of 28x28 1462 / 1091 and 1464 / 1100; 11x11 96
// to 128, 64 of 28x28 203 / 146 and 246 / 203; 13x13 with stride 2 64 to 128, 32 of 56x56 113 / 79 and 210 / 180; 7x7 24 to 40, 64 of 56x56 57 / 49 and 83 / 84.
// ------------------------------------------------------------------------------------------------
struct ConvDma {
    GemmConv g;
    int nkt;                      // k-steps of a tile
    unsigned ci_mul, ci_shift, s_mul, s_shift;
    int run_rows;                 // kRuns: rows of a window in a run; 0: parts of a row
};

constexpr unsigned kNoRow = 0x80000000u;                   // row -2^15: outside under every tap's row (below 2^15)

// What leaves with a tile: whole 16-byte pieces of rows (columns a multiple of 8); any number of columns and the statistics; any number of columns; the pixels
// of a stride grid.
enum ConvDmaOut { kRows, kStats, kAny, kGrid };
enum ConvDmaIn { kChunks, kPadded, kPieces, kRuns, kTaps, kOnce };

template <int TMA, int TMB, int TN, int WN, ConvDmaIn IN, ConvDmaOut OUT>
__global__ void __launch_bounds__(2 * WN * 64, 2) conv_dma_kernel(const ConvDma pp) {
    const GemmConv& p = pp.g;
    constexpr int BM = 16 * (TMA + TMB), BN = 16 * TN * WN, NW = 2 * WN;
    constexpr int NA = BM / 8, NB = BN / 8;                // loads of a stage
    constexpr int LA = (NA + NW - 1) / NW, LB = NB / NW;
    constexpr int STAGE = (BM + BN) * 128;
    constexpr int kOutPitch = TN * 32 + 16;                // bytes
    static_assert(NB % NW == 0, "tile shape");
    extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
    unsigned char* const bounce = smem + 2 * STAGE;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave / WN, wn = wave % WN;
    const int nbn = (p.N + BN - 1) / BN;
    const int nkt = pp.nkt;
    const uint16_t* const A = static_cast<const uint16_t*>(p.a);
    const uint16_t* const B = static_cast<const uint16_t*>(p.b);
    const int Hi_ = p.Hi, Wi_ = p.Wi, Ci_ = p.Ci, R_ = p.R, S_ = p.S, M_ = p.M, N_ = p.N, Kg_ = p.Kg, ldd_ = p.ldd;
    const int sh_ = p.sh, sw_ = p.sw, ph_ = p.ph, pw_ = p.pw, Po_ = p.Po, Qo_ = p.Qo;
    const unsigned qmul = p.qo_mul, qsh = p.qo_shift, pmul = p.po_mul, psh = p.po_shift;
    const int taps = R_ * S_;

    const SkWalk walk(p, nkt);
    const int F = walk.steps(), rounds = walk.rounds, bid = walk.bid;
    if (F == 0) return;

    // ---------------- load side ----------------
    int l_seg = -1, l_k = 0, l_k1 = 0;                     // segment being loaded, next k-step, end
    const int lrow = lane >> 3;
    const int piece = (lane & 7) ^ (((wave & 1) * 4 + (lrow >> 1)) & 7);     // row / 2 % 8 of every row this lane loads: 8 * (i * NW + wave) + lrow
    unsigned a_voff[LA], a_inv[LA];                        // kTaps: a_inv is the place of the window's first tap in the image, row in the upper half
    u32x4 a_rsrc = {0, 0, 0, 0}, b_rsrc = a_rsrc;
    constexpr bool by_tap = IN == kChunks || IN == kPadded || IN == kRuns || IN == kOnce;
    const unsigned b_voff = (unsigned)((wave * 8 + lrow) * Kg_ * 2 + piece * 16);
    int u_c = 0, u_tap = 0, u_r = 0, u_s = 0;              // first channel and tap; kPieces, kTaps: u_c is the k-step
    int u_first = 0, l_stop = 0;                           // kRuns: the run's first tap; the k-step behind the run or the segment
    const unsigned lds0 = lds_address(smem);
    unsigned l_lds = lds0;
    auto loader_setup = [&](int tile, int k0) __attribute__((always_inline)) {
        const int tm = tile / nbn;
        const int m0 = tm * BM, n0 = (tile - tm * nbn) * BN;
        const int img0 = div_by(div_by(m0, qmul, qsh), pmul, psh);
        const int phb = max(ph_, 0), pwb = max(pw_, 0);
        int row_base = 0;                                  // the row of the first image that offsets count from: within it, so that the next image's rows lie behind
        if constexpr (IN == kRuns || IN == kTaps) {
            const int t0 = div_by(m0, qmul, qsh);
            row_base = min((t0 - img0 * Po_) * sh_, Hi_);
        }
        auto place = [&]() __attribute__((always_inline)) {
            if constexpr (by_tap) {
                const int chunk = k0 / taps;
                u_tap = k0 - chunk * taps;
                u_c = chunk * 64;
                u_r = u_tap / S_;
                u_s = u_tap - u_r * S_;
            } else {
                u_c = k0;
            }
        };
        int run_r = 0, run_s = 0, rows = R_, cols = S_;    // the part of the window that the masks are for
        if constexpr (IN == kRuns) {
            place();
            if (pp.run_rows > 0) {
                run_r = u_r / pp.run_rows * pp.run_rows;
                rows = min(pp.run_rows, R_ - run_r);
            } else {
                run_r = u_r;
                run_s = u_s & ~31;
                rows = 1;
                cols = min(32, S_ - run_s);
            }
            u_first = run_r * S_ + run_s;
            l_stop = min(l_k1, k0 + (u_first + rows * cols - u_tap));
        }
        const int run_h = ph_ - run_r, run_w = pw_ - run_s, first_h = phb - run_r - row_base, first_w = pwb - run_s;
        const WindowTaps window(IN != kTaps ? rows : 1, IN != kTaps ? cols : 1);
#pragma unroll
        for (int i = 0; i < LA; ++i) {
            const int row = (i * NW + wave) * 8 + lrow, m = m0 + row;
            const int t = div_by(m, qmul, qsh), qo = m - t * Qo_;
            const int img = div_by(t, pmul, psh), po = t - img * Po_;
            const int h0 = po * sh_ - run_h, w0 = qo * sw_ - run_w;      // the run's first row and column in the image
            bool ok;
            if constexpr (IN == kTaps) {
                ok = (m < M_) & (h0 < Hi_) & (h0 + R_ > 0) & (w0 < Wi_) & (w0 + S_ > 0);
                a_inv[i] = ok ? (unsigned)h0 << 16 | ((unsigned)w0 & 0xffffu) : kNoRow;
            } else {
                const unsigned inv = window.outside(h0, w0, Hi_, Wi_, rows, cols);
                ok = (m < M_) & (inv != ~0u);
                a_inv[i] = ok ? inv : ~0u;
            }
            a_voff[i] = ok ? (unsigned)(((((img - img0) * Hi_ + h0 + first_h) * Wi_) + w0 + first_w) * Ci_ * 2 + (by_tap ? piece * 16 : 0)) : 0u;
        }
        const long long a_first = (((long long)img0 * Hi_ + row_base) * Wi_ - ((long long)phb * Wi_ + pwb)) * Ci_;
        a_rsrc = buffer_words(A + a_first, kBufferBytes);
        const long long b_left = (long long)(N_ - n0) * Kg_ * 2;       // rows past N lie past the end of the buffer
        b_rsrc = buffer_words(B + (long long)n0 * Kg_, b_left > 0x7fffffffLL ? 0x7fffffffu : (unsigned)b_left);
        if constexpr (IN != kRuns) place();
    };
    // the next k-step of the block's sequence (past its end: nothing)
    unsigned v_off = 0, v_up = 0, v_bad = 0;               // this lane's piece: byte offset from the window's first value, tap; bit 31: no such channel
    typedef short s16x2 __attribute__((ext_vector_type(2)));
    s16x2 v_rs = {0, 0};                                   // kTaps: the tap's column and row
    const s16x2 last = {(short)(Wi_ - 1), (short)(Hi_ - 1)};
    int l_tile = 0;
    auto load_begin = [&]() __attribute__((always_inline)) {
        if constexpr (IN == kRuns) {
            if (l_k == l_stop) {
                if (l_k == l_k1) walk.segment(++l_seg, l_tile, l_k, l_k1);
                loader_setup(l_tile, l_k);
            }
        } else if (l_k == l_k1) {
            int tile;
            ++l_seg;
            walk.segment(l_seg, tile, l_k, l_k1);
            loader_setup(tile, l_k);
        }
        if constexpr (IN == kPadded || IN == kRuns) v_bad = u_c + piece * 8 < Ci_ ? 0u : kBufferBytes;
        if constexpr (!by_tap) {
            const int kg = u_c * 64 + piece * 8;
            const int rs = div_by(kg, pp.ci_mul, pp.ci_shift), c = kg - rs * Ci_;
            const int r = div_by(rs, pp.s_mul, pp.s_shift), s = rs - r * S_;
            v_off = (unsigned)(((r * Wi_ + s) * Ci_ + c) * 2);
            v_bad = kg < Kg_ ? 0u : kBufferBytes;
            v_up = (unsigned)max(31 - rs, 0);
            v_rs = s16x2{(short)s, (short)r};
        }
    };
    auto load_one = [&](int l) __attribute__((always_inline)) {
        if (l < LA) {
            const int load = l * NW + wave;
            if (NA % NW != 0 && load >= NA) return;
            if constexpr (by_tap) {
                const unsigned vo = (((a_inv[l] << (31 - (u_tap - u_first))) & kBufferBytes) | a_voff[l]) | v_bad;
                if constexpr (IN == kOnce) load_to_lds_nt(a_rsrc, vo, ((u_r * Wi_ + u_s) * Ci_ + u_c) * 2, l_lds + load * 1024);
                else load_to_lds(a_rsrc, vo, ((u_r * Wi_ + u_s) * Ci_ + u_c) * 2, l_lds + load * 1024);
            } else if constexpr (IN == kTaps) {            // a sign bit of the place, or of what is left to the last row and column: outside
                const s16x2 at = __builtin_bit_cast(s16x2, a_inv[l]) + v_rs;
                const unsigned out = __builtin_bit_cast(unsigned, at) | __builtin_bit_cast(unsigned, last - at);
                load_to_lds(a_rsrc, ((out << 16 | out) & kBufferBytes) | v_bad | (a_voff[l] + v_off), 0, l_lds + load * 1024);
            } else {
                load_to_lds(a_rsrc, ((a_inv[l] << v_up) & kBufferBytes) | v_bad | (a_voff[l] + v_off), 0, l_lds + load * 1024);
            }
        } else {
            const int load = (l - LA) * NW + wave;
            const int rows = (l - LA) * NW * 8 * Kg_ * 2;
            load_to_lds(b_rsrc, b_voff | v_bad, rows + (by_tap ? (u_tap * Ci_ + u_c) * 2 : u_c * 128), l_lds + BM * 128 + load * 1024);
        }
    };
    auto load_end = [&]() __attribute__((always_inline)) {
        if constexpr (by_tap) {
            ++u_tap;
            ++u_s;
            const bool row = u_s == S_;
            u_s = row ? 0 : u_s;
            u_r += row ? 1 : 0;
            const bool chunk = u_tap == taps;
            u_tap = chunk ? 0 : u_tap;
            u_r = chunk ? 0 : u_r;
            u_c += chunk ? 64 : 0;
        } else {
            ++u_c;
        }
        ++l_k;
        l_lds = l_lds == lds0 ? lds0 + STAGE : lds0;
    };

    // ---------------- compute side ----------------
    auto run = [&]<int TM>(std::integral_constant<int, TM>) __attribute__((always_inline)) {
        const int row0 = wm * TMA * 16;                    // this wave's first row of the tile
        f32x4 acc[TM][TN];
        bf16x8 fa[4], fb[2][TN];
        // fragment: row lane % 16, pieces lane / 16 (first half of the k-step) and 4 + lane / 16
        const int sw = ((lane & 15) >> 1), fp = lane >> 4;
        const unsigned char* const a_lane = smem + (row0 + (lane & 15)) * 128;
        const unsigned char* const b_lane = smem + BM * 128 + (wn * TN * 16 + (lane & 15)) * 128;
        const int half0 = ((fp ^ sw) & 7) * 16, half1 = (((4 + fp) ^ sw) & 7) * 16;
        auto read_a = [&](int stage, int h, int i, int slot) __attribute__((always_inline)) {
            fa[slot] = *reinterpret_cast<const bf16x8*>(a_lane + stage + (h ? half1 : half0) + i * 2048);
        };
        auto read_b = [&](int stage, int h, int j) __attribute__((always_inline)) {
            fb[h][j] = *reinterpret_cast<const bf16x8*>(b_lane + stage + (h ? half1 : half0) + j * 2048);
        };
        auto clear_acc = [&]() __attribute__((always_inline)) {
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
        };
        int c_seg = 0, c_tile, c_k0, c_k, c_k1;
        walk.segment(0, c_tile, c_k0, c_k1);
        c_k = c_k0;
        unsigned char* const mine = bounce + wave * (16 * kOutPitch);
        const bool whole_rows = OUT == kRows || ((N_ | ldd_) & 7) == 0;
        auto epilogue = [&]() __attribute__((always_inline)) {
            const int tm = c_tile / nbn;
            const int m0 = tm * BM, n0 = (c_tile - tm * nbn) * BN;
            if (!(c_k0 == 0 && c_k1 == nkt)) {
                // part of a tile: the first piece of this block's stream-K range (slot 2 * bid) or the last (2 * bid + 1)
                const __amdgpu_buffer_rsrc_t part_rsrc = __builtin_amdgcn_make_buffer_rsrc(
                    (void*)(p.partial + ((size_t)2 * bid + (c_seg == rounds ? 0 : 1)) * (BM * BN)), 0, BM * BN * 4, (int)kBufferWords3);
#pragma unroll
                for (int i = 0; i < TM; ++i)
#pragma unroll
                    for (int j = 0; j < TN; ++j)
                        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, acc[i][j]), part_rsrc, lane * 16 + wave * 1024,
                                                               (i * TN + j) * NW * 1024, 0);
                return;
            }
            // 16 rows at a time through the wave's own LDS, so that a store covers whole rows of the wave's part.  Rows past M lie past the end of the buffer
            // or have bit 31 of the offset set, columns past N the latter.
            constexpr int CPR = TN * 2, RPI = 64 / CPR;    // lanes per row, rows per store
            const int mw = m0 + row0, lr = lane / CPR, col = n0 + wn * TN * 16 + lane % CPR * 8;
            constexpr bool scatter = OUT == kGrid;
            long long first_px = mw;
            if (scatter) {
                const int t0 = div_by(mw, qmul, qsh), i0 = div_by(t0, pmul, psh);
                first_px = ((long long)i0 * p.Ho + (t0 - i0 * Po_) * p.esh) * p.Wo + (mw - t0 * Qo_) * p.esw;
            }
            const long long left = scatter ? 0x7fffffffLL : (long long)(M_ - mw) * ldd_ * 2;
            const __amdgpu_buffer_rsrc_t d_rsrc = __builtin_amdgcn_make_buffer_rsrc(
                (void*)(static_cast<uint16_t*>(p.d) + first_px * ldd_), 0, (int)(left > 0x7fffffffLL ? 0x7fffffffLL : left > 0 ? left : 0), (int)kBufferWords3);
            const unsigned d_voff = col < N_ ? (unsigned)(lr * ldd_ + col) * 2u : kBufferBytes;
            auto row_off = [&](int m) __attribute__((always_inline)) {       // byte offset of a row of the result; bit 31 past M
                int px = m - mw;
                if (scatter) {
                    const int t = div_by(m, qmul, qsh), img = div_by(t, pmul, psh);
                    px = (int)(((long long)img * p.Ho + (t - img * Po_) * p.esh) * p.Wo + (m - t * Qo_) * p.esw - first_px);
                }
                return m < M_ ? (unsigned)(px * ldd_) * 2u : kBufferBytes;
            };
            // Statistics on the matrix pipe: the stored values come back through the transposing read as [column][row], 32 rows at a time; multiplied by ones they give
            // the column sums in every row of a piece, multiplied by themselves the sums of squares on its diagonal.  (Summed lane by lane and then over sixteen lanes they were 350
            // vector instructions a tile, more than the products of a short reduction: 1x1 32 to 96, 254 images of 46x46 44 -> 36 us; over 450 layers 0.96.)
            constexpr bool stats = OUT == kStats;
            static_assert(!stats || TM % 2 == 0, "rows of pieces in pairs");
            f32x4 sum[TN], sq[TN];
            s16x4 even[TN];
            if constexpr (stats) {
#pragma unroll
                for (int j = 0; j < TN; ++j) sum[j] = sq[j] = f32x4{0.f, 0.f, 0.f, 0.f};
            }
#pragma unroll
            for (int i = 0; i < TM; ++i) {
#pragma unroll
                for (int j = 0; j < TN; ++j) {
                    const uint2 u = make_uint2(lc_bf16x2_rne(acc[i][j][0], acc[i][j][1]), lc_bf16x2_rne(acc[i][j][2], acc[i][j][3]));
                    *reinterpret_cast<uint2*>(mine + (lane & 15) * kOutPitch + j * 32 + (lane >> 4) * 8) = u;
                }
                asm volatile("s_waitcnt lgkmcnt(0)" : : : "memory");
                if constexpr (stats) {                     // of the values as stored; rows past M are zeros
#pragma unroll
                    for (int j = 0; j < TN; ++j) {
                        const unsigned char* const q = mine + (lane >> 2) * kOutPitch + j * 32 + (lane & 3) * 8;
                        const s16x4 rows = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)(uintptr_t)q);
                        if (i % 2 == 0) {
                            even[j] = rows;
                        } else {
                            const bf16x8 v = __builtin_bit_cast(bf16x8, s16x8{even[j][0], even[j][1], even[j][2], even[j][3], rows[0], rows[1], rows[2], rows[3]});
                            const bf16x8 ones = __builtin_bit_cast(bf16x8, u32x4{0x3f803f80u, 0x3f803f80u, 0x3f803f80u, 0x3f803f80u});
                            sum[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ones, v, sum[j], 0, 0, 0);
                            sq[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(v, v, sq[j], 0, 0, 0);
                        }
                    }
                }
                if (whole_rows) {
                    u32x4 out[16 / RPI];
#pragma unroll
                    for (int e = 0; e < 16 / RPI; ++e) out[e] = *reinterpret_cast<const u32x4*>(mine + (e * RPI + lr) * kOutPitch + lane % CPR * 16);
                    asm volatile("s_waitcnt lgkmcnt(0)" : : : "memory");
#pragma unroll
                    for (int e = 0; e < 16 / RPI; ++e) {
                        if constexpr (!scatter) {
                            if (__builtin_expect(p.stream_d, 0)) __builtin_amdgcn_raw_buffer_store_b128(out[e], d_rsrc, (int)d_voff, (i * 16 + e * RPI) * ldd_ * 2, kNonTemporal);
                            else __builtin_amdgcn_raw_buffer_store_b128(out[e], d_rsrc, (int)d_voff, (i * 16 + e * RPI) * ldd_ * 2, 0);
                        } else {
                            const unsigned off = row_off(mw + i * 16 + e * RPI + lr);
                            if (__builtin_expect(p.stream_d, 0)) __builtin_amdgcn_raw_buffer_store_b128(out[e], d_rsrc, (int)(col < N_ ? off + (unsigned)col * 2u : kBufferBytes), 0, kNonTemporal);
                            else __builtin_amdgcn_raw_buffer_store_b128(out[e], d_rsrc, (int)(col < N_ ? off + (unsigned)col * 2u : kBufferBytes), 0, 0);
                        }
                    }
                } else {
                    // rows that start anywhere: neighbouring lanes store neighbouring columns, in pairs where there is an even number of them
                    // (a loop: unrolled, the two forms for every row of pieces are more code than the instruction cache holds)
                    auto store = [&](auto pair) __attribute__((always_inline)) {
                        constexpr int V = decltype(pair)::value, PER = TN * 16 / V, RWS = 64 / PER;      // columns per lane; lanes per row, rows per store
                        const int c = lane % PER * V, cc = n0 + wn * TN * 16 + c;
                        const unsigned char* q = mine + lane / PER * kOutPitch + c * 2;
                        const unsigned voff = cc < N_ ? (unsigned)(lane / PER * ldd_ + cc) * 2u : kBufferBytes;
                        int so = i * 16 * ldd_ * 2;
#pragma unroll 4
                        for (int e = 0; e < 16 / RWS; ++e) {
                            const unsigned v = V == 2 ? *reinterpret_cast<const unsigned*>(q) : *reinterpret_cast<const unsigned short*>(q);
                            int o = (int)voff, at = so;
                            if constexpr (OUT == kGrid) {
                                o = (int)(cc < N_ ? row_off(mw + i * 16 + e * RWS + lane / PER) + (unsigned)cc * 2u : kBufferBytes);
                                at = 0;
                            }
                            if constexpr (V == 2) __builtin_amdgcn_raw_buffer_store_b32(v, d_rsrc, o, at, 0);
                            else __builtin_amdgcn_raw_buffer_store_b16((short)v, d_rsrc, o, at, 0);
                            q += RWS * kOutPitch;
                            so += RWS * ldd_ * 2;
                        }
                    };
                    if (((N_ | ldd_) & 1) == 0) store(std::integral_constant<int, 2>{});
                    else store(std::integral_constant<int, 1>{});
                }
            }
            if constexpr (stats) {                         // lane 16 g + c holds rows 4 g .. 4 g + 3 of column c
                typedef float flt2 __attribute__((ext_vector_type(2)));
                flt2* const st = reinterpret_cast<flt2*>(p.stats) + ((size_t)tm * 2 + wm) * N_;
                const bool diagonal = (lane >> 4) == ((lane & 15) >> 2);
#pragma unroll
                for (int j = 0; j < TN; ++j) {
                    const float b = lane & 2 ? (lane & 1 ? sq[j][3] : sq[j][2]) : (lane & 1 ? sq[j][1] : sq[j][0]);
                    const int c = n0 + (wn * TN + j) * 16 + (lane & 15);
                    if (diagonal && c < N_) st[c] = flt2{sum[j][0], b};
                }
            }
        };

        load_begin();
#pragma unroll
        for (int l = 0; l < LA + LB; ++l) load_one(l);
        load_end();
        if (F > 1) {
            load_begin();
#pragma unroll
            for (int l = 0; l < LA + LB; ++l) load_one(l);
            load_end();
        }
        clear_acc();
        if (F > 1 && wave < NA - (LA - 1) * NW) wait_loads_and_barrier<LA + LB>();
        else if (F > 1) wait_loads_and_barrier<LA - 1 + LB>();
        else wait_loads_and_barrier<0>();
        read_a(0, 0, 0, 0);
        read_a(0, 0, 1, 1);
#pragma unroll
        for (int j = 0; j < TN; ++j) read_b(0, 0, j);
        bool stored = false;                               // the last step ended in stores that may still be under way
        auto step = [&]<int BUF>(std::integral_constant<int, BUF>, int f) __attribute__((always_inline)) {
            constexpr int stage = BUF * STAGE, other = STAGE - stage, OFF = (BUF * 2 * TM) & 3;
#pragma unroll
            for (int q = 0; q < 2 * TM; ++q) {
                const int h = q / TM;
                if (q + 2 < 2 * TM) {
                    read_a(stage, (q + 2) / TM, (q + 2) % TM, (q + 2 + OFF) & 3);
                    if (q < TN) read_b(stage, 1, q);
                } else if (q + 2 == 2 * TM) {
                    // this stage has been read, the next has arrived
                    if (stored) wait_loads_and_barrier<TM * 16 * TN * 32 / 1024>();
                    else wait_loads_and_barrier<0>();
                    stored = false;
                    read_a(other, 0, 0, (q + 2 + OFF) & 3);
#pragma unroll
                    for (int j = 0; j < TN; ++j) read_b(other, 0, j);
                } else {
                    read_a(other, 0, 1, (q + 2 + OFF) & 3);
                }
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int j = 0; j < TN; ++j)
                    acc[q % TM][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[h][j], fa[(q + OFF) & 3], acc[q % TM][j], 0, 0, 0);
                if (q + 2 >= 2 * TM && f + 2 < F) {        // k-step f + 2 into the stage just read
                    constexpr int half = (LA + LB + 1) / 2;
                    if (q + 2 == 2 * TM) load_begin();
#pragma unroll
                    for (int l = 0; l < LA + LB; ++l)
                        if ((l < half) == (q + 2 == 2 * TM)) load_one(l);
                    if (q + 1 == 2 * TM) load_end();
                }
                __builtin_amdgcn_sched_barrier(0);
            }
            if (++c_k == c_k1) {
                epilogue();
                stored = c_k0 == 0 && c_k1 == nkt && OUT != kStats && whole_rows;
                clear_acc();
                ++c_seg;
                walk.segment(c_seg, c_tile, c_k0, c_k1);
                c_k = c_k0;
            }
        };
        // (the last step reads fragments that are never used)
        for (int f = 0; f < F; f += 2) {
            step(std::integral_constant<int, 0>{}, f);
            if (f + 1 < F) step(std::integral_constant<int, 1>{}, f + 1);
        }
    };
    if constexpr (TMA == TMB) {
        run(std::integral_constant<int, TMA>{});
    } else {
        if (wm == 0) run(std::integral_constant<int, TMA>{});
        else run(std::integral_constant<int, TMB>{});
    }
}

// Adds the parts of every tile that stream-K blocks share, in k order, and stores the tile: block (t, y) takes piece y of each wave's part.
template <int TM, int TN, int WN>
__global__ void __launch_bounds__(2 * WN * 64) conv_dma_fixup_kernel(const GemmConv p, int nkt) {
    constexpr int BM = 32 * TM, BN = 16 * TN * WN, NW = 2 * WN;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int nbn = (p.N + BN - 1) / BN;
    int sk_tile, j, j1;
    if (!sk_shared_tile<false>(p, nkt, blockIdx.x, &sk_tile, &j, &j1)) return;  // one block did the whole tile and stored it
    const int tb = sk_tile * nkt;                                        // this tile's first k-step in stream-K positions
    const f32x4* part = reinterpret_cast<const f32x4*>(p.partial) + (blockIdx.y * NW + wave) * 64 + lane;
    constexpr size_t kSlot = BM * BN / 4;
    // the first block's piece is the last of its range unless its range starts here; all others start their ranges in this tile
    f32x4 sum = part[((size_t)2 * j + (sk_begin(p, j) >= tb ? 0 : 1)) * kSlot];
    for (++j; j + 4 <= j1; j += 4) {
        f32x4 v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) v[u] = part[(size_t)2 * (j + u) * kSlot];
#pragma unroll
        for (int u = 0; u < 4; ++u) sum += v[u];
    }
    for (; j < j1; ++j) sum += part[(size_t)2 * j * kSlot];
    const int tile = p.dp_tiles + sk_tile, tm = tile / nbn;
    const int ti = blockIdx.y / TN, tj = blockIdx.y - ti * TN;
    const int m = tm * BM + (wave / WN) * TM * 16 + ti * 16 + (lane & 15);
    const int col = (tile - tm * nbn) * BN + (wave % WN) * TN * 16 + tj * 16 + 4 * (lane >> 4);
    if (m >= p.M || col >= p.N) return;
    long long px = m;
    if (p.scatter) {
        const int qo = m % p.Qo, t = m / p.Qo;
        const int po = t % p.Po, img = t / p.Po;
        px = ((long long)img * p.Ho + (long long)po * p.esh) * p.Wo + (long long)qo * p.esw;
    }
    uint16_t* d = static_cast<uint16_t*>(p.d) + px * p.ldd + col;
    const uint2 u = make_uint2(lc_bf16x2_rne(sum[0], sum[1]), lc_bf16x2_rne(sum[2], sum[3]));
    if (((p.N | p.ldd) & 3) == 0 && (reinterpret_cast<uintptr_t>(p.d) & 7) == 0) {
        *reinterpret_cast<uint2*>(d) = u;
    } else {
#pragma unroll
        for (int v = 0; v < 4; ++v)
            if (col + v < p.N) d[v] = (uint16_t)((v < 2 ? u.x : u.y) >> (16 * (v & 1)));
    }
}

// Windows over channels that are nearly a multiple of 64: chunk by chunk all the same, also where that leaves up to a 32nd of the products to zeros.  With all
// channels of a tap before the next tap, a tile's rows come from beyond L2 once per tap (3x3, us, pieces / padded: 1120 to 64 253 / 175, 1272 to 96 212 / 161,
// 696 to 1984 439 / 417; but with a ninth of zeros 288 to 1048 380 / 407).
bool conv_dma_by_tap(const GemmConv& p) { return p.Ci % 64 == 0 || (p.R * p.S > 1 && (p.Ci + 63) / 64 * 64 * 32LL <= p.Ci * 33LL); }
// Bytes from the first value that a tile of 256 rows (128 of a stride grid) reads to its last: counted from its first image, or -- images of 256 pixels and more, of which it touches two
// at most -- from its first row.
long long conv_dma_span(const GemmConv& p, bool from_row) {
    const int tile = p.scatter ? 128 : 256;
    long long rows = (tile / ((long long)p.Po * p.Qo) + 2) * p.Hi;
    if (from_row) {
        if ((long long)p.Po * p.Qo < tile) return 1LL << 62;
        rows = (tile / p.Qo + 3LL) * p.sh + std::max(0LL, p.Hi - (p.Po - 1LL) * p.sh) + (p.ph < 0 ? -p.ph : 0);
    }
    return ((rows + (p.ph > 0 ? p.ph : 0) + p.R + 1) * p.Wi + p.S + 1) * p.Ci * 2;
}
constexpr long long kSpanLimit = 0x7fff0000LL;
bool conv_dma_far(const GemmConv& p) { return conv_dma_span(p, false) >= kSpanLimit; }
ConvDmaIn conv_dma_in(const GemmConv& p) {
    if ((long long)p.R * p.S > 32 || conv_dma_far(p)) return conv_dma_by_tap(p) ? kRuns : kTaps;
    return p.Ci % 64 == 0 ? kChunks : conv_dma_by_tap(p) ? kPadded : kPieces;
}
int conv_dma_steps(const GemmConv& p) { return conv_dma_by_tap(p) ? (p.Ci + 63) / 64 * p.R * p.S : (p.Kg + 63) / 64; }

// Tiles, and what a k-step of them takes in us where a block has its compute unit to itself, per block where `per_cu` take turns, and the same for what a tile costs
// beyond its k-steps.
struct ConvTile {
    int bm, bn, per_cu;
    float alone, shared, tile;
};
constexpr int kWide = 0, kSquare = 1, kNarrow = 2, kNarrowTwoWaves = 3, kSlim = 4, kOtherRows = 5;
constexpr ConvTile kConvTiles[] = {{256, 256, 1, 1.4f, 1.065f, 1.9f}, {128, 128, 2, 0.41f, 0.2f, 0.8f}, {128, 64, 3, 0.355f, 0.181f, 0.7f}, {128, 64, 3, 0.545f, 0.17f, 0.62f},
                                   {128, 32, 3, 0.36f, 0.115f, 0.45f},
                                   {240, 256, 1, 1.2f, 1.0f, 2.2f},   {224, 256, 1, 1.1f, 0.915f, 2.05f}, {208, 256, 1, 0.88f, 0.86f, 2.2f}, {192, 256, 1, 0.72f, 0.8f, 2.2f}};

struct ConvDmaPlan {
    int tile;                     // of kConvTiles
    int nkt;
    long long tiles;
    SkPlan sk;
};

// Tile and work split by cost, in us: rounds of whole tiles, then the rest whole to one block each, to S blocks each in equal parts, or end to end over the resident
// blocks; shared tiles cost the fix-up's launch, each of a tile's parts in its turn, and what the parts move.  Memory (4.2 MB per us) and what the tiles read from the L2s (15 MB) are taken in by the
// fourth-power mean, since none hides behind another entirely.  Fitted to 178 layers of 1 to 512 images, forward, every tile with up to nine splits: the choice is 1.7 %
// off the best in the mean, 6 % or more in one of ten, and 1.3 times as fast in the mean as the kernels with staging registers that took these layers before
// (3x3 over 256 channels, 512 images of 14x14: 147 -> 106 us).  Results of at most 32 columns have a tile of their own (64 to 32 1x1, 512 images of 56x56: 61 us, 83 with 64 columns).
// Row counts other than 128 and 256 fill the rounds of wide results (that layer has 392 tiles of 256 rows: two rounds for one and a half; 483 of 208: 116 -> 106).  They
// replace a tile that no blocks share, where every sum is the same: so the result does not depend on whether statistics, which come in pieces of 64 or 128 rows, are wanted.
bool conv_dma_plan(const GemmConv& p, bool any_rows, ConvDmaPlan* out) {
    const int cus = device_cu_count(), nkt = conv_dma_steps(p);
    const float pixels = p.R == 1 && p.S == 1 ? (float)p.M : (float)p.M / ((float)p.Po * (float)p.Qo) * (float)p.Hi * (float)p.Wi;
    const float memory = (pixels * (float)p.Ci + (float)p.M * (float)p.N) * (2e-6f / 4.2f);
    auto fourth = [](float x) { return x * x * x * x; };
    const bool rows = !p.scatter && p.N % 8 == 0 && p.ldd % 8 == 0, large = (long long)p.R * p.S > 32 || conv_dma_far(p);
    float best = 1e30f;
    out->nkt = nkt;
    auto tile_cost = [&](int i) {
        const ConvTile& t = kConvTiles[i];
        const long long tiles = (long long)((p.M + t.bm - 1) / t.bm) * ((p.N + t.bn - 1) / t.bn);
        if (tiles * nkt >= 0x7fffffffLL) return;
        const int resident = t.per_cu * cus, rest = (int)(tiles % resident);
        const float whole = (float)(tiles / resident * t.per_cu) * ((float)nkt * t.shared + t.tile);
        const float others = fourth(memory) + fourth((float)tiles * (float)nkt * (float)(t.bm + t.bn) * (128e-6f / 15.f));
        auto consider = [&](int blocks, bool even) {
            const int steps = rest ? (int)(((long long)rest * nkt + blocks - 1) / blocks) : 0;
            float us = whole;
            if (rest) {
                const float turns = (float)((blocks + cus - 1) / cus);
                float r = std::max((float)steps * t.alone + t.tile, turns * ((float)steps * t.shared + t.tile));
                if (!even) r *= 1.15f;                     // (unequal parts: blocks no longer read the same rows together)
                us += r;
                if (blocks != rest) us += 3.2f + 0.35f * (float)((blocks + rest - 1) / rest) + 0.016f * (float)blocks * (float)(t.bm * t.bn) / 16384.f;
            }
            us = sqrtf(sqrtf(fourth(us) + others));
            if (us < best) {
                best = us;
                out->tile = i;
                out->tiles = tiles;
                out->sk.dp_tiles = (int)(tiles - rest);
                out->sk.sk_blocks = rest ? blocks : 0;
                out->sk.sk_iters = (long long)rest * nkt;
            }
        };
        consider(rest ? rest : 1, true);
        if (rest == 0 || i == kWide || i >= kOtherRows) return;
        // (kRuns and kTaps: every number of parts; 512 to 512 7x7, 64 images of 7x7, 392 k-steps: five parts 85 us, end to end 117, staging registers 111)
        for (int s = 2; s <= 16 && rest * s <= resident && nkt >= 2 * s; s += large || s < 4 ? 1 : s < 8 ? 2 : 4) consider(rest * s, true);
        const int all = (int)std::min<long long>(resident, (long long)rest * nkt / 2);
        if (all > rest) consider(all, false);
    };
    if (p.N > 128 && rows) tile_cost(kWide);
    if (p.N > 64) tile_cost(kSquare);
    tile_cost(kNarrow);
    if (!large) tile_cost(kNarrowTwoWaves);               // (kRuns and kTaps are built for three of the tiles)
    if (!large && p.N <= 32) tile_cost(kSlim);
    if (best >= 1e30f) return false;
    if (any_rows && !large && p.N > 128 && rows && out->sk.sk_iters == (long long)out->sk.sk_blocks * nkt)
        for (int i = kOtherRows; i < (int)(sizeof(kConvTiles) / sizeof(kConvTiles[0])); ++i) tile_cost(i);
    return true;
}
bool conv_dma_shares(const ConvDmaPlan& c) { return c.sk.sk_iters != (long long)c.sk.sk_blocks * c.nkt; }

// kOnce: kChunks with the rows past the caches.  Each is read once -- a 1x1 window, one tile of columns -- and the memory-side cache does not hold the image (us, 512 to 128
// at 28x28, 512 images 105 / 102, 256 to 64 at 56x56 188 / 182).  Windows and further tiles of columns read them again: 3x3 over 128 channels 130 / 167, 256 to 1024 at 14x14 72 / 82.
// (An instance of its own: the choice within the loop cost windows 1 to 2 %.)
bool conv_dma_once(const GemmConv& p, int bn) { return p.N <= bn && p.R * p.S == 1 && !p.scatter && ((p.N | p.ldd) & 7) == 0 && (double)p.M * p.Ci * 2 >= 256e6; }

template <int TMA, int TMB, int TN, int WN>
lc_status launch_conv_dma(const GemmConv& q, const ConvDmaPlan& plan, hipStream_t stream) {
    constexpr int BM = 16 * (TMA + TMB), BN = 16 * TN * WN, threads = 2 * WN * 64;
    constexpr int lds = 2 * (BM + BN) * 128 + 2 * WN * 16 * (TN * 32 + 16);
    ConvDma c = {q, plan.nkt, 0, 0, 0, 0, 32 / q.S};
    GemmConv& p = c.g;
    const long long tiles = plan.tiles;
    const int nkt = plan.nkt, resident = kConvTiles[plan.tile].per_cu * device_cu_count();
    SkPlan pl = plan.sk;
    if (pl.sk_blocks > 0 && !p.partial) pl.sk_blocks = 0;
    if (pl.sk_blocks == 0) {
        const long long rest = tiles % resident;
        pl.dp_tiles = (int)(tiles - rest);
        pl.sk_blocks = (int)rest;
        pl.sk_iters = rest * nkt;
    }
    p.dp_tiles = pl.dp_tiles;
    p.sk_blocks = pl.sk_blocks;
    p.sk_iters = pl.sk_iters;
    sk_constants(&p);
    magic_for(p.Qo, &p.qo_mul, &p.qo_shift);
    magic_for(p.Po, &p.po_mul, &p.po_shift);
    magic_for(p.Ci, &c.ci_mul, &c.ci_shift);
    magic_for(p.S, &c.s_mul, &c.s_shift);
    const unsigned grid = pl.dp_tiles > 0 ? (unsigned)resident : (unsigned)pl.sk_blocks;
    lc_status st = LC_OK;
    auto launch = [&]<ConvDmaIn IN, ConvDmaOut OUT>() {
        static const bool once = hipFuncSetAttribute(reinterpret_cast<const void*>(conv_dma_kernel<TMA, TMB, TN, WN, IN, OUT>),
                                                     hipFuncAttributeMaxDynamicSharedMemorySize, lds) == hipSuccess;
        if (!once) st = LC_ERR_LAUNCH;
        else hipLaunchKernelGGL((conv_dma_kernel<TMA, TMB, TN, WN, IN, OUT>), dim3(grid), dim3(threads), lds, stream, c);
    };
    auto out = [&]<ConvDmaIn IN>() {
        if constexpr (WN != 4 || (TMA == 8 && TMB == 8)) {
            if (p.stats) return launch.template operator()<IN, kStats>();
        }
        if constexpr (WN != 4 && IN != kOnce) {
            if (p.scatter) return launch.template operator()<IN, kGrid>();
            if (((p.N | p.ldd) & 7) != 0) return launch.template operator()<IN, kAny>();
        }
        launch.template operator()<IN, kRows>();
    };
    switch (conv_dma_in(p)) {
        case kChunks:
            if constexpr (TMA == TMB && TMA != 7 && TMA != 6) {
                if (conv_dma_once(p, BN)) {
                    out.template operator()<kOnce>();
                    break;
                }
            }
            out.template operator()<kChunks>();
            break;
        case kPadded: out.template operator()<kPadded>(); break;
        case kPieces: out.template operator()<kPieces>(); break;
        default:
            if constexpr (TMA == TMB && TMA != 7 && TMA != 6 && WN != 1) conv_dma_in(p) == kRuns ? out.template operator()<kRuns>() : out.template operator()<kTaps>();
            else st = LC_ERR_UNSUPPORTED;
    }
    if (st != LC_OK) return st;
    // (the plan shares tiles of up to 128 columns, among more blocks than tiles: ranges shorter than a tile)
    if constexpr (WN != 4) {
        if (pl.sk_blocks > 0 && pl.sk_iters != (long long)pl.sk_blocks * nkt)
            hipLaunchKernelGGL((conv_dma_fixup_kernel<TMA, TN, WN>), dim3((unsigned)(tiles - pl.dp_tiles), TMA * TN), dim3(threads), 0, stream, p, nkt);
    }
    return lc_end_call();
}

// ------------------------------------------------------------------------------------------------
// 3x3 windows (stride 1, padding 1) from 64 channels to 33 to 64 filters, forward and backward-data: every wave holds the whole filter in registers (288 of its
// 512: one wave per SIMD) and only pixels move.
//
// With so few columns a wave of a tile kernel reads as many bytes of LDS as it multiplies, and fetches its pixels nine times: 512 images of 56x56 took 174 us (slab
// kernel of conv_igemm.hip, half of its fragment reads the filter's) to 189 (conv_dma_kernel) of the 86 its products take.  Here 1 KB of pixels feeds four matrix instructions, half of
// what LDS gives.  Bound by its one wave per SIMD, beside which nothing hides a wait: the matrix pipe is busy in 42 % of the cycles at 2.03 GHz, LDS in 30 % (half of that bank conflicts), memory
// moves 3.1 TB/s.  us against the slab kernel in the same run: 512 images of 56x56 to 64 153 / 218 (with
// statistics 162 / 203), to 48 123 / 182, 256 images 66 / 90, 128 images of 112x112 149 / 200.
//
// A block is persistent; its tile is `tr` whole rows of an image, whose pixels with their halo go straight into LDS, one tile ahead: two planes of 32 channels (64
// bytes a pixel), so that a half is an immediate offset, 16-byte pieces at piece ^ (column / 4 % 4), so that a piece of sixteen neighbouring pixels meets every bank once (by the counters half
// of the cycles LDS is busy are conflicts all the same, against 2 to 7 % in conv_dma_kernel's windows: not explained yet).  A tap is a
// displacement of the lane's address; rows above the image are masked and rows below it lie past the end of the buffer.  The four waves take 16 pixels at a time in turn;
// a group's results leave while the next one is multiplied.  The sums run over the taps of 32 channels and then of the others, as in the slab kernel: the same bits.
// ------------------------------------------------------------------------------------------------
constexpr int kHeldPixels = 592;                           // of a tile with its halo
struct ConvHeld {
    GemmConv g;
    int tr, per_image, tiles, groups, turns;               // rows of a tile, tiles of an image, all tiles; loads of 16 pixels, turns of 64 pixels
    unsigned w_mul, w_shift, w2_mul, w2_shift, t_mul, t_shift;
};

template <bool STATS>
__global__ void __launch_bounds__(256, 1) conv3x3_held_kernel(const ConvHeld pp) {
    const GemmConv& p = pp.g;
    constexpr int PLANE = kHeldPixels * 64, STAGE = 2 * PLANE, LOADS = (kHeldPixels / 16 + 3) / 4, kOutPitch = 144, AHEAD = 5, SLOTS = 6;
    extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int H = p.Hi, W = p.Wi, W2 = W + 2, N_ = p.N, ldd_ = p.ldd, tr = pp.tr, G = gridDim.x;
    const int lpx = lane & 15, g = lane >> 4;
    unsigned char* const mine = smem + 2 * STAGE + wave * (16 * kOutPitch);
    const unsigned lds0 = lds_address(smem);

    // ---------------- load side: load j of this wave is pixels 16 * (4 j + wave) .. + 15 of the slab, four lanes each ----------------
    unsigned a_voff[LOADS];
#pragma unroll
    for (int j = 0; j < LOADS; ++j) {
        const int px = (j * 4 + wave) * 16 + (lane >> 2);
        const int row = div_by(px, pp.w2_mul, pp.w2_shift), col = px - row * W2;
        const bool ok = (row < tr + 2) & (col >= 1) & (col <= W);
        a_voff[j] = ok ? (unsigned)((row * W + col - 1) * 128 + (((lane & 3) ^ ((col >> 2) & 3)) * 16)) : kBufferBytes;
    }
    auto load_tile = [&](int tile, int stage) __attribute__((always_inline)) {
        const int img = div_by(tile, pp.t_mul, pp.t_shift), row0 = (tile - img * pp.per_image) * tr;
        const uint16_t* const first = static_cast<const uint16_t*>(p.a) + ((long long)img * H + row0 - 1) * W * 64;
        const u32x4 rsrc = buffer_words(first, (unsigned)((H - row0 + 1) * W * 128));
#pragma unroll
        for (int j = 0; j < LOADS; ++j) {
            const int group = j * 4 + wave;
            if (group < pp.groups) {
                unsigned v = a_voff[j];
                if (row0 == 0 && group * 16 < W2) v |= group * 16 + (lane >> 2) < W2 ? kBufferBytes : 0u;      // the row above the image
                load_to_lds(rsrc, v, 0, lds0 + stage + group * 1024);
                load_to_lds(rsrc, v, 64, lds0 + stage + PLANE + group * 1024);
            }
        }
    };

    int n = blockIdx.x, stage = 0;                         // the grid is at most the tiles
    int tile = xcd_tile(n, pp.tiles);
    load_tile(tile, 0);

    // the filter: tap, half of the channels, 16 filters
    bf16x8 wf[9][2][4];
    {
        const __amdgpu_buffer_rsrc_t b_rsrc = __builtin_amdgcn_make_buffer_rsrc((void*)p.b, 0, N_ * 9 * 128, (int)kBufferWords3);
#pragma unroll
        for (int t = 0; t < 9; ++t)
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    wf[t][h][j] = __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(b_rsrc, (lpx * 9 * 64 + g * 8) * 2, (j * 16 * 9 * 64 + t * 64 + h * 32) * 2, 0));
    }

    // (the compiler would keep the fragments that don't fit in vector registers in accumulation registers and copy them for every use)
#pragma unroll
    for (int t = 4; t < 9; ++t)
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int j = 0; j < 4; ++j) asm volatile("" : "+a"(wf[t][h][j]));

    // ---------------- compute side ----------------
    f32x4 acc[2][4];
    bf16x8 fa[SLOTS];
    unsigned at[9], tap0[3];
    const int pixels = tr * W, row_bytes = W2 * 64;
    auto turn_addresses = [&](int turn) __attribute__((always_inline)) {       // this lane's pixel under the first row of taps
        const int m = min((turn * 4 + wave) * 16 + lpx, pixels - 1);
        const int row = div_by(m, pp.w_mul, pp.w_shift), q = m - row * W;
#pragma unroll
        for (int s = 0; s < 3; ++s) tap0[s] = (unsigned)((row * W2 + q + s) * 64 + ((g ^ (((q + s) >> 2) & 3)) * 16));
    };
    auto tap_address = [&](int rs, int stage) __attribute__((always_inline)) { at[rs] = tap0[rs % 3] + (unsigned)(stage + rs / 3 * row_bytes); };
    auto read = [&](int k) __attribute__((always_inline)) {                    // k-step k = 9 half + tap
        fa[k % SLOTS] = *reinterpret_cast<const bf16x8*>(smem + at[k % 9] + k / 9 * PLANE);
    };
    float sum[8], sq[8];                                   // of the stored values in this lane's columns of a row
    int valid = 0;                                         // pixels of the tile inside the image
    __amdgpu_buffer_rsrc_t d_rsrc = __builtin_amdgcn_make_buffer_rsrc((void*)p.d, 0, 0, (int)kBufferWords3);
    const unsigned d_voff = lane % 8 * 8 < N_ ? (unsigned)((lane / 8 * ldd_ + lane % 8 * 8) * 2) : kBufferBytes;
    u32x4 out[2];
    auto out_write = [&](const f32x4(&a)[4], int j) __attribute__((always_inline)) {
        const uint2 u = make_uint2(lc_bf16x2_rne(a[j][0], a[j][1]), lc_bf16x2_rne(a[j][2], a[j][3]));
        *reinterpret_cast<uint2*>(mine + lpx * kOutPitch + j * 32 + g * 8) = u;
    };
    auto out_read = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int e = 0; e < 2; ++e) out[e] = *reinterpret_cast<const u32x4*>(mine + (e * 8 + lane / 8) * kOutPitch + lane % 8 * 16);
    };
    auto out_store = [&](int turn) __attribute__((always_inline)) {
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            const int m = (turn * 4 + wave) * 16 + e * 8;
            if (__builtin_expect(p.stream_d, 0)) __builtin_amdgcn_raw_buffer_store_b128(out[e], d_rsrc, (int)d_voff, m * ldd_ * 2, kNonTemporal);
            else __builtin_amdgcn_raw_buffer_store_b128(out[e], d_rsrc, (int)d_voff, m * ldd_ * 2, 0);
            if (STATS) {
                const unsigned in = m + lane / 8 < valid ? ~0u : 0u;
#pragma unroll
                for (int c = 0; c < 8; ++c) {
                    if (c % 2 == 0) out[e][c / 2] &= in;   // (the store has read it)
                    const float x = __uint_as_float(c & 1 ? out[e][c / 2] & 0xffff0000u : out[e][c / 2] << 16);
                    sum[c] += x;
                    sq[c] = fmaf(x, x, sq[c]);
                }
            }
        }
    };
    const int turns = pp.turns;
    // One turn.  Fragments are read five k-steps ahead, behind the last ones those of the next turn (of the next tile: read again behind the barrier); a tap's
    // address is the next turn's as soon as its fragments are under way; the former turn's results leave on the way.
    auto turn = [&]<int CUR>(std::integral_constant<int, CUR>, int i, int stage) __attribute__((always_inline)) {
        const bool last = i + 1 == turns;
        const int next_stage = last ? STAGE - stage : stage;
        turn_addresses(last ? 0 : i + 1);
        int former = i;
        asm volatile("" : "+s"(former));                   // (one loop for the first turn and the others)
#pragma unroll
        for (int k = 0; k < 18; ++k) {
            if (k + AHEAD < 18) read(k + AHEAD);
            else read(k + AHEAD - 18);
            if (k >= 4 && k <= 12) tap_address(k - 4, next_stage);
            if (former) {
                if (k == 2 || k == 3) {
                    out_write(acc[CUR ^ 1], 2 * (k - 2));
                    out_write(acc[CUR ^ 1], 2 * (k - 2) + 1);
                }
                if (k == 6) out_read();
                if (k == 12) out_store(i - 1);
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const f32x4 c = k == 0 ? f32x4{0.f, 0.f, 0.f, 0.f} : acc[CUR][j];
                acc[CUR][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[k % 9][k / 9][j], fa[k % SLOTS], c, 0, 0, 0);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
    };

    turn_addresses(0);
#pragma unroll
    for (int rs = 0; rs < 9; ++rs) tap_address(rs, 0);
    wait_loads_and_barrier<0>();
    for (;;) {
        const int img = div_by(tile, pp.t_mul, pp.t_shift), in_image = tile - img * pp.per_image, row0 = in_image * tr;
        valid = min(tr, H - row0) * W;
        d_rsrc = __builtin_amdgcn_make_buffer_rsrc((void*)(static_cast<uint16_t*>(p.d) + ((long long)img * H + row0) * W * ldd_), 0, valid * ldd_ * 2, (int)kBufferWords3);
        if (STATS) {
#pragma unroll
            for (int c = 0; c < 8; ++c) sum[c] = sq[c] = 0.f;
        }
#pragma unroll
        for (int k = 0; k < AHEAD; ++k) read(k);
        n += G;
        const int following = n < pp.tiles ? xcd_tile(n, pp.tiles) : -1;
        if (following >= 0) load_tile(following, STAGE - stage);
        for (int i = 0; i < turns; i += 2) {
            turn(std::integral_constant<int, 0>{}, i, stage);
            if (i + 1 < turns) turn(std::integral_constant<int, 1>{}, i + 1, stage);
        }
        auto flush = [&](const f32x4(&a)[4]) __attribute__((always_inline)) {
#pragma unroll
            for (int j = 0; j < 4; ++j) out_write(a, j);
            out_read();
            out_store(turns - 1);
        };
        // this stage has been read, the next has arrived: the two youngest operations are stores
        if (turns > 1) wait_loads_and_barrier<2>();
        else wait_loads_and_barrier<0>();
        if (turns & 1) flush(acc[0]);
        else flush(acc[1]);
        if (STATS) {                                       // a piece per wave and tile
            typedef float flt2 __attribute__((ext_vector_type(2)));
            flt2* const st = reinterpret_cast<flt2*>(p.stats) + ((size_t)tile * 4 + wave) * N_;
#pragma unroll
            for (int c = 0; c < 8; ++c) {
                float a = sum[c], b = sq[c];               // lanes 8, 16 and 32 apart hold the same column
#pragma unroll
                for (int o = 8; o < 64; o *= 2) {
                    a += __shfl_xor(a, o);
                    b += __shfl_xor(b, o);
                }
                if (lane < 8 && lane * 8 < N_) st[lane * 8 + c] = flt2{a, b};
            }
        }
        if (following < 0) break;
        tile = following;
        stage = STAGE - stage;
    }
}

// Rows of a tile: as many as LDS holds, or fewer where that wastes less on whole groups of 64 pixels, on the last tile of an image and on the last round.  False
// where more than a fifth of the products would be wasted all the same, or a block has so few turns that fetching the filter and the first
// tile (some 10 us) is not worth it.  us, this kernel / slab kernel, plain and with statistics: 512 images of 16x16, 8 turns 21 / 19 and 25 / 19;
// 64 of 56x56, 14 turns 27 / 28 and 31 / 29; 128 of 56x56, 28 turns 43 / 49 and 52 / 51; 256 of 56x56, 49 turns 66 / 90 and 80 / 91.  Both give the same bits.
bool conv_held_plan(const GemmConv& p, bool stats, ConvHeld* c) {
    const int cus = device_cu_count(), W2 = p.Wi + 2, most = std::min(p.Hi, kHeldPixels / W2 - 2);
    const char* e = getenv("LARSCONV_HELD_MIN_TURNS");     // tests lower it to send small shapes here
    const long long min_turns = e ? atoll(e) : stats ? 32 : 16;
    float best = 0.f;
    for (int tr = 1; tr <= most; ++tr) {
        const int per_image = (p.Hi + tr - 1) / tr, turns = (tr * p.Wi + 63) / 64;
        const long long tiles = (long long)p.M / ((long long)p.Hi * p.Wi) * per_image, rounds = (tiles + cus - 1) / cus;
        if (tiles > 0x7fffffff || rounds * turns < min_turns) continue;
        // (what a tile costs beyond its turns: a third of one)
        const float share = (float)p.M / ((float)rounds * (float)cus * ((float)turns + 0.33f) * 64.f);
        if (share > best) {
            best = share;
            c->tr = tr;
            c->per_image = per_image;
            c->tiles = (int)tiles;
            c->groups = ((tr + 2) * W2 + 15) / 16;
            c->turns = turns;
        }
    }
    return best >= 0.8f;
}

// ------------------------------------------------------------------------------------------------
// Filter gradient: D[k][j] = sum_m dY[m][k] * X(m, j), j = (r, s, c), a reduction over the rows m with both operands contiguous along their output
// index.  LDS holds [row][W columns] as the rows arrive; the matrix operands come from the transposing LDS read.
//
// A stage is 32 rows of each operand.  One load fills 1 KB: 512 / W whole rows.  The transposing read of a wave takes 32 bytes of rows
// 8g + 0..3 (then 8g + 4..7) for g = 0..3, and LDS serves the lanes of two g at a time: those eight rows are spread over loads 1056 bytes apart (and, with
// W = 64, over the halves of a load), which puts their pieces on eight distinct eighths of the banks.
//
// Bound: wide tiles by power (256x256: the matrix pipe busy in 67 % of the cycles at 1.71 GHz, 128x256 on windows 56 % at 1.89; LDS 36 %), 1x1 layers by
// memory.  Whole calls at batch 512, us, gathering / plain / slab kernel with staging registers before -> now: 3x3 over 256 channels at 14x14 174 -> 108 (1,090 TFLOP/s),
// 3x3 over 128 at 28x28 188 -> 127, 1x1 stride 2 512 to 1024 at 28x28 177 -> 110, 512 to 128 1x1 at 28x28 130 -> 102 (5.0 TB/s), 256 to 64 at 56x56 209 -> 181.
// ------------------------------------------------------------------------------------------------
template <int W>
struct WgradRows {
    static constexpr int kRowBytes = 2 * W, kPerLoad = 512 / W, kLoads = 32 / kPerLoad, kPitch = 1024 + 32, kBytes = kLoads * kPitch;
    static __device__ __forceinline__ int first_row(int load) { return (load & 3) + 8 * (load >> 2); }
    // the u-th row of a load, counted from its first; row and columns of a lane
    static __device__ __forceinline__ int row_of(int u) {
        if (W == 256) return 4 * u;
        if (W == 128) return 4 * (u & 1) + 16 * (u >> 1);
        return 8 * (u & 1) + 4 * ((u >> 1) & 1) + 16 * (u >> 2);
    }
    static __device__ __forceinline__ int lane_row(int lane) { return row_of(lane * 16 / kRowBytes); }
    static __device__ __forceinline__ int lane_col(int lane) { return lane * 16 % kRowBytes / 2; }
    // the transposing read: this lane's byte offset for the rows 8g + 0..3 of columns 0..15, and how far the rows 8g + 4..7 are behind
    static constexpr int kSecond = W == 64 ? 256 : kRowBytes;
    static __device__ __forceinline__ int frag(int lane) {
        const int g = lane >> 4, r = (lane & 15) >> 2;
        const int row = W == 256 ? (r + 4 * g) * kPitch : W == 128 ? (r + 4 * (g & 1)) * kPitch + (g >> 1) * 512
                                                                   : r * kPitch + (g & 1) * 128 + (g >> 1) * 512;
        return row + (lane & 3) * 8;
    }
};

struct WgradDma {
    GemmWgrad g;
    int chain;                    // stages (an even number) after which a wave's sums go to a second set
    unsigned q_mul, q_shift, p_mul, p_shift;
};

// Rows that may go into one running sum: those of a split where the splits fill a round of the staging-register kernels' blocks, or of the slab kernel's where it would
// take the layer if that had 64 channels and filters.  The error of a sum in fp32 grows with the root of its length, and fewer splits than that would show (1x1, 512 images of 28x28,
// 512 to 128: 64 splits of 6272 rows 4.0e-7, 256 splits 2.0e-7; 3x3, 440 of 24x24, 448 to 64: sums of 7904 rows 4.6e-7, of 3472 2.9e-7).
inline int wgrad_former_splits(const GemmWgrad& p) {
    int splits = lc_wgrad_round_splits(p), positions;
    const int imgs = (int)(p.M / ((long long)p.P * p.Q));
    if (p.R == 3 && p.S == 3 && p.sh == 1 && p.sw == 1 && p.ph == 1 && p.pw == 1 && p.C % 64 == 0 && p.K % 64 == 0 && p.W >= kWgradSlabMinW)
        splits = std::max(splits, lc_wgrad_slab_splits(imgs, p.H, p.W, p.C, p.K, &positions));
    return splits;
}
inline int wgrad_chain_rows(const GemmWgrad& p) { return (p.M + wgrad_former_splits(p) - 1) / wgrad_former_splits(p); }
// Stages of a running sum, an even number.  Where one split has taken the place of several, their additions (lc_reduce_splits: four interleaved sums) are saved, and the sums may be
// longer by as much: 48 rows round as often as one addition of everything (measured: 64; 3x3 over 512 channels, 37 images of 7x7, ten stages for eight: 28 -> 26 us, error 0.93 of the seven
// splits', with eight 0.86).
inline int wgrad_chain_stages(const GemmWgrad& p) {
    int rows = wgrad_chain_rows(p);
    const int parts = wgrad_former_splits(p), each = parts / 4, first = each + parts % 4;
    if (p.splits == 1 && parts > 2) {
        int added = first * (first + 1) / 2 - 1;           // how many parts the result of each addition holds
        if (each > 0) added += 3 * (each * (each + 1) / 2 - 1) + 2 * parts;
        rows += 48 * (added - parts) / parts;
    }
    return std::max(2, rows / 64 * 2);
}

// Columns of the result: one pixel's channels in 256-wide pieces (or, kPlain -- a 1x1 window with stride 1 and no padding -- any of the widths).
enum WgradIn { kWindow, kPlain, kAround };
template <int BM, int BN, int WM, int WN, int NS, WgradIn IN>
__global__ void __launch_bounds__(WM* WN * 64, BM * BN <= 64 * 128 ? 3 : 2) wgrad_dma_kernel(const WgradDma pp) {
    const GemmWgrad& p = pp.g;
    using RA = WgradRows<BM>;
    using RB = WgradRows<BN>;
    constexpr int NW = WM * WN, LA = RA::kLoads / NW, LB = RB::kLoads / NW, LPW = LA + LB;
    constexpr int TM = BM / WM / 16, TN = BN / WN / 16;
    constexpr int STAGE = RA::kBytes + RB::kBytes;
    static_assert(RA::kLoads % NW == 0 && RB::kLoads % NW == 0 && TM % 4 == 0 && 64 % (LB * RB::kPerLoad) == 0, "tile shape");
    extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave / WN, wn = wave % WN;
    const int nbn = (p.J + BN - 1) / BN;
    // split-major, dealt to the XCDs in contiguous runs: the tiles of a split read the same rows and share one L2
    const int tiles_ = ((p.K + BM - 1) / BM) * nbn;
    const int work = xcd_tile(blockIdx.x, tiles_ * p.splits);
    const int z = work / tiles_, tile = work - z * tiles_;
    const int k0 = (tile / nbn) * BM, j0 = (tile % nbn) * BN;
    const int m_begin = z * p.m_per_split;
    const int m_end = min(p.M, m_begin + p.m_per_split);
    const int K_ = p.K, C_ = p.C, J_ = p.J, H_ = p.H, W_ = p.W, R_ = p.R, S_ = p.S, P_ = p.P, Q_ = p.Q;
    const int sh_ = p.sh, sw_ = p.sw, ph_ = p.ph, pw_ = p.pw;

    // dY: rows past the end of the split lie past the end of the buffer
    const uint16_t* const DY = static_cast<const uint16_t*>(p.dy);
    const uint16_t* const X = static_cast<const uint16_t*>(p.x);
    constexpr bool PLAIN = IN != kWindow, AROUND = IN == kAround;      // AROUND: stage t of split z is rows 32 * (t * splits + z) and on
    const int rows = AROUND ? max(((p.M + 31) / 32 - z + p.splits - 1) / p.splits, 0) * 32 : max(m_end - m_begin, 0);
    u32x4 a_rsrc = buffer_words(DY + (long long)m_begin * K_, (unsigned)rows * (unsigned)K_ * 2u);
    const int a_col = k0 + RA::lane_col(lane);
    const unsigned a_voff = a_col < K_ ? (unsigned)(RA::lane_row(lane) * K_ + a_col) * 2u : kBufferBytes;
    // X
    const int img_first = PLAIN ? 0 : m_begin / (P_ * Q_);
    const int phb = max(ph_, 0), pwb = max(pw_, 0);
    u32x4 b_rsrc = PLAIN ? buffer_words(X + (long long)m_begin * C_, (unsigned)rows * (unsigned)C_ * 2u)
                               : buffer_words(X + ((long long)img_first * H_ * W_ - ((long long)phb * W_ + pwb)) * C_, kBufferBytes);
    const int b_col = j0 + RB::lane_col(lane);
    unsigned b_voff = kBufferBytes, b_up = 0;
    if (b_col < J_) {
        if constexpr (PLAIN) {
            b_voff = (unsigned)(RB::lane_row(lane) * C_ + b_col) * 2u;
        } else {
            const int rs = b_col / C_, fc = b_col - rs * C_;
            const int fr = rs / S_, fs = rs - fr * S_;
            b_voff = (unsigned)(((fr * W_ + fs) * C_ + fc) * 2);
            b_up = 31u - (unsigned)rs;
        }
    }
    const WindowTaps window(R_, S_);
    const unsigned lds0 = lds_address(smem);

    int mt = 0;                                            // first row (from m_begin) of the stage being loaded
    unsigned l_lds = lds0;                                 // its LDS address
    // Rows of X that are pixels under a window: the byte offset of the window and its taps outside the image, one row per lane for sixteen stages of
    // this wave's loads at a time, through LDS (worked out row by row on the scalar unit: 3x3 over 256 channels, 512 images of 14x14 174 -> 100 us).
    constexpr int kPix = LB * RB::kPerLoad, kPixStages = 64 / kPix;
    uint2* const pixels = reinterpret_cast<uint2*>(smem + NS * STAGE) + wave * 64;
    int pix = 0;                                           // stages loaded
    auto pixels_of_stages = [&]() __attribute__((always_inline)) {
        const int e = lane % kPix, load = e / RB::kPerLoad * NW + wave;
        const int m = m_begin + mt + lane / kPix * 32 + RB::first_row(load) + RB::row_of(e % RB::kPerLoad);
        const int t = div_by(m, pp.q_mul, pp.q_shift), q = m - t * Q_;
        const int im = div_by(t, pp.p_mul, pp.p_shift), pq = t - im * P_;
        const int h0 = pq * sh_ - ph_, w0 = q * sw_ - pw_;
        const unsigned inv = window.outside(h0, w0, H_, W_, R_, S_);
        const bool ok = (m < m_end) & (inv != ~0u);
        pixels[lane] = make_uint2(ok ? (unsigned)((((im - img_first) * H_ + h0 + phb) * W_ + w0 + pwb) * C_ * 2) : 0u, ok ? inv : ~0u);
        asm volatile("s_waitcnt lgkmcnt(0)" : : : "memory");
    };
    uint2 px[LB];
    auto read_pixels = [&]() __attribute__((always_inline)) {
        if constexpr (!PLAIN) {
            if (pix % kPixStages == 0) pixels_of_stages();
#pragma unroll
            for (int l = 0; l < LB; ++l) px[l] = pixels[pix % kPixStages * kPix + l * RB::kPerLoad + lane * 16 / RB::kRowBytes];
            ++pix;
        }
    };
    auto load_one = [&](int l) __attribute__((always_inline)) {       // load l of this wave's LPW for the stage at mt
        if (l < LA) {
            const int load = l * NW + wave;
            if constexpr (AROUND) load_to_lds_nt(a_rsrc, a_voff, RA::first_row(load) * K_ * 2, l_lds + load * RA::kPitch);
            else load_to_lds(a_rsrc, a_voff, (mt + RA::first_row(load)) * K_ * 2, l_lds + load * RA::kPitch);
        } else {
            const int load = (l - LA) * NW + wave;
            const unsigned dst = l_lds + RA::kBytes + load * RB::kPitch;
            if constexpr (AROUND) load_to_lds_nt(b_rsrc, b_voff, RB::first_row(load) * C_ * 2, dst);
            else if constexpr (PLAIN) load_to_lds(b_rsrc, b_voff, (mt + RB::first_row(load)) * C_ * 2, dst);
            else load_to_lds(b_rsrc, ((px[l - LA].y << b_up) & kBufferBytes) | (b_voff + px[l - LA].x), 0, dst);
        }
    };
    auto place_stage = [&]() __attribute__((always_inline)) {
        if constexpr (AROUND) {
            const long long first = ((long long)(mt / 32) * p.splits + z) * 32;
            const int left = (int)max(0ll, min(32ll, (long long)p.M - first));
            a_rsrc = buffer_words(DY + first * K_, (unsigned)left * (unsigned)K_ * 2u);
            b_rsrc = buffer_words(X + first * C_, (unsigned)left * (unsigned)C_ * 2u);
        }
    };
    place_stage();
    auto next_stage = [&]() __attribute__((always_inline)) {
        mt += 32;
        place_stage();
        l_lds += STAGE;
        if (l_lds == lds0 + NS * STAGE) l_lds = lds0;
    };

    f32x4 acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    bf16x8 fa[4], fb[2][TN];
    const unsigned char* const a_lane = smem + RA::frag(lane) + wm * (TM * 32);
    const unsigned char* const b_lane = smem + RA::kBytes + RB::frag(lane) + wn * (TN * 32);
    auto frag = [&](const unsigned char* q, int second) __attribute__((always_inline)) {
        const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)(uintptr_t)q);
        const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)(uintptr_t)(q + second));
        const s16x8 v = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
        return __builtin_bit_cast(bf16x8, v);
    };
    auto read_a = [&](int stage, int i) __attribute__((always_inline)) { fa[i & 3] = frag(a_lane + stage + i * 32, RA::kSecond); };
    auto read_b = [&](int stage, int slot) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < TN; ++j) fb[slot][j] = frag(b_lane + stage + j * 32, RB::kSecond);
    };

    const int nkt = (rows + 31) / 32;
    // NS - 1 stages under way (rows past the end fetch nothing and arrive as zeros)
#pragma unroll
    for (int s = 0; s < NS - 1; ++s) {
        read_pixels();
#pragma unroll
        for (int l = 0; l < LPW; ++l) load_one(l);
        next_stage();
    }
    wait_loads_and_barrier<(NS - 2) * LPW>();
    int stage = 0;                                         // LDS offset of the stage being multiplied
    read_b(0, 0);
    read_a(0, 0);
    read_a(0, 1);
    // One stage.  The loads of the stage NS - 1 further on go to the buffer of the one before this; fragments of dY are read two tiles ahead; behind
    // the barrier before the last two tiles (this stage has been read, the next has arrived) the next stage's first fragments follow.
    auto step = [&](int slot) __attribute__((always_inline)) {
        int following = stage + STAGE;
        if (following == NS * STAGE) following = 0;
        read_pixels();
#pragma unroll
        for (int i = 0; i < TM; ++i) {
            if (i + 2 < TM) {
                read_a(stage, i + 2);
            } else if (i + 2 == TM) {
                wait_loads_and_barrier<(NS - 2) * LPW>();
                read_b(following, slot ^ 1);
                read_a(following, 0);
            } else {
                read_a(following, 1);
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int j = 0; j < TN; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[slot][j], fa[i & 3], acc[i][j], 0, 0, 0);
            // (spread over the tiles before the barrier)
            constexpr int SLOTS = TM - 2;
#pragma unroll
            for (int l = 0; l < LPW; ++l)
                if (l * SLOTS / LPW == i) load_one(l);
            __builtin_amdgcn_sched_barrier(0);
        }
        next_stage();
        stage = following;
    };
    constexpr bool TWO = TM * TN <= 16;                    // (256x256: no registers left, and its splits are as short)
    f32x4 sum[TWO ? TM : 1][TWO ? TN : 1];
    if constexpr (TWO) {
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j) sum[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    int chain = pp.chain;
    for (int kt = 0; kt < nkt; kt += 2) {
        step(0);
        if (kt + 1 < nkt) step(1);
        if constexpr (TWO) {
            if (kt + 2 >= chain) {
                // What an addition to the second set rounds away starts the next run of stages, so that many additions lose no more than one.  (Where a sum
                // is infinite that would be no number: then the whole wave starts from zeros.)
                chain += pp.chain;
                float most = 0.f;
#pragma unroll
                for (int i = 0; i < TM; ++i)
#pragma unroll
                    for (int j = 0; j < TN; ++j) {
                        const f32x4 total = sum[i][j] + acc[i][j];
                        acc[i][j] -= total - sum[i][j];
                        sum[i][j] = total;
#pragma unroll
                        for (int e = 0; e < 4; ++e) most = fmaxf(most, fabsf(total[e]));
                    }
                if (__builtin_amdgcn_ballot_w64(most > 3.4028234e38f)) {
#pragma unroll
                    for (int i = 0; i < TM; ++i)
#pragma unroll
                        for (int j = 0; j < TN; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
                }
            }
        }
    }
    if constexpr (TWO) {
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j) acc[i][j] += sum[i][j];
    }
    // (loads past the end may still be on their way into this block's LDS, and other waves may still read it)
    wait_loads_and_barrier<0>();

    // A lane holds four neighbouring columns of one filter; 16 filters at a time leave through the wave's own LDS slice, so that a store covers whole
    // rows of the wave's part.  Filters past K lie past the end of the buffer.
    constexpr int kOutPitch = TN * 16 + 4, CPR = TN * 4, RPI = 64 / CPR;      // floats; lanes per row, rows per store
    static_assert(NW * 16 * kOutPitch * 4 <= NS * STAGE, "output staging");
    float* const mine = reinterpret_cast<float*>(smem) + wave * (16 * kOutPitch);
    const int kw = k0 + wm * TM * 16;                      // this wave's first filter
    const long long left = (long long)(K_ - kw) * J_ * 4;
    const __amdgpu_buffer_rsrc_t d_rsrc = __builtin_amdgcn_make_buffer_rsrc(
        (void*)(p.d + ((long long)z * K_ + kw) * J_), 0, (int)(left > 0x7fffffffLL ? 0x7fffffffLL : left > 0 ? left : 0), (int)kBufferWords3);
    const int lr = lane / CPR, col = j0 + wn * TN * 16 + lane % CPR * 4;
    const unsigned d_voff = col < J_ ? (unsigned)(lr * J_ + col) * 4u : kBufferBytes;
#pragma unroll
    for (int i = 0; i < TM; ++i) {
#pragma unroll
        for (int j = 0; j < TN; ++j) *reinterpret_cast<f32x4*>(mine + (lane & 15) * kOutPitch + j * 16 + 4 * (lane >> 4)) = acc[i][j];
        asm volatile("s_waitcnt lgkmcnt(0)" : : : "memory");
        f32x4 out[16 / RPI];
#pragma unroll
        for (int e = 0; e < 16 / RPI; ++e) out[e] = *reinterpret_cast<const f32x4*>(mine + (e * RPI + lr) * kOutPitch + lane % CPR * 4);
        asm volatile("s_waitcnt lgkmcnt(0)" : : : "memory");
#pragma unroll
        for (int e = 0; e < 16 / RPI; ++e)
            __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, out[e]), d_rsrc, (int)d_voff, (i * 16 + e * RPI) * J_ * 4, 0);
    }
}

template <int BM, int BN, int WM, int WN, int NS, WgradIn IN>
lc_status launch_wgrad_dma(const GemmWgrad& p, hipStream_t stream) {
    constexpr int lds = NS * (WgradRows<BM>::kBytes + WgradRows<BN>::kBytes) + (IN != kWindow ? 0 : WM * WN * 512);
    static const bool once =
        hipFuncSetAttribute(reinterpret_cast<const void*>(wgrad_dma_kernel<BM, BN, WM, WN, NS, IN>), hipFuncAttributeMaxDynamicSharedMemorySize, lds) ==
        hipSuccess;
    if (!once) return LC_ERR_LAUNCH;
    const long long tiles = (long long)((p.K + BM - 1) / BM) * ((p.J + BN - 1) / BN);
    if (tiles <= 0 || tiles * p.splits > 0x7fffffffLL) return LC_ERR_UNSUPPORTED;
    WgradDma q = {p, wgrad_chain_stages(p), 0, 0, 0, 0};
    magic_for(p.Q, &q.q_mul, &q.q_shift);
    magic_for(p.P, &q.p_mul, &q.p_shift);
    hipLaunchKernelGGL((wgrad_dma_kernel<BM, BN, WM, WN, NS, IN>), dim3((unsigned)(tiles * p.splits)), dim3(WM * WN * 64), lds, stream, q);
    return lc_end_call();
}

bool wgrad_plain(const GemmWgrad& p) {                     // output pixel m reads input pixel m
    return p.R == 1 && p.S == 1 && p.sh == 1 && p.sw == 1 && p.ph == 0 && p.pw == 0 && p.H == p.P && p.W == p.Q;
}

// Tiles, and what a stage (32 rows) of them takes in us: where a block has its compute unit to itself, and per block where `per_cu` take turns.
struct WgradTile {
    int bm, bn, per_cu;
    float alone, shared;
};
constexpr WgradTile kWgradTiles[] = {{256, 256, 1, 0.70f, 0.787f}, {256, 128, 1, 0.37f, 0.44f},  {128, 256, 1, 0.37f, 0.438f}, {128, 128, 2, 0.228f, 0.291f},
                                     {256, 64, 2, 0.344f, 0.219f}, {64, 256, 2, 0.388f, 0.294f}, {128, 64, 3, 0.18f, 0.16f},   {64, 128, 3, 0.197f, 0.195f}};

}  // namespace

// bf16 operands of 16-byte pieces, byte offsets within a tile (the images it can touch plus a window; its filters; its result) below 2^31.
bool lc_conv_dma_ok(const GemmConv& p) {
    static const bool off = getenv("LARSCONV_NO_CONV_DMA") != nullptr;       // comparison runs
    if (off || !p.bf16 || p.Ci % 8 != 0 || !aligned16(p.a) || !aligned16(p.b) || p.dh > 1 || p.dw > 1) return false;
    if (p.M >= 0x7fff0000) return false;
    if (conv_dma_in(p) == kTaps && ((long long)p.Hi + p.R > 1 << 15 || (long long)p.Wi + p.S > 1 << 15)) return false;       // (rows and columns in 16 bits)
    // (large images to at most 64 columns: the main kernel's tile of 256 rows)
    if (conv_dma_far(p) && ((p.N <= 64 && !p.scatter) || conv_dma_span(p, true) >= kSpanLimit)) return false;
    const long long d_span = p.scatter ? (128LL / ((long long)p.Po * p.Qo) + 2) * p.Ho * p.Wo * p.ldd * 2 : 288LL * p.ldd * 2;       // (stride grids have tiles of 128 rows)
    return 257LL * p.Kg * 2 < kSpanLimit && d_span < kSpanLimit;
}

size_t lc_conv_dma_workspace(const GemmConv& p) {
    ConvDmaPlan c;
    if (!conv_dma_plan(p, true, &c) || !conv_dma_shares(c)) return 0;
    return (size_t)2 * c.sk.sk_blocks * kConvTiles[c.tile].bm * kConvTiles[c.tile].bn * sizeof(float);
}

size_t lc_conv_dma_stats_tiles(const GemmConv& p) {
    ConvDmaPlan c;
    if (!conv_dma_plan(p, false, &c)) return 0;
    const int bm = kConvTiles[c.tile].bm;
    return (size_t)2 * ((p.M + bm - 1) / bm);
}

void lc_conv_dma_describe(const GemmConv& p, bool stats, char* text, size_t size) {
    ConvDmaPlan c;
    static const char* const in[] = {"chunks", "padded", "pieces", "runs", "taps"};
    if (!conv_dma_plan(p, !stats, &c)) snprintf(text, size, "none");
    else
        snprintf(text, size, "conv_dma %dx%d%s %s%s", kConvTiles[c.tile].bm, kConvTiles[c.tile].bn, c.tile == kNarrowTwoWaves ? " two waves" : "",
                 in[conv_dma_in(p)], conv_dma_shares(c) ? " shared" : "");
}

lc_status lc_launch_conv_dma(const GemmConv& p, hipStream_t stream) {
    ConvDmaPlan c;
    if (!conv_dma_plan(p, p.stats == nullptr, &c)) return LC_ERR_UNSUPPORTED;
    if (p.scatter && p.stats) return LC_ERR_UNSUPPORTED;
    auto go = [&]<int TMA, int TMB, int TN, int WN>() { return launch_conv_dma<TMA, TMB, TN, WN>(p, c, stream); };
    lc_status st = LC_ERR_UNSUPPORTED;
    switch (c.tile) {
        case kWide: st = go.template operator()<8, 8, 4, 4>(); break;
        case kSquare: st = go.template operator()<4, 4, 4, 2>(); break;
        case kNarrow: st = go.template operator()<4, 4, 2, 2>(); break;
        case kNarrowTwoWaves: st = go.template operator()<4, 4, 4, 1>(); break;
        case kSlim: st = go.template operator()<4, 4, 2, 1>(); break;
        case kOtherRows: st = go.template operator()<8, 7, 4, 4>(); break;
        case kOtherRows + 1: st = go.template operator()<7, 7, 4, 4>(); break;
        case kOtherRows + 2: st = go.template operator()<7, 6, 4, 4>(); break;
        case kOtherRows + 3: st = go.template operator()<6, 6, 4, 4>(); break;
    }
    if (st == LC_OK && p.stats && conv_dma_shares(c) && p.partial) {
        lc_tile_stats(p, kConvTiles[c.tile].bm, kConvTiles[c.tile].bn, c.sk.dp_tiles, c.tiles, stream);
        st = lc_end_call();
    }
    return st;
}

// What conv3x3_held_kernel takes; results whose rows are whole 16-byte pieces.
static bool conv_held_ok(const GemmConv& p, bool stats, ConvHeld* c) {
    static const bool off = getenv("LARSCONV_NO_HELD") != nullptr || getenv("LARSCONV_NO_CONV_DMA") != nullptr;      // comparison runs
    if (off || !p.bf16 || p.Ci != 64 || p.Kg != 576 || p.N <= 32 || p.N > 64 || (p.N | p.ldd) % 8 != 0 || p.scatter || p.dh > 1 || p.dw > 1) return false;
    if (p.R != 3 || p.S != 3 || p.sh != 1 || p.sw != 1 || p.ph != 1 || p.pw != 1 || p.Po != p.Hi || p.Qo != p.Wi) return false;
    if (!aligned16(p.a) || !aligned16(p.b) || !aligned16(p.d)) return false;
    const long long hw = (long long)p.Hi * p.Wi;
    if (p.M % hw != 0 || (hw + 2 * p.Wi) * 128 >= 0x7fff0000LL || 2LL * kHeldPixels * p.ldd * 2 >= 0x7fff0000LL) return false;
    return conv_held_plan(p, stats, c);
}
bool lc_conv_held_ok(const GemmConv& p, bool stats) {
    ConvHeld c;
    return conv_held_ok(p, stats, &c);
}

size_t lc_conv_held_stats_tiles(const GemmConv& p) {
    ConvHeld c;
    return conv_held_ok(p, true, &c) ? (size_t)4 * c.tiles : 0;
}

lc_status lc_launch_conv_held(const GemmConv& p, hipStream_t stream) {
    constexpr int lds = 4 * kHeldPixels * 64 + 4 * 16 * 144;
    static const bool once =
        hipFuncSetAttribute(reinterpret_cast<const void*>(conv3x3_held_kernel<false>), hipFuncAttributeMaxDynamicSharedMemorySize, lds) == hipSuccess &&
        hipFuncSetAttribute(reinterpret_cast<const void*>(conv3x3_held_kernel<true>), hipFuncAttributeMaxDynamicSharedMemorySize, lds) == hipSuccess;
    if (!once) return LC_ERR_LAUNCH;
    ConvHeld c;
    if (!conv_held_ok(p, p.stats != nullptr, &c)) return LC_ERR_UNSUPPORTED;
    c.g = p;
    magic_for(p.Wi, &c.w_mul, &c.w_shift);
    magic_for(p.Wi + 2, &c.w2_mul, &c.w2_shift);
    magic_for(c.per_image, &c.t_mul, &c.t_shift);
    const dim3 grid((unsigned)std::min(c.tiles, device_cu_count()));
    if (p.stats) hipLaunchKernelGGL(conv3x3_held_kernel<true>, grid, dim3(256), lds, stream, c);
    else hipLaunchKernelGGL(conv3x3_held_kernel<false>, grid, dim3(256), lds, stream, c);
    return lc_end_call();
}

// Tile and splits by cost, in us: the stages of a block alone on its compute unit, of blocks that take turns, the operands' bytes at 3.85 MB (as
// few as 23 blocks reach that from what is cached) and what the tiles read from the L2s at 21.5 MB, in the fourth-power mean, since none hides behind
// another entirely; partial sums of several splits cost 0.3 a MB to write and to read again, and the launch that adds them 3.1.  Fitted to 188 layers of 1
// to 512 images with every tile and up to a dozen splits of each timed: the choice is 1.0 % off the best in the mean, 3 % or more in one of ten.
// Against what these layers had before (a round of 128x128 or narrower tiles with register staging, as many splits as fill the chip) 1.4 times as fast in the
// mean; e.g. 3x3 over 512 channels, 37 images of 7x7: seven splits 42, one split, no partial sums at all, 28.
bool lc_wgrad_dma_plan(const GemmWgrad& p, int* bm, int* bn, int* splits) {
    static const bool off = getenv("LARSCONV_NO_WGRAD_DMA") != nullptr || getenv("LARSCONV_NO_UNIFORM_TAP") != nullptr;      // comparison runs
    if (off || !p.bf16 || p.C % 8 != 0 || p.K % 8 != 0 || (long long)p.R * p.S > 32 || getenv("LARSCONV_WGRAD_WIDEN")) return false;
    if (p.M >= 0x7fff0000) return false;                   // (row numbers past the end are worked with)
    if (p.K <= 64 && p.J <= 64) return false;              // (bound by memory and launches; 64x64 tiles of the other kernels)
    const int cus = device_cu_count();
    const float mb = (float)p.K * (float)p.J * 4e-6f;           // one set of partial sums
    const float x_rows = p.R == 1 && p.S == 1 ? (float)p.M : (float)p.M / ((float)p.P * (float)p.Q) * (float)p.H * (float)p.W;
    const float operands = (x_rows * (float)p.C + (float)p.M * (float)p.K) * 2e-6f;      // MB
    auto fourth = [](float x) { return x * x * x * x; };
    const int chain_rows = wgrad_chain_rows(p);
    float best = 1e30f;
    *bm = 0;
    for (const WgradTile& t : kWgradTiles) {
        if ((t.bm > 64 && t.bm >= 2 * p.K) || (t.bn > 64 && t.bn >= 2 * p.J)) continue;      // (half of it would do)
        const long long all = (long long)((p.K + t.bm - 1) / t.bm) * ((p.J + t.bn - 1) / t.bn);
        if (all > 0x7fffff) continue;
        const int tiles = (int)all, most = std::max(1, std::min(t.per_cu * cus / tiles, (p.M + 31) / 32));
        const float read = (float)(t.bm + t.bn) * (64e-6f / 21.5f);
        auto consider = [&](int s) {
            if (s < 1 || s > most) return;
            const int stages = ((p.M + s - 1) / s + 31) / 32;
            if (t.bm * t.bn == 256 * 256 && (p.M + s - 1) / s > chain_rows) return;      // (it has no second set of sums)
            const float steps = (float)stages, blocks = (float)(tiles * s), turns = (float)((tiles * s + cus - 1) / cus);
            if (steps * t.alone >= best || turns * steps * t.shared >= best) return;
            float us = sqrtf(sqrtf(fourth(steps * t.alone) + fourth(turns * steps * t.shared) + fourth(operands / std::min(3.85f, 0.167f * blocks)) +
                                   fourth(blocks * steps * read)));
            if (s > 1) us += 3.1f + 0.3f * mb * (float)s;
            if (us < best) {
                best = us;
                *bm = t.bm;
                *bn = t.bn;
                *splits = s;
            }
        };
        for (int s = 1; s <= 4; ++s) consider(s);
        for (int s = 6; s < most; s += s / 2) consider(s);
        for (int r = 1; r <= t.per_cu; ++r) consider(r * cus / tiles);
        consider(most);
    }
    if (*bm == 0) return false;
    // byte offsets of a split's rows and (but for plain layers, which have no use for them) of the images it touches, and of a wave's filters in the result, below 2^31
    const long long rows = (p.M + *splits - 1) / *splits + 64 + 32 * 6;
    const long long spanned = rows / ((long long)p.P * p.Q) + 2;
    const long long x_span = ((spanned * p.H + (p.ph > 0 ? p.ph : 0) + p.R + 1) * p.W + p.S + 1) * p.C * 2;
    return rows * std::max(p.K, p.C) * 2 < 0x7fff0000LL && (wgrad_plain(p) || x_span < 0x7fff0000LL) && 257LL * p.J * 4 < 0x7fff0000LL;
}

int lc_wgrad_dma_sum_rows(const GemmWgrad& p) {
    return p.dma_bm * p.dma_bn == 256 * 256 ? p.m_per_split : std::min(p.m_per_split, wgrad_chain_stages(p) * 32);
}

lc_status lc_launch_wgrad_dma(const GemmWgrad& p, hipStream_t stream) {
    if (!aligned16(p.dy) || !aligned16(p.x)) return LC_ERR_ALIGN;
    const bool plain = wgrad_plain(p);
    auto go = [&]<int BM, int BN, int WM, int WN, int NS>() {
        // One tile of large operands, bound by memory: all blocks work on one narrow stretch of both (and past the caches: nothing reads them again) instead of each
        // on rows of its own.  64 to 256 1x1, 512 images of 56x56 173 -> 150 us (6.8 TB/s), 256 to 64 172 -> 152.  Several tiles read the same rows, and the L2s
        // hold them better in one place: 512 to 128 at 28x28 104 / 108, 512 to 2048 at 7x7 64 / 73.
        if (plain && p.K <= BM && p.J <= BN && (double)p.M * (p.K + p.C) * 2 >= 128e6) return launch_wgrad_dma<BM, BN, WM, WN, NS, kAround>(p, stream);
        return plain ? launch_wgrad_dma<BM, BN, WM, WN, NS, kPlain>(p, stream) : launch_wgrad_dma<BM, BN, WM, WN, NS, kWindow>(p, stream);
    };
    switch (p.dma_bm * 1000 + p.dma_bn) {
        case 256256: return go.template operator()<256, 256, 2, 4, 4>();
        case 256128: return go.template operator()<256, 128, 4, 2, 5>();
        case 128256: return go.template operator()<128, 256, 2, 4, 5>();
        case 128128: return go.template operator()<128, 128, 2, 2, 4>();
        case 256064: return go.template operator()<256, 64, 4, 1, 3>();
        case 64256: return go.template operator()<64, 256, 1, 4, 3>();
        case 128064: return go.template operator()<128, 64, 2, 2, 4>();
        case 64128: return go.template operator()<64, 128, 1, 4, 4>();
    }
    return LC_ERR_UNSUPPORTED;
}

