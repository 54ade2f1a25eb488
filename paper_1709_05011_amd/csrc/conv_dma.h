// conv_dma_kernel, its plan and its launch: bf16 forward and backward-data with operands straight into LDS.  Instances: tiles of up to 128 columns in conv_dma.hip, of 256
// in conv_dma_wide.hip (they compile side by side).
#pragma once
#include "dma_common.h"

namespace {

// ------------------------------------------------------------------------------------------------
// Forward and backward-data.  A k-step is 64 values of the reduction: 128 bytes of a row, so that a load of 64 lanes covers eight whole lines.  LDS holds a
// stage as [row][128 bytes] with the 16-byte pieces of a row at piece ^ (row / 2 % 8) -- the lanes fetch them in that order -- and a fragment of sixteen rows then
// meets every bank once.  NS stages, two or four; while one is multiplied the others arrive, across tile boundaries (persistent blocks, segments as in SkWalk).
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

template <int TMA, int TMB, int TN, int WN, int NS, ConvDmaIn IN, ConvDmaOut OUT>
__global__ void __launch_bounds__(2 * WN * 64, 2) conv_dma_kernel(const ConvDma pp) {
    const GemmConv& p = pp.g;
    constexpr int BM = 16 * (TMA + TMB), BN = 16 * TN * WN, NW = 2 * WN;
    constexpr int NA = BM / 8, NB = BN / 8;                // loads of a stage
    constexpr int LA = (NA + NW - 1) / NW, LB = NB / NW;
    constexpr int STAGE = (BM + BN) * 128;
    constexpr int kOutPitch = TN * 32 + 16;                // bytes
    static_assert(NB % NW == 0, "tile shape");
    extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
    unsigned char* const bounce = smem + NS * STAGE;

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
    int l_tile = 0, l_f = 0;
    auto load_begin = [&]() __attribute__((always_inline)) {
        if (NS > 2 && l_f >= F) {                          // (the number of loads under way stays the same: these fetch nothing)
            v_bad = kBufferBytes;
            return;
        }
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
            int place = rows + (by_tap ? (u_tap * Ci_ + u_c) * 2 : u_c * 128);
            constexpr bool vector = NS > 2 && !by_tap;     // (the compiler counts u_c in a vector register there)
            if constexpr (vector) place = __builtin_amdgcn_readfirstlane(place);
            load_to_lds<vector>(b_rsrc, b_voff | v_bad, place, l_lds + BM * 128 + load * 1024);
        }
    };
    auto load_end = [&]() __attribute__((always_inline)) {
        if (NS > 2 && l_f >= F) {
            l_lds = l_lds == lds0 + (NS - 1) * STAGE ? lds0 : l_lds + STAGE;
            return;
        }
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
        if constexpr (NS > 2) ++l_f;
        l_lds = l_lds == lds0 + (NS - 1) * STAGE ? lds0 : l_lds + STAGE;
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
        // (the policy of the stores is the whole epilogue's: a choice store by store cost 128 to 1368 1x1, 201 images of 9x9 1.7 %)
        auto leave = [&](auto policy) __attribute__((always_inline)) {
            constexpr int kPolicy = decltype(policy)::value;
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
                            __builtin_amdgcn_raw_buffer_store_b128(out[e], d_rsrc, (int)d_voff, (i * 16 + e * RPI) * ldd_ * 2, kPolicy);
                        } else {
                            const unsigned off = row_off(mw + i * 16 + e * RPI + lr);
                            __builtin_amdgcn_raw_buffer_store_b128(out[e], d_rsrc, (int)(col < N_ ? off + (unsigned)col * 2u : kBufferBytes), 0, kPolicy);
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
        auto epilogue = [&]() __attribute__((always_inline)) {
            if constexpr (OUT == kAny) {
                leave(std::integral_constant<int, 0>{});
            } else {
                if (__builtin_expect(p.stream_d, 0)) leave(std::integral_constant<int, kNonTemporal>{});
                else leave(std::integral_constant<int, 0>{});
            }
        };

        constexpr int kAhead = (NS - 2) * (LA + LB);       // loads that may still be under way when the next step's have arrived
        if constexpr (NS == 2) {
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
        } else {
            static_assert(NS == 2 || (NA % NW == 0 && TM % 2 == 0), "the same number of loads for every wave");
            for (int i = 0; i < NS; ++i) {
                load_begin();
#pragma unroll
                for (int l = 0; l < LA + LB; ++l) load_one(l);
                load_end();
            }
            clear_acc();
            wait_loads_and_barrier<kAhead + LA + LB>();
        }
        read_a(0, 0, 0, 0);
        read_a(0, 0, 1, 1);
#pragma unroll
        for (int j = 0; j < TN; ++j) read_b(0, 0, j);
        bool stored = false;                               // the last step ended in stores that may still be under way
        auto step = [&]<int BUF>(std::integral_constant<int, BUF>, int f, int stage, int other) __attribute__((always_inline)) {
            constexpr int OFF = (BUF * 2 * TM) & 3;
#pragma unroll
            for (int q = 0; q < 2 * TM; ++q) {
                const int h = q / TM;
                if (q + 2 < 2 * TM) {
                    read_a(stage, (q + 2) / TM, (q + 2) % TM, (q + 2 + OFF) & 3);
                    if (q < TN) read_b(stage, 1, q);
                } else if (q + 2 == 2 * TM) {
                    // this stage has been read, the next has arrived
                    if (stored) wait_loads_and_barrier<kAhead + TM * 16 * TN * 32 / 1024>();
                    else wait_loads_and_barrier<kAhead>();
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
                if (q + 2 >= 2 * TM && (NS > 2 || f + 2 < F)) {        // k-step f + NS into the stage just read
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
        if constexpr (NS == 2) {
            for (int f = 0; f < F; f += 2) {
                step(std::integral_constant<int, 0>{}, f, 0, STAGE);
                if (f + 1 < F) step(std::integral_constant<int, 1>{}, f + 1, STAGE, 0);
            }
        } else {
            int stage = 0;
            for (int f = 0; f < F; ++f) {
                const int other = stage == (NS - 1) * STAGE ? 0 : stage + STAGE;
                step(std::integral_constant<int, 0>{}, f, stage, other);
                stage = other;
            }
            wait_loads_and_barrier<0>();                   // (loads past the end may still be on their way into this block's LDS)
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

// kOnce: kChunks with the rows past the caches.  Each is read once -- a 1x1 window, one tile of columns -- and the memory-side cache does not hold the image (us, ordinary loads / so: 512 to 128
// at 28x28, 512 images 105 / 102, 256 to 64 at 56x56 192 / 184, 512 to 64 at 28x28 99 / 90, 1024 to 128, 2048 images of 14x14 186 / 175; tiles of 256 columns within 1 %).  Windows and further tiles of columns read them
// again: 3x3 over 128 channels 130 / 167, 256 to 1024 at 14x14 72 / 82.  A single k-step has nothing to be ahead of: 64 to 32, 512 of 112x112 241 / 249, to 64, 800 of 56x56 127.4 / 126.3, to 256 292 / 295.
// (An instance of its own: the choice within the loop cost windows 1 to 2 %.)
bool conv_dma_once(const GemmConv& p, int bn) { return p.N <= bn && p.R * p.S == 1 && p.Ci > 64 && !p.scatter && ((p.N | p.ldd) & 7) == 0 && (double)p.M * p.Ci * 2 >= 256e6; }

// Blocks that have a compute unit each, and eight k-steps and more: four stages in flight, and 128x128 tiles by eight waves.  One block alone waits for its own loads, which take longer than a k-step's
// products where they come from beyond its L2, and with one wave a SIMD for every read of LDS.  The same sums.  us, two stages / four, forward and backward-data, 24 sets of tensors in turn: 512 to 512
// 3x3, 37 images of 7x7 27.7 / 22.9 and 31.6 / 30.6, one image of 28x28 21.9 / 16.7 and 25.8 / 24.2; 128 to 128 3x3, 16 of 28x28 13.7 / 11.8 and 17.0 / 15.1; 1024 to 256 1x1, 16 of 14x14 12.8 / 10.6; at eight
// and nine k-steps 512 to 512 1x1, four of 14x14 7.8 / 7.5 and 10.9 / 10.5, 64 to 192 3x3, eight of 28x28 8.7 / 8.2 and 15.9 / 15.6.  Of 110 such passes none is slower but 512 to 128 1x1 of one
// image of 5x5, whose sets the L2s hold, 6.0 / 6.9.  So do all forward passes that run again on tensors that the L2s still hold: 0.9 us more at eight k-steps, 1.2 at eighteen (6.4 / 7.2, 10.3 / 11.5), while
// their backward passes, whose filter has just been re-ordered on other units, gain (15.7 / 14.3).
// The ragged layer's times depend on where its tensors lie: 24 or 25 / 26 to 32 and 32 / 28 to 32 over eight places of one set, 26.4 / 27.6 and 33.3 / 28.3 at another; its three passes
// in turn 78.3 -> 68.7 to 69.0 us on three cards and 77.0 on one, with the filter gradient's eight waves.
bool conv_dma_deep(const GemmConv& p, const ConvDmaPlan& c) {
    if ((c.tile != kSquare && c.tile != kNarrow) || c.sk.dp_tiles > 0 || c.sk.sk_blocks > device_cu_count() || conv_dma_in(p) > kPieces) return false;
    return c.sk.sk_blocks > 0 && c.sk.sk_iters >= 8LL * c.sk.sk_blocks;
}

template <int TMA, int TMB, int TN, int WN, int NS>
lc_status launch_conv_dma(const GemmConv& q, const ConvDmaPlan& plan, hipStream_t stream) {
    constexpr int BM = 16 * (TMA + TMB), BN = 16 * TN * WN, threads = 2 * WN * 64;
    constexpr int lds = NS * (BM + BN) * 128 + 2 * WN * 16 * (TN * 32 + 16);
    constexpr bool WIDE = BN == 256;
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
        static const bool once = hipFuncSetAttribute(reinterpret_cast<const void*>(conv_dma_kernel<TMA, TMB, TN, WN, NS, IN, OUT>),
                                                     hipFuncAttributeMaxDynamicSharedMemorySize, lds) == hipSuccess;
        if (!once) st = LC_ERR_LAUNCH;
        else hipLaunchKernelGGL((conv_dma_kernel<TMA, TMB, TN, WN, NS, IN, OUT>), dim3(grid), dim3(threads), lds, stream, c);
    };
    auto out = [&]<ConvDmaIn IN>() {
        if constexpr (!WIDE || (TMA == 8 && TMB == 8)) {
            if (p.stats) return launch.template operator()<IN, kStats>();
        }
        if constexpr (!WIDE && IN != kOnce) {
            if (p.scatter) return launch.template operator()<IN, kGrid>();
            if (((p.N | p.ldd) & 7) != 0) return launch.template operator()<IN, kAny>();
        }
        launch.template operator()<IN, kRows>();
    };
    switch (conv_dma_in(p)) {
        case kChunks:
            if constexpr (TMA == TMB && TMA != 7 && TMA != 6 && NS == 2) {
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
            if constexpr (TMA == TMB && TMA != 7 && TMA != 6 && WN != 1 && NS == 2) conv_dma_in(p) == kRuns ? out.template operator()<kRuns>() : out.template operator()<kTaps>();
            else st = LC_ERR_UNSUPPORTED;
    }
    if (st != LC_OK) return st;
    // (the plan shares tiles of up to 128 columns, among more blocks than tiles: ranges shorter than a tile)
    if constexpr (!WIDE) {
        if (pl.sk_blocks > 0 && pl.sk_iters != (long long)pl.sk_blocks * nkt)
            hipLaunchKernelGGL((conv_dma_fixup_kernel<TMA, TN, WN>), dim3((unsigned)(tiles - pl.dp_tiles), TMA * TN), dim3(threads), 0, stream, p, nkt);
    }
    return lc_end_call();
}

}  // namespace
