// fp32 backward-data and filter gradients on the bf16 matrix pipe of gfx950, with every fp32 operand taken apart into three bf16 values.
// (The forward pass stays with the fp32 matrix instructions of conv_igemm.hip: its last bits decide ReLUs.)
//
// x = h + m + l with h = x rounded to bf16, m = (x - h) rounded to bf16, l the rest: 8 + 8 + 8 significant bits.  Operands are scaled by 2^16 first,
// so that the parts of the smallest fp32 number are above bf16's smallest (2^-133) and the three parts are exact down to 2^-149.  Of the
// nine partial products of a * b the six hh, hm, mh, mm, hl, lh reach the last bit of an fp32 product (the three left out are below 2^-24 of
// it together); each is exact in the matrix pipe.  Six v_mfma_f32_16x16x32_bf16 take 96 cycles
// where the same sums cost v_mfma_f32_32x32x2_f32 256.  The products of one k-step are summed by themselves and then added to the accumulators with
// one rounding, which leaves errors of a fifth to a half of those of fp32 instructions (see sum_products()).
// Measured at batch 256, whole calls, fp32 matrix instructions at 75 to 80 % of their peak -> this kernel:
//   backward-data    3x3, 128 channels, 28x28: 498 -> 310 us;  1x1, 256 -> 64, 56x56: 297 -> 238 us;  1x1 stride 2, 1024 -> 512: 514 -> 346 us
//   filter gradient  the same layers: 489 -> 371, 264 -> 209, 423 -> 327 us
// Backward-data is bound by power (3x3: matrix pipe busy in 60 % of the cycles at 1.77 GHz), the filter gradient by the split's arithmetic, its scalar
// work per pixel and the chains of six products (44 % at 1.92 GHz).
//
// The split happens once per staged element, on the way from the load registers into LDS.
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <stdlib.h>
#include <type_traits>

#include "conv_common.h"

namespace {

// Two values at a time.  (v_dot2_f32_bf16 would take the widening and the subtraction in one instruction, but it runs on the matrix pipe's
// time: a loop of one MFMA and four of them takes 25 ns per MFMA, with subtractions 19.)
constexpr float kScale = 65536.f;
struct Split2 {
    unsigned h, m, l;
};
__device__ __forceinline__ Split2 split2(float x0, float x1, float scale) {      // kScale or -kScale, see sum_products()
    x0 *= scale;
    x1 *= scale;
    Split2 s;
    s.h = lc_bf16x2_rne(x0, x1);
    const float r0 = x0 - __uint_as_float(s.h << 16), r1 = x1 - __uint_as_float(s.h & 0xffff0000u);
    s.m = lc_bf16x2_rne(r0, r1);
    s.l = lc_bf16x2_rne(r0 - __uint_as_float(s.m << 16), r1 - __uint_as_float(s.m & 0xffff0000u));
    return s;
}

constexpr int BK = 32;                     // k-step: 128 bytes of a row, one v_mfma_f32_16x16x32_bf16 deep
constexpr int kBlock16 = 3072;             // LDS bytes of 16 rows x 32 k: three bf16 planes

// One k-step's products of N 16x16 tiles, t[n] = mfma(n, plane of the first operand, plane of the second, t[n]) from the smallest products up, in
// sums of their own; add_sums() adds them to the accumulators.  The matrix instruction rounds its sum to the accumulator's last bit after every
// eight terms, four times: that is 24 roundings a k-step with the six products straight into the accumulators (as many as 48 terms on the fp32
// instructions, which round every second term), and one this way.  Errors against 64 bits, fp32 instructions / straight / this way: 3x3 over
// 128 channels at 28x28, 256 images dx 5.9e-7 / 5.1e-7 / 1.2e-7, 32 images (where the fp32 kernel's sums are cut into parts) 3.0e-7 / 5.1e-7 / 1.2e-7.
// Time: backward-data 3 %, filter gradient 4 % more than straight.
// It also cuts addends far below the last bit downwards, always the same way; over a filter gradient's 25,000 steps that shows (1x1 at 56x56: error
// 1.1e-6, all of it mean, where fp32 instructions give 4.2e-7).  So every other k-step runs with the first operand negated: 1.7e-7.
template <int N, typename F>
__device__ __forceinline__ void sum_products(f32x4 (&t)[N], F&& mfma) {
    constexpr int kParts[6][2] = {{2, 0}, {0, 2}, {1, 1}, {1, 0}, {0, 1}, {0, 0}};
#pragma unroll
    for (int q = 0; q < 6; ++q)
#pragma unroll
        for (int n = 0; n < N; ++n) t[n] = mfma(n, kParts[q][0], kParts[q][1], q == 0 ? f32x4{0.f, 0.f, 0.f, 0.f} : t[n]);
}
__device__ __forceinline__ float turn_of(int k_step) { return (k_step & 1) ? -1.f : 1.f; }
// unscale: the k-step's turn over the scales of both operands
__device__ __forceinline__ void add_sums(f32x4& acc, const f32x4& t, float unscale) {
#pragma unroll
    for (int v = 0; v < 4; ++v) acc[v] = fmaf(t[v], unscale, acc[v]);
}

// Blocks per compute unit (LDS: 48 KB for the 128x128 tile).  The generic addressing needs more registers.
constexpr int split_blocks_per_cu(int bn, bool ut) { return ut && bn == 64 ? 3 : 2; }

// Persistent blocks, whole tiles first, then a stream-K range, loads one k-step ahead across tile boundaries, as in conv_igemm.hip.
// Waves are 2 x 2; a wave owns BM/2 x BN/2 as 16x16 tiles with the operands swapped (the filter is the MFMA's first operand), so that a
// lane holds four consecutive columns of one output pixel: acc[i][j] = pixel row i*16 + l%16, columns j*16 + 4*(l/16) .. +3.
//
// LDS (one stage): per 16 rows [plane h, m, l][k 0-7, 8-15, 16-23, 24-31][16 rows][8 bf16]; a fragment is 1 KB read in lane order.  Row r of
// k group g sits at r ^ 2g, which puts the 16 lanes that a store serves per cycle (two rows x eight 4-value pieces) on 128 distinct bytes.
//
// A block is in its matrix phase or in its split-and-store phase; the other block of the compute unit (of the narrow tile with uniform taps: the other
// two) fills the pipe meanwhile.
template <int BM, int BN, bool SMALLC, bool UT, bool SCATTER>
__global__ void __launch_bounds__(256, split_blocks_per_cu(BN, UT)) conv_gemm_split_kernel(const GemmConv p) {
    constexpr int WTM = BM / 2, WTN = BN / 2, TM = WTM / 16, TN = WTN / 16;
    constexpr int LA = BM / 32, LB = BN / 32, LPT = LA + LB;

    constexpr int kOutPitch = WTN + 4;                     // floats; 16 rows fall on distinct banks
    __shared__ __attribute__((aligned(1024))) unsigned char lds[(BM + BN) / 16 * kBlock16];
    __shared__ __attribute__((aligned(16))) uint2 row_lds[UT ? BM : 1];   // per tile row: byte offset of its pixel's window, taps outside the image
    static_assert(16 * kOutPitch * 4 * 4 <= sizeof(lds), "output staging");

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave >> 1, wn = wave & 1;
    const int nbn = (p.N + BN - 1) / BN;
    const int nkt = (p.Kg + BK - 1) / BK;
    const float* __restrict__ A = static_cast<const float*>(p.a);
    const float* __restrict__ B = static_cast<const float*>(p.b);
    const int lrow = lane >> 3, kq = lane & 7;            // a wave's load: 8 rows of 128 bytes
    const int Hi_ = p.Hi, Wi_ = p.Wi, Ci_ = p.Ci, R_ = p.R, S_ = p.S, M_ = p.M, N_ = p.N, Kg_ = p.Kg, ldd_ = p.ldd;
    const int sh_ = p.sh, sw_ = p.sw, ph_ = p.ph, pw_ = p.pw, Po_ = p.Po, Qo_ = p.Qo;
    const unsigned qmul = p.qo_mul, qsh = p.qo_shift, pmul = p.po_mul, psh = p.po_shift;
    const int frow = lane & 15, fgrp = lane >> 4;

    // ---- this block's segments: `rounds` whole tiles, then its stream-K range cut at the tile boundaries ----
    const SkWalk walk(p, nkt);
    const int F = walk.steps(), rounds = walk.rounds, bid = walk.bid;
    if (F == 0) return;
    auto segment = [&](int s, int& tile, int& k0, int& k1) __attribute__((always_inline)) { walk.segment(s, tile, k0, k1); };

    // ---------------- load side ----------------
    int l_seg = -1, l_k = 0, l_k1 = 0;                     // segment being loaded, next k-step, end
    // generic addressing (pointer per row, position in the window per lane)
    long long a_base[LA];
    int a_h[LA], a_w[LA];
    int l_n0 = 0, kg = 0, c = 0, r = 0, s = 0;
    // uniform-tap addressing: see conv_igemm.hip
    __amdgpu_buffer_rsrc_t a_rsrc = __builtin_amdgcn_make_buffer_rsrc((void*)A, 0, 0, (int)kBufferWords3);
    __amdgpu_buffer_rsrc_t b_rsrc = a_rsrc;
    int u_kt = 0, u_c = 0, u_s = 0, u_r = 0;
    const unsigned b_voff = (unsigned)((wave * 8 + lrow) * Kg_ * 4 + kq * 16);
    const int b_step = 32 * Kg_ * 4;                       // bytes between a thread's filter rows

    auto loader_setup = [&](int tile, int k0) __attribute__((always_inline)) {
        const int tm = tile / nbn;
        const int m0 = tm * BM, n0 = (tile - tm * nbn) * BN;
        if constexpr (UT) {
            const int pq = Po_ * Qo_;
            const int img0 = m0 / pq;
            const int phb = max(ph_, 0), pwb = max(pw_, 0);
            const WindowTaps window(R_, S_);
            if (lane < LA * 8) {                       // this wave's rows, one per lane; nobody else reads them
                const int row = ((lane >> 3) * 4 + wave) * 8 + (lane & 7), m = m0 + row;
                const int t = div_by(m, qmul, qsh), qo = m - t * Qo_;
                const int img = div_by(t, pmul, psh), po = t - img * Po_;
                const int h0 = po * sh_ - ph_, w0 = qo * sw_ - pw_;
                const unsigned inv = window.outside(h0, w0, Hi_, Wi_, R_, S_);
                const bool ok = (m < M_) & (inv != ~0u);
                row_lds[row] = make_uint2(ok ? (unsigned)(((((img - img0) * Hi_ + h0 + phb) * Wi_) + w0 + pwb) * Ci_ * 4) : 0u,
                                          ok ? inv : ~0u);
            }
            asm volatile("s_waitcnt lgkmcnt(0)" : : : "memory");
            const long long a_first = ((long long)img0 * Hi_ * Wi_ - ((long long)phb * Wi_ + pwb)) * Ci_;
            a_rsrc = __builtin_amdgcn_make_buffer_rsrc((void*)(A + a_first), 0, (int)kBufferBytes, (int)kBufferWords3);
            // filter rows past N lie past the end of the buffer
            const long long b_left = (long long)(N_ - n0) * Kg_ * 4;
            b_rsrc = __builtin_amdgcn_make_buffer_rsrc((void*)(B + (long long)n0 * Kg_), 0, (int)(b_left > 0x7fffffffLL ? 0x7fffffffLL : b_left),
                                                       (int)kBufferWords3);
            u_kt = k0;
            const int kg0 = k0 * BK, rs0 = kg0 / Ci_;
            u_c = kg0 - rs0 * Ci_;
            u_r = rs0 / S_;
            u_s = rs0 - u_r * S_;
        } else {
#pragma unroll
            for (int i = 0; i < LA; ++i) {
                const int m = m0 + (i * 4 + wave) * 8 + lrow;
                if (m < M_) {
                    const int t = div_by(m, qmul, qsh), qo = m - t * Qo_;
                    const int img = div_by(t, pmul, psh), po = t - img * Po_;
                    a_h[i] = po * sh_ - ph_;
                    a_w[i] = qo * sw_ - pw_;
                    a_base[i] = (long long)img * Hi_ * Wi_ * Ci_;
                } else {
                    a_h[i] = -(1 << 28);              // every tap fails the bounds test
                    a_w[i] = 0;
                    a_base[i] = 0;
                }
            }
            l_n0 = n0 + wave * 8 + lrow;
            kg = k0 * BK + kq * 4;
            const int rs = kg / Ci_;
            c = kg - rs * Ci_;
            r = rs / S_;
            s = rs - r * S_;
        }
    };

    float4 g[LPT];                                // the k-step in flight between global memory and LDS
    auto gload_tile = [&]() __attribute__((always_inline)) {
        if constexpr (UT) {
            const int tap = u_r * S_ + u_s;
            const unsigned up = 31u - (unsigned)tap;
            const int a_soff = ((u_r * Wi_ + u_s) * Ci_ + u_c) * 4;
            const int b_soff = u_kt * BK * 4;
#pragma unroll
            for (int l = 0; l < LA; ++l) {
                const uint2 row = row_lds[(l * 4 + wave) * 8 + lrow];
                const unsigned vo = ((row.y << up) & kBufferBytes) | (row.x + (unsigned)kq * 16u);
                g[l] = __builtin_bit_cast(float4, __builtin_amdgcn_raw_buffer_load_b128(a_rsrc, (int)vo, a_soff, 0));
            }
#pragma unroll
            for (int l = 0; l < LB; ++l)
                g[LA + l] = __builtin_bit_cast(float4, __builtin_amdgcn_raw_buffer_load_b128(b_rsrc, (int)b_voff, b_soff + l * b_step, 0));
            ++u_kt;
            u_c += BK;
            const bool wrap = u_c == Ci_;
            u_c = wrap ? 0 : u_c;
            u_s += wrap ? 1 : 0;
            const bool wrap2 = u_s == S_;
            u_s = wrap2 ? 0 : u_s;
            u_r += wrap2 ? 1 : 0;
        } else {
            const bool kok = r < R_;              // same as kg < Kg
#pragma unroll
            for (int l = 0; l < LA; ++l) {
                const int h = a_h[l] + r, w = a_w[l] + s;
                const bool ok = kok & ((unsigned)h < (unsigned)Hi_) & ((unsigned)w < (unsigned)Wi_);
                g[l] = load_global16(pick(ok, A + a_base[l] + ((long long)h * Wi_ + w) * Ci_ + c, g_zero_chunk));
            }
#pragma unroll
            for (int l = 0; l < LB; ++l)
                g[LA + l] = load_global16(pick(kok & (l_n0 + l * 32 < N_), B + (long long)(l_n0 + l * 32) * Kg_ + kg, g_zero_chunk));
            kg += BK;
            c += BK;
            if (SMALLC) {
                while (c >= Ci_) {
                    c -= Ci_;
                    if (++s == S_) {
                        s = 0;
                        ++r;
                    }
                }
            } else {
                const bool wrap = c >= Ci_;
                c = wrap ? c - Ci_ : c;
                s += wrap ? 1 : 0;
                const bool wrap2 = s == S_;
                s = wrap2 ? 0 : s;
                r += wrap2 ? 1 : 0;
            }
        }
    };
    // fetch the next k-step of the block's sequence (the caller knows there is one)
    auto load_step = [&]() __attribute__((always_inline)) {
        if (l_k == l_k1) {
            int tile;
            ++l_seg;
            segment(l_seg, tile, l_k, l_k1);
            loader_setup(tile, l_k);
        }
        gload_tile();
        ++l_k;
    };
    unsigned char* const st = lds + (wave >> 1) * kBlock16 + (kq >> 1) * 256 + ((((wave & 1) * 8 + lrow) ^ (kq & 6)) * 16) + (kq & 1) * 8;
    auto split_store = [&](float scale_a) __attribute__((always_inline)) {
#pragma unroll
        for (int l = 0; l < LPT; ++l) {
            const float scale = l < LA ? scale_a : kScale;
            const Split2 a = split2(g[l].x, g[l].y, scale), b = split2(g[l].z, g[l].w, scale);
            unsigned char* q = st + (l < LA ? l * 2 : BM / 16 + (l - LA) * 2) * kBlock16;
            *reinterpret_cast<uint2*>(q) = make_uint2(a.h, b.h);
            *reinterpret_cast<uint2*>(q + 1024) = make_uint2(a.m, b.m);
            *reinterpret_cast<uint2*>(q + 2048) = make_uint2(a.l, b.l);
        }
    };

    // ---------------- compute side ----------------
    f32x4 acc[TM][TN];
    const unsigned char* const fr = lds + fgrp * 256 + ((frow ^ (fgrp << 1)) * 16);
    auto frag = [&](int block, int plane) __attribute__((always_inline)) {
        return *reinterpret_cast<const bf16x8*>(fr + block * kBlock16 + plane * 1024);
    };
    // one k-step out of LDS: the filter's fragments are held, the activations' fetched one row of tiles ahead, and a row's sums are added between
    // the next row's matrix instructions (behind them: 3 % slower)
    auto matrix_phase = [&](float unscale) __attribute__((always_inline)) {
        bf16x8 fa[2][3], fb[3][TN];
        f32x4 t[2][TN];
#pragma unroll
        for (int pl = 0; pl < 3; ++pl)
#pragma unroll
            for (int j = 0; j < TN; ++j) fb[pl][j] = frag(BM / 16 + wn * TN + j, pl);
#pragma unroll
        for (int pl = 0; pl < 3; ++pl) fa[0][pl] = frag(wm * TM, pl);
#pragma unroll
        for (int i = 0; i <= TM; ++i) {
            if (i + 1 < TM) {
#pragma unroll
                for (int pl = 0; pl < 3; ++pl) fa[(i + 1) & 1][pl] = frag(wm * TM + i + 1, pl);
            }
            if (i < TM)
                sum_products(t[i & 1], [&](int j, int pa, int pb, f32x4 c) {
                    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[pb][j], fa[i & 1][pa], c, 0, 0, 0);
                });
            if (i > 0) {
#pragma unroll
                for (int j = 0; j < TN; ++j) add_sums(acc[i - 1][j], t[(i - 1) & 1][j], unscale);
            }
            if (i > 0 && i < TM) {
#pragma unroll
                for (int n = 0; n < 2 * TN; ++n) {
                    __builtin_amdgcn_sched_group_barrier(0x8 /* matrix */, 2, 0);
                    __builtin_amdgcn_sched_group_barrier(0x2 /* vector ALU */, 2, 0);
                }
            }
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    auto clear_acc = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    };
    // An infinity or a NaN does not survive the split (inf - inf), nor does a value past 2^112 or a product past 2^96 (the scale): this wave's part of
    // the segment [k0, k1) once more with fp32 matrix instructions straight from memory, where the split's result is not finite.  Every such
    // operand makes its whole row or column of the split's result NaN, so looking at the result finds them all; a sum that overflows by
    // itself comes here too and leaves as fp32 arithmetic has it.
    auto redo_not_finite = [&](int m0, int n0, int k0, int k1) __attribute__((always_inline)) {
        float t[TN];
#pragma unroll
        for (int j = 0; j < TN; ++j) t[j] = 0.f;
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int v = 0; v < 4; ++v)
#pragma unroll
                for (int j = 0; j < TN; ++j) t[j] = fmaf(acc[i][j][v], 0.f, t[j]);
#pragma unroll
        for (int j = 1; j < TN; ++j) t[0] += t[j];
        if (__builtin_expect(__ballot(t[0] != t[0]) == 0, 1)) return;
        clear_acc();
        for (int kk = k0 * BK + fgrp; kk < k1 * BK + fgrp; kk += 4) {
            const int rs = kk / Ci_, cc = kk - rs * Ci_, rr = rs / S_, ss = rs - rr * S_;
            float a[TM], b[TN];
#pragma unroll
            for (int i = 0; i < TM; ++i) {
                const int m = m0 + wm * WTM + i * 16 + frow;
                const int q = div_by(m, qmul, qsh), qo = m - q * Qo_;
                const int img = div_by(q, pmul, psh), po = q - img * Po_;
                const int h = po * sh_ - ph_ + rr, w = qo * sw_ - pw_ + ss;
                const bool ok = (m < M_) & (kk < Kg_) & ((unsigned)h < (unsigned)Hi_) & ((unsigned)w < (unsigned)Wi_);
                a[i] = *(const __attribute__((address_space(1))) float*)(uintptr_t)pick(
                    ok, A + (((long long)img * Hi_ + h) * Wi_ + w) * Ci_ + cc, g_zero_chunk);
            }
#pragma unroll
            for (int j = 0; j < TN; ++j) {
                const int n = n0 + wn * WTN + j * 16 + frow;
                b[j] = *(const __attribute__((address_space(1))) float*)(uintptr_t)pick((n < N_) & (kk < Kg_), B + (long long)n * Kg_ + kk,
                                                                                        g_zero_chunk);
            }
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(b[j], a[i], acc[i][j], 0, 0, 0);
        }
    };

    int c_seg = 0, c_tile, c_k0, c_k, c_k1;
    segment(0, c_tile, c_k0, c_k1);
    c_k = c_k0;
    // store (or park) the finished segment
    auto epilogue = [&]() __attribute__((always_inline)) {
        const int tm = c_tile / nbn;
        const int m0 = tm * BM, n0 = (c_tile - tm * nbn) * BN;
        redo_not_finite(m0, n0, c_k0, c_k1);
        if (!(c_k0 == 0 && c_k1 == nkt)) {
            // part of a tile: it is the first piece of this block's stream-K range (slot 2*bid) or the last (2*bid + 1)
            // (a buffer descriptor: 16 lane pointers would be computed ahead of the loop and cost 32 registers in it)
            const __amdgpu_buffer_rsrc_t part_rsrc = __builtin_amdgcn_make_buffer_rsrc(
                (void*)(p.partial + ((size_t)2 * bid + (c_seg == rounds ? 0 : 1)) * (BM * BN)), 0, BM * BN * 4, (int)kBufferWords3);
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j)
                    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, acc[i][j]), part_rsrc, lane * 16 + wave * 1024,
                                                           (i * TN + j) * 4096, 0);
            return;
        }
        // 16 rows at a time through the wave's own LDS slice, so that a store covers whole rows of the wave's part (4 x 256 or 8 x 128 bytes, in
        // lane order) and not 16 bytes of each of 16 rows per 16 lanes: 1x1 over 64 channels at 56x56, batch 256, 270 -> 245 us.
        // Rows past M: bit 31 of the lane offset; columns past N likewise, per group of four (value by value where N is not a multiple of
        // four).  Offsets count from the tile's first row (scatter: from its first pixel).
        long long base_px = m0;
        if constexpr (SCATTER) {
            const int t0 = div_by(m0, qmul, qsh), i0 = div_by(t0, pmul, psh);
            base_px = ((long long)i0 * p.Ho + (t0 - i0 * Po_) * p.esh) * p.Wo + (m0 - t0 * Qo_) * p.esw;
        }
        const __amdgpu_buffer_rsrc_t d_rsrc = __builtin_amdgcn_make_buffer_rsrc((void*)(static_cast<float*>(p.d) + base_px * ldd_), 0,
                                                                                (int)kBufferBytes, (int)kBufferWords3);
        const bool quads = (N_ & 3) == 0;
        constexpr int CPR = WTN / 4, RPI = 64 / CPR;           // lanes per row, rows per store
        const int lr = lane / CPR, col = n0 + wn * WTN + (lane % CPR) * 4;
        float* const mine = reinterpret_cast<float*>(lds) + wave * (16 * kOutPitch);     // every wave has read its last fragments of the tile
        // (the policy of the stores is the whole epilogue's: store by store chosen, 256 to 64 1x1 over 32 images of 56x56 took 36.2 us for
        // 34.3, 512 to 128 over 256 of 28x28 189 for 184, and 24 to 96 3x3 with stride 2 over 289 of 8x8 53.7 for 52.7.  Past the caches go whole lines, so
        // whole groups of four.)
        auto leave = [&](auto past) __attribute__((always_inline)) {
            constexpr bool kPast = decltype(past)::value;
#pragma unroll
            for (int i = 0; i < TM; ++i) {
#pragma unroll
                for (int j = 0; j < TN; ++j) *reinterpret_cast<f32x4*>(mine + frow * kOutPitch + j * 16 + 4 * fgrp) = acc[i][j];
                asm volatile("s_waitcnt lgkmcnt(0)" : : : "memory");
                f32x4 out[16 / RPI];
#pragma unroll
                for (int e = 0; e < 16 / RPI; ++e) out[e] = *reinterpret_cast<const f32x4*>(mine + (e * RPI + lr) * kOutPitch + (lane % CPR) * 4);
                asm volatile("s_waitcnt lgkmcnt(0)" : : : "memory");
#pragma unroll
                for (int e = 0; e < 16 / RPI; ++e) {
                    const int m = m0 + wm * WTM + i * 16 + e * RPI + lr;
                    int px;
                    if constexpr (SCATTER) {
                        const int t = div_by(m, qmul, qsh), img = div_by(t, pmul, psh);
                        px = (int)(((long long)img * p.Ho + (t - img * Po_) * p.esh) * p.Wo + (m - t * Qo_) * p.esw - base_px);
                    } else {
                        px = m - m0;
                    }
                    const unsigned off = m < M_ ? (unsigned)(px * ldd_ + col) * 4u : kBufferBytes;
                    if (kPast || quads) {
                        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, out[e]), d_rsrc, (int)(col < N_ ? off : kBufferBytes), 0, kPast ? kNonTemporal : 0);
                    } else {
#pragma unroll
                        for (int v = 0; v < 4; ++v)
                            __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(out[e][v]), d_rsrc, (int)(col + v < N_ ? off : kBufferBytes), v * 4, 0);
                    }
                }
            }
        };
        if (__builtin_expect(p.stream_d, 0)) leave(std::true_type{});
        else leave(std::false_type{});
    };

    // ---------------- the pipeline ----------------
    load_step();                                  // k-step 0 of the sequence
    clear_acc();
    for (int f = 0; f < F; ++f) {
        const float turn = turn_of(c_k);
        split_store(turn * kScale);
        if (f + 1 < F) load_step();               // stays in flight over the matrix phase
        lds_barrier();
        __builtin_amdgcn_s_setprio(1);
        matrix_phase(turn / (kScale * kScale));
        __builtin_amdgcn_s_setprio(0);
        lds_barrier();                            // every wave has read its last fragments
        if (++c_k == c_k1) {                      // the segment is complete: store it, the next step starts a new one
            epilogue();
            lds_barrier();                        // the staging of the result is over before the next step is stored
            clear_acc();
            ++c_seg;
            segment(c_seg, c_tile, c_k0, c_k1);
            c_k = c_k0;
        }
    }
}

// Adds the parts of every tile that stream-K blocks split between them, in k order, and stores the tile: block (t, y) handles the 16x16
// tile y of each of the four waves of stream-K tile t.  Eight parts are fetched at a time.
template <int BM, int BN, bool MEET>
__global__ void __launch_bounds__(256) conv_split_fixup_kernel(const GemmConv p) {
    constexpr int TN = BN / 32;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int nbn = (p.N + BN - 1) / BN;
    const int nkt = (p.Kg + BK - 1) / BK;
    int sk_tile, j, j1;
    if (!sk_shared_tile<MEET>(p, nkt, blockIdx.x, &sk_tile, &j, &j1)) return;  // one block did the whole tile and stored it
    const int tb = sk_tile * nkt;                                        // this tile's first k-step in stream-K positions
    const f32x4* part = reinterpret_cast<const f32x4*>(p.partial) + (blockIdx.y * 4 + wave) * 64 + lane;
    constexpr size_t kSlot = BM * BN / 4;
    // the first block's piece is the last of its range unless its range starts here; all others start their ranges in this tile
    f32x4 sum = part[((size_t)2 * j + (sk_begin(p, j) >= tb ? 0 : 1)) * kSlot];
    for (++j; j < j1; j += 8) {
        f32x4 v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u)
            if (j + u < j1) v[u] = part[(size_t)2 * (j + u) * kSlot];
#pragma unroll
        for (int u = 0; u < 8; ++u)
            if (j + u < j1) sum += v[u];
    }
    const int tile = p.dp_tiles + sk_tile, tm = tile / nbn;
    const int ti = blockIdx.y / TN, tj = blockIdx.y - ti * TN;
    const int m = tm * BM + (wave >> 1) * (BM / 2) + ti * 16 + (lane & 15);
    const int col = (tile - tm * nbn) * BN + (wave & 1) * (BN / 2) + tj * 16 + 4 * (lane >> 4);
    if (m >= p.M || col >= p.N) return;
    long long px = m;
    if (p.scatter) {
        const int qo = m % p.Qo, t = m / p.Qo;
        const int po = t % p.Po, img = t / p.Po;
        px = ((long long)img * p.Ho + (long long)po * p.esh) * p.Wo + (long long)qo * p.esw;
    }
    float* d = static_cast<float*>(p.d) + px * p.ldd + col;
    if ((p.N & 3) == 0 && (p.ldd & 3) == 0 && aligned16(p.d)) {
        *reinterpret_cast<f32x4*>(d) = sum;
    } else {
#pragma unroll
        for (int v = 0; v < 4; ++v)
            if (col + v < p.N) d[v] = sum[v];
    }
}

// ------------------------------------------------------------------------------------------------
// Backward-weight: D[k][j] = sum_m dY[m][k] * X(m, j), j = (r, s, c), the same split arithmetic.  The reduction index is the strided one of
// both operands, and an MFMA wants eight consecutive reduction values of one column from a lane: a wave owns eight of a step's 32 rows, a lane
// loads its one or two columns of all eight (one row per load instruction), and the packing of value pairs into bf16 pairs along the
// rows is the transposition -- each column's eight values leave as one 16-byte LDS store per plane.
//
// LDS: per 16 columns [plane][row group of 8][16 columns][8 rows]; with two columns per lane a block holds the even columns first, then the odd
// ones, so that eight lanes store 128 consecutive bytes; the epilogue undoes that.
// A load covers one output pixel, so its byte offset and the set of its taps inside the image are wave-uniform; a lane holds its column's tap offset and bit, and
// a tap outside the image moves its offset past the end of the buffer.  Offsets and sets are worked out for the wave's rows of eight steps at once, a row per
// lane, and read lane by lane.  (Row by row on the scalar unit a step's loads took 2.3 us to issue, half of a step where a block has its compute unit to itself, and three
// blocks did not hide it.  us, before / now: 3x3 over 128 channels, 256 images of 28x28 401 / 353, over 256, 256 of 14x14 409 / 343, 32 images 75 / 66, two images 27 / 22; over 64, 32 of
// 56x56 95 / 73; 1x1 stride 2 512 to 1024, 32 of 28x28 71 / 63.)
// PLAIN: a 1x1 window with stride 1 and no padding -- pixel m reads pixel m.
// Three 128x128 blocks per compute unit (168 registers, 48 KB of LDS): 364 us with two of them on the 3x3 layer above, 320 with three.
// ------------------------------------------------------------------------------------------------
constexpr int wgrad_split_blocks_per_cu(int bm, int bn) { return bm == 128 && bn == 128 ? 3 : bm == 64 && bn == 64 ? 5 : 4; }

template <int V> struct RowVec;
template <> struct RowVec<1> { using type = float; };
template <> struct RowVec<2> { using type = float2; };

template <int BM, int BN, bool PLAIN>
__global__ void __launch_bounds__(256, wgrad_split_blocks_per_cu(BM, BN)) wgrad_split_kernel(const GemmWgrad p) {
    constexpr int VA = BM / 64, VB = BN / 64;              // columns per lane
    constexpr int TM = BM / 32, TN = BN / 32;              // 16x16 tiles per wave (2 x 2 waves)

    __shared__ __attribute__((aligned(1024))) unsigned char lds[(BM + BN) / 16 * kBlock16];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave >> 1, wn = wave & 1;
    const int nbn = (p.J + BN - 1) / BN;
    // split-major, dealt to the XCDs in contiguous runs: the tiles of a split read the same rows and share one L2
    const int tiles_ = ((p.K + BM - 1) / BM) * nbn;
    const int work = xcd_tile(blockIdx.x, tiles_ * p.splits);
    const int z = work / tiles_, tile = work - z * tiles_;
    const int k0 = (tile / nbn) * BM, j0 = (tile % nbn) * BN;
    const int m_begin = z * p.m_per_split;
    const int m_end = min(p.M, m_begin + p.m_per_split);
    const int H_ = p.H, W_ = p.W, C_ = p.C, P_ = p.P, Q_ = p.Q, R_ = p.R, S_ = p.S, K_ = p.K, J_ = p.J;
    const int sh_ = p.sh, sw_ = p.sw, ph_ = p.ph, pw_ = p.pw;
    const int frow = lane & 15, fgrp = lane >> 4;

    // dY: rows past the end of the split lie past the end of the buffer
    const int a_col = k0 + lane * VA;
    const unsigned a_voff = a_col < K_ ? (unsigned)a_col * 4u : kBufferBytes;
    const __amdgpu_buffer_rsrc_t a_rsrc = __builtin_amdgcn_make_buffer_rsrc(
        (void*)(static_cast<const float*>(p.dy) + (long long)m_begin * K_), 0, (int)((unsigned)(m_end - m_begin) * (unsigned)K_ * 4u),
        (int)kBufferWords3);
    // X: the lane's column j = (r, s, c): byte offset of the tap relative to the pixel's window origin, bit position
    const int b_col = j0 + lane * VB;
    unsigned b_voff = kBufferBytes, b_up = 0;
    if (b_col < J_) {
        const int rs = b_col / C_, fc = b_col - rs * C_;
        const int fr = rs / S_, fs = rs - fr * S_;
        b_voff = PLAIN ? (unsigned)b_col * 4u : (unsigned)(((fr * W_ + fs) * C_ + fc) * 4);
        b_up = 31u - (unsigned)rs;
    }
    const int img_first = m_begin / (P_ * Q_);
    const int phb = max(ph_, 0), pwb = max(pw_, 0);
    const float* const X = static_cast<const float*>(p.x);
    const __amdgpu_buffer_rsrc_t b_rsrc =
        PLAIN ? __builtin_amdgcn_make_buffer_rsrc((void*)(X + (long long)m_begin * C_), 0, (int)((unsigned)(m_end - m_begin) * (unsigned)C_ * 4u),
                                                  (int)kBufferWords3)
              : __builtin_amdgcn_make_buffer_rsrc((void*)(X + ((long long)img_first * H_ * W_ - ((long long)phb * W_ + pwb)) * C_), 0,
                                                  (int)kBufferBytes, (int)kBufferWords3);
    int mt = m_begin + wave * 8;                           // this wave's first row of the step being loaded
    const WindowTaps window(R_, S_);
    // pixel offset and taps outside the image of row lane % 8 of step lane / 8 of the eight steps from pix_step on
    int pix_off = 0, pix_step = 8;
    unsigned pix_inv = 0;
    auto pixels_of_steps = [&]() __attribute__((always_inline)) {
        const int m = mt + (lane >> 3) * BK + (lane & 7);
        const int t = div_by(m, p.q_mul, p.q_shift), q = m - t * Q_;
        const int im = div_by(t, p.p_mul, p.p_shift), pp = t - im * P_;
        const int h0 = pp * sh_ - ph_, w0 = q * sw_ - pw_;
        const unsigned inv = window.outside(h0, w0, H_, W_, R_, S_);
        const bool ok = ((unsigned)m < (unsigned)m_end) & (inv != ~0u);      // (m may lie past 2^31)
        pix_inv = ok ? inv : ~0u;
        pix_off = ok ? (((im - img_first) * H_ + h0 + phb) * W_ + w0 + pwb) * C_ * 4 : 0;
        pix_step = 0;
    };

    typename RowVec<VA>::type ga[8];
    typename RowVec<VB>::type gb[8];
    auto load_row = [&](auto& dst, const __amdgpu_buffer_rsrc_t& rsrc, unsigned vo, int so) __attribute__((always_inline)) {
        if constexpr (sizeof(dst) == 8)
            dst = __builtin_bit_cast(float2, __builtin_amdgcn_raw_buffer_load_b64(rsrc, (int)vo, so, 0));
        else
            dst = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rsrc, (int)vo, so, 0));
    };
    auto load_step = [&]() __attribute__((always_inline)) {
        const int row0 = mt - m_begin;
#pragma unroll
        for (int i = 0; i < 8; ++i) load_row(ga[i], a_rsrc, a_voff, (row0 + i) * K_ * 4);
        if constexpr (PLAIN) {
#pragma unroll
            for (int i = 0; i < 8; ++i) load_row(gb[i], b_rsrc, b_voff, (row0 + i) * C_ * 4);
        } else {
            if (pix_step == 8) pixels_of_steps();
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const unsigned inv = (unsigned)__builtin_amdgcn_readlane((int)pix_inv, pix_step * 8 + i);
                load_row(gb[i], b_rsrc, ((inv << b_up) & kBufferBytes) | b_voff, __builtin_amdgcn_readlane(pix_off, pix_step * 8 + i));
            }
            ++pix_step;
        }
        mt += BK;
    };
    // one operand's columns of this lane: eight rows each, three planes
    auto split_store_cols = [&](auto& g, unsigned char* base, float scale) __attribute__((always_inline)) {
        constexpr int V = sizeof(g[0]) / 4;
#pragma unroll
        for (int e = 0; e < V; ++e) {
            Split2 s[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                if constexpr (V == 2) s[u] = e == 0 ? split2(g[2 * u].x, g[2 * u + 1].x, scale) : split2(g[2 * u].y, g[2 * u + 1].y, scale);
                else s[u] = split2(g[2 * u], g[2 * u + 1], scale);
            }
            unsigned char* q = base + (V == 2 ? (lane >> 3) * kBlock16 + ((lane & 7) + 8 * e) * 16 : (lane >> 4) * kBlock16 + (lane & 15) * 16) + wave * 256;
            *reinterpret_cast<u32x4*>(q) = u32x4{s[0].h, s[1].h, s[2].h, s[3].h};
            *reinterpret_cast<u32x4*>(q + 1024) = u32x4{s[0].m, s[1].m, s[2].m, s[3].m};
            *reinterpret_cast<u32x4*>(q + 2048) = u32x4{s[0].l, s[1].l, s[2].l, s[3].l};
        }
    };

    f32x4 acc[TM][TN];
    const unsigned char* const fr = lds + fgrp * 256 + frow * 16;
    auto frag = [&](int block, int plane) __attribute__((always_inline)) {
        return *reinterpret_cast<const bf16x8*>(fr + block * kBlock16 + plane * 1024);
    };
    // one k-step out of LDS, in blocks of 2 x 2 tiles -- four sums in flight with 64 registers for fragments and sums, which leaves room for three
    // blocks per compute unit; neighbouring blocks keep one operand's fragments
    auto matrix_phase = [&](float unscale) __attribute__((always_inline)) {
        bf16x8 fa[3][2], fb[3][2];
        auto read_a = [&](int i0) __attribute__((always_inline)) {
#pragma unroll
            for (int pl = 0; pl < 3; ++pl)
#pragma unroll
                for (int i = 0; i < 2; ++i) fa[pl][i] = frag(wm * TM + i0 + i, pl);
        };
        auto read_b = [&](int j0) __attribute__((always_inline)) {
#pragma unroll
            for (int pl = 0; pl < 3; ++pl)
#pragma unroll
                for (int j = 0; j < 2; ++j) fb[pl][j] = frag(BM / 16 + wn * TN + j0 + j, pl);
        };
        read_b(0);
#pragma unroll
        for (int i0 = 0; i0 < TM; i0 += 2) {
            read_a(i0);
#pragma unroll
            for (int jj = 0; jj < TN; jj += 2) {
                const int j0 = (i0 & 2) ? TN - 2 - jj : jj;
                if (jj > 0) read_b(j0);
                f32x4 t[4];
                sum_products(t, [&](int n, int pa, int pb, f32x4 c) {
                    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa[pa][n >> 1], fb[pb][n & 1], c, 0, 0, 0);
                });
#pragma unroll
                for (int n = 0; n < 4; ++n) add_sums(acc[i0 + (n >> 1)][j0 + (n & 1)], t[n], unscale);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    };
    auto clear_acc = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    };
    // columns of a 16-block in the order the LDS blocks hold them
    auto col_of = [](int v, int r) __attribute__((always_inline)) { return v == 2 ? (r < 8 ? 2 * r : 2 * r - 15) : r; };

    clear_acc();
    const int nkt = (m_end - m_begin + BK - 1) / BK;
    if (nkt > 0) load_step();
    for (int kt = 0; kt < nkt; ++kt) {
        const float turn = turn_of(kt);
        split_store_cols(ga, lds, turn * kScale);
        split_store_cols(gb, lds + BM / 16 * kBlock16, kScale);
        if (kt + 1 < nkt) load_step();                // stays in flight over the matrix phase
        lds_barrier();
        __builtin_amdgcn_s_setprio(1);
        matrix_phase(turn / (kScale * kScale));
        __builtin_amdgcn_s_setprio(0);
        lds_barrier();                                // every wave has read its last fragments
    }

    // (the lane's place once more from a value that the loop does not know: five registers less in it)
    int late = tid;
    asm("" : "+v"(late));
    const int row_l = late & 15, grp_l = (late & 63) >> 4;
    // operands that the split cannot carry (see redo_not_finite above): this wave's part once more with fp32 matrix instructions
    {
        float t[TN];
#pragma unroll
        for (int j = 0; j < TN; ++j) t[j] = 0.f;
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int v = 0; v < 4; ++v)
#pragma unroll
                for (int j = 0; j < TN; ++j) t[j] = fmaf(acc[i][j][v], 0.f, t[j]);
#pragma unroll
        for (int j = 1; j < TN; ++j) t[0] += t[j];
        if (__builtin_expect(__ballot(t[0] != t[0]) != 0, 0)) {
            clear_acc();
            const float* const DY = static_cast<const float*>(p.dy);
            for (int m = m_begin + grp_l; m < m_end + grp_l; m += 4) {
                const int q = m / Q_, qo = m - q * Q_, img = q / P_, po = q - img * P_;
                float a[TM], b[TN];
#pragma unroll
                for (int i = 0; i < TM; ++i) {
                    const int k = k0 + (wm * TM + i) * 16 + col_of(VA, row_l);
                    a[i] = *(const __attribute__((address_space(1))) float*)(uintptr_t)pick((m < m_end) & (k < K_), DY + (long long)m * K_ + k,
                                                                                            g_zero_chunk);
                }
#pragma unroll
                for (int j = 0; j < TN; ++j) {
                    const int jj = j0 + (wn * TN + j) * 16 + col_of(VB, row_l);
                    const int rs = jj / C_, fc = jj - rs * C_, fr_ = rs / S_, fs = rs - fr_ * S_;
                    const int h = po * sh_ - ph_ + fr_, w = qo * sw_ - pw_ + fs;
                    const bool ok = (m < m_end) & (jj < J_) & ((unsigned)h < (unsigned)H_) & ((unsigned)w < (unsigned)W_);
                    b[j] = *(const __attribute__((address_space(1))) float*)(uintptr_t)pick(
                        ok, X + (((long long)img * H_ + h) * W_ + w) * C_ + fc, g_zero_chunk);
                }
#pragma unroll
                for (int i = 0; i < TM; ++i)
#pragma unroll
                    for (int j = 0; j < TN; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[i], b[j], acc[i][j], 0, 0, 0);
            }
        }
    }
    float* __restrict__ D = p.d + (long long)z * K_ * J_;
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int k = k0 + (wm * TM + i) * 16 + col_of(VA, 4 * grp_l + v);
            if (k >= K_) continue;
#pragma unroll
            for (int j = 0; j < TN; ++j) {
                const int jj = j0 + (wn * TN + j) * 16 + col_of(VB, row_l);
                if (jj < J_) D[(long long)k * J_ + jj] = acc[i][j][v];
            }
        }
}

template <int BM, int BN>
lc_status launch_wgrad_split(const GemmWgrad& q, hipStream_t stream) {
    GemmWgrad p = q;
    magic_for(p.Q, &p.q_mul, &p.q_shift);
    magic_for(p.P, &p.p_mul, &p.p_shift);
    const long long tiles = (long long)((p.K + BM - 1) / BM) * ((p.J + BN - 1) / BN);
    if (tiles <= 0 || tiles * p.splits > 0x7fffffffLL) return LC_ERR_UNSUPPORTED;
    const bool plain = p.R == 1 && p.S == 1 && p.sh == 1 && p.sw == 1 && p.ph == 0 && p.pw == 0 && p.H == p.P && p.W == p.Q;
    if (plain) hipLaunchKernelGGL((wgrad_split_kernel<BM, BN, true>), dim3((unsigned)(tiles * p.splits)), dim3(256), 0, stream, p);
    else hipLaunchKernelGGL((wgrad_split_kernel<BM, BN, false>), dim3((unsigned)(tiles * p.splits)), dim3(256), 0, stream, p);
    return lc_end_call();
}

// Whether the uniform-tap variant takes this problem: k-steps that do not straddle taps, a tap mask that fits 32 bits, and tile-relative
// byte offsets (the images a tile can touch plus one filter window, and the tile's filter rows) that stay below 2^31.
bool split_uniform_tap(const GemmConv& p) {
    static const bool off = getenv("LARSCONV_NO_UNIFORM_TAP") != nullptr;     // comparison runs
    if (off || p.Ci % BK != 0 || (long long)p.R * p.S > 32) return false;
    const long long pq = (long long)p.Po * p.Qo;
    const long long images = 128 / pq + 2;
    const long long a_span = ((images * p.Hi + (p.ph > 0 ? p.ph : 0) + p.R + 1) * p.Wi + p.S + 1) * p.Ci * 4;
    return a_span < 0x7fff0000LL && 129LL * p.Kg * 4 < 0x7fff0000LL;
}

struct SplitPlan {
    bool ut;
    int bn, resident, nkt;
    long long tiles;
    SkPlan sk;
};

// Rows: 128; columns 64 for narrow results, otherwise 128.
bool split_plan(const GemmConv& p, SplitPlan* s) {
    s->ut = split_uniform_tap(p);
    s->bn = p.N <= 64 ? 64 : 128;
    s->resident = split_blocks_per_cu(s->bn, s->ut) * device_cu_count();
    s->tiles = (long long)((p.M + 127) / 128) * ((p.N + s->bn - 1) / s->bn);
    s->nkt = (p.Kg + BK - 1) / BK;
    if (s->tiles <= 0 || s->tiles * s->nkt >= 0x7fffffffLL) return false;
    // (the k-step costs are fitted to these kernels' own times, every form of the split over 190 drawn layers of 1 to 512 images: the form chosen is 0.6 to
    // 0.8 % off the best one in the mean, 11 % at most; with 1.2 / 1.2 and 0.7 / 0.6 2 to 3 % and 37 %)
    s->sk = sk_plan_by_cost(s->tiles, s->nkt, s->resident, s->bn == 128 ? StepCost{1.6, 1.0, 1.0, 4} : StepCost{1.3, 0.5, 0.5, 4});
    return true;
}

template <int BN, bool SMALLC, bool UT, bool SCATTER>
void launch_split(const GemmConv& p, unsigned grid, hipStream_t stream) {
    hipLaunchKernelGGL((conv_gemm_split_kernel<128, BN, SMALLC, UT, SCATTER>), dim3(grid), dim3(256), 0, stream, p);
}

template <int BN>
lc_status launch_split_tile(const GemmConv& p, const SplitPlan& s, bool whole, unsigned grid, hipStream_t stream) {
    if (s.ut) {
        if (p.scatter) launch_split<BN, false, true, true>(p, grid, stream);
        else launch_split<BN, false, true, false>(p, grid, stream);
    } else if (p.Ci >= BK) {
        if (p.scatter) launch_split<BN, false, false, true>(p, grid, stream);
        else launch_split<BN, false, false, false>(p, grid, stream);
    } else {
        if (p.scatter) launch_split<BN, true, false, true>(p, grid, stream);
        else launch_split<BN, true, false, false>(p, grid, stream);
    }
    if (!whole) {
        if (!sk_ranges_meet(p, s.nkt))
            hipLaunchKernelGGL((conv_split_fixup_kernel<128, BN, false>), dim3((unsigned)(s.tiles - p.dp_tiles), 16 * BN / 128), dim3(256), 0, stream, p);
        else if (p.sk_blocks > 1)
            hipLaunchKernelGGL((conv_split_fixup_kernel<128, BN, true>), dim3((unsigned)p.sk_blocks - 1, 16 * BN / 128), dim3(256), 0, stream, p);
    }
    return lc_end_call();
}

}  // namespace

size_t lc_conv_split_workspace(const GemmConv& p) {
    SplitPlan s;
    if (!split_plan(p, &s) || s.sk.sk_iters == (long long)s.sk.sk_blocks * s.nkt) return 0;      // (no tile is shared)
    return (size_t)2 * s.sk.sk_blocks * 128 * s.bn * sizeof(float);
}

lc_status lc_launch_conv_split(GemmConv p, hipStream_t stream) {
    SplitPlan s;
    if (!split_plan(p, &s)) return LC_ERR_UNSUPPORTED;
    if (p.stats) return LC_ERR_UNSUPPORTED;
    if (p.scatter) {                          // the scatter epilogue addresses the result relative to the tile's first pixel
        const long long span = (128LL / ((long long)p.Po * p.Qo) + 2) * p.Ho * p.Wo * p.ldd * 4;
        if (span >= 0x7fff0000LL) return LC_ERR_UNSUPPORTED;
    }
    // one round of resident blocks, each taking dp_tiles / grid whole tiles and then its stream-K range; without a workspace for partial
    // tiles the ranges are whole tiles
    if (s.sk.sk_blocks > 0 && !p.partial) s.sk.sk_blocks = 0;
    if (s.sk.sk_blocks == 0) {
        const long long rest = s.tiles % s.resident;
        s.sk.dp_tiles = (int)(s.tiles - rest);
        s.sk.sk_blocks = (int)rest;
        s.sk.sk_iters = rest * s.nkt;
    }
    p.dp_tiles = s.sk.dp_tiles;
    p.sk_blocks = s.sk.sk_blocks;
    p.sk_iters = s.sk.sk_iters;
    sk_constants(&p);
    magic_for(p.Qo, &p.qo_mul, &p.qo_shift);
    magic_for(p.Po, &p.po_mul, &p.po_shift);
    const unsigned grid = p.dp_tiles > 0 ? (unsigned)s.resident : (unsigned)p.sk_blocks;
    const bool whole = p.sk_blocks == 0 || p.sk_iters == (long long)p.sk_blocks * s.nkt;
    return s.bn == 128 ? launch_split_tile<128>(p, s, whole, grid, stream) : launch_split_tile<64>(p, s, whole, grid, stream);
}

int lc_wgrad_split_blocks_per_cu(int bm, int bn) { return wgrad_split_blocks_per_cu(bm, bn); }

lc_status lc_launch_wgrad_split(const GemmWgrad& p, int bm, int bn, hipStream_t stream) {
    if (bm == 128) return bn == 128 ? launch_wgrad_split<128, 128>(p, stream) : launch_wgrad_split<128, 64>(p, stream);
    return bn == 128 ? launch_wgrad_split<64, 128>(p, stream) : launch_wgrad_split<64, 64>(p, stream);
}
