// fp32 forward / backward-data on the bf16 matrix pipe of gfx950: D[m][n] = sum_kg A(m, kg) * B[n][kg], the implicit GEMM of
// conv_igemm.hip, with every fp32 operand taken apart into three bf16 values.
//
// x = h + m + l with h = x rounded to bf16, m = (x - h) rounded to bf16, l the rest: 8 + 8 + 8 significant bits, exact.  Of the nine partial
// products of a * b the six hh, hm, mh, mm, hl, lh reach the last bit of an fp32 product (the three left out are below 2^-25 of it); each is
// exact in the matrix pipe and is added to the fp32 accumulator there.  Six v_mfma_f32_16x16x32_bf16 take 96 cycles where the same
// sums cost v_mfma_f32_32x32x2_f32 256.  The error against 64-bit sums is the fp32 kernel's or smaller (one rounding per 32 terms and
// product instead of one per two terms): 3x3 over 128 channels 5.2e-7 against 5.9e-7 of the result's norm, 1x1 over 64 channels 1.0e-7 both.
//
// The split happens once per staged element, on the way from the load registers into LDS.
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <stdlib.h>

#include "conv_common.h"

namespace {

// Two values at a time.  (v_dot2_f32_bf16 would take the widening and the subtraction in one instruction, but it runs on the matrix pipe's
// time: a loop of one MFMA and four of them takes 25 ns per MFMA, with subtractions 19.)
struct Split2 {
    unsigned h, m, l;
};
__device__ __forceinline__ Split2 split2(float x0, float x1) {
    Split2 s;
    s.h = lc_bf16x2_rne(x0, x1);
    const float r0 = x0 - __uint_as_float(s.h << 16), r1 = x1 - __uint_as_float(s.h & 0xffff0000u);
    s.m = lc_bf16x2_rne(r0, r1);
    s.l = lc_bf16x2_rne(r0 - __uint_as_float(s.m << 16), r1 - __uint_as_float(s.m & 0xffff0000u));
    return s;
}

constexpr int BK = 32;                     // k-step: 128 bytes of a row, one v_mfma_f32_16x16x32_bf16 deep
constexpr int kBlock16 = 3072;             // LDS bytes of 16 rows x 32 k: three bf16 planes

// Blocks per compute unit (LDS: 48 KB for the 128x128 tile).  The generic addressing needs more registers.
constexpr int split_blocks_per_cu(int bn, bool ut) { return ut && bn == 64 ? 3 : 2; }

// Persistent blocks, whole tiles first, then a stream-K range, loads one k-step ahead across tile boundaries, as in conv_igemm.hip.
// Waves are 2 x 2; a wave owns BM/2 x BN/2 as 16x16 tiles with the operands swapped (the filter is the MFMA's first operand), so that a
// lane holds four consecutive columns of one output pixel: acc[i][j] = pixel row i*16 + l%16, columns j*16 + 4*(l/16) .. +3.
//
// LDS (one stage): per 16 rows [plane h, m, l][k 0-7, 8-15, 16-23, 24-31][16 rows][8 bf16]; a fragment is 1 KB read in lane order.  Row r of
// k group g sits at r ^ 2g, which puts the 16 lanes that a store serves per cycle (two rows x eight 4-value pieces) on 128 distinct bytes.
//
// A block is in its matrix phase or in its split-and-store phase; the other two blocks of the compute unit fill the pipe meanwhile.
template <int BM, int BN, bool SMALLC, bool UT, bool SCATTER>
__global__ void __launch_bounds__(256, split_blocks_per_cu(BN, UT)) conv_gemm_split_kernel(const GemmConv p) {
    constexpr int WTM = BM / 2, WTN = BN / 2, TM = WTM / 16, TN = WTN / 16;
    constexpr int LA = BM / 32, LB = BN / 32, LPT = LA + LB;

    constexpr int kOutPitch = WTN + 4;                     // floats; 16 rows fall on distinct banks
    __shared__ __attribute__((aligned(1024))) unsigned char lds[(BM + BN) / 16 * kBlock16];
    __shared__ __attribute__((aligned(16))) float out_lds[4 * 16 * kOutPitch];

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
    const int G = gridDim.x, bid = blockIdx.x;
    const int rounds = p.dp_tiles / G;                     // the launcher makes dp_tiles a multiple of the grid
    int sk_it = 0, sk_len = 0;
    if (bid < p.sk_blocks) {
        sk_it = (int)((long long)bid * p.sk_iters / p.sk_blocks);
        sk_len = (int)((long long)(bid + 1) * p.sk_iters / p.sk_blocks) - sk_it;
    }
    const int sk_tile = sk_it / nkt, sk_k0 = sk_it - sk_tile * nkt;
    const int F = rounds * nkt + sk_len;                   // k-steps this block runs
    if (F == 0) return;
    auto segment = [&](int s, int& tile, int& k0, int& k1) __attribute__((always_inline)) {
        if (s < rounds) {
            tile = xcd_tile(s * G + bid, p.dp_tiles);
            k0 = 0;
            k1 = nkt;
        } else {                                           // piece s - rounds of the stream-K range
            const int t = sk_tile + (s - rounds);
            tile = p.dp_tiles + t;
            k0 = s == rounds ? sk_k0 : 0;
            k1 = min(nkt, sk_it + sk_len - t * nkt);
        }
    };

    // ---------------- load side ----------------
    int l_seg = -1, l_k = 0, l_k1 = 0;                     // segment being loaded, next k-step, end
    // generic addressing (pointer per row, position in the window per lane)
    long long a_base[LA];
    int a_h[LA], a_w[LA];
    int l_n0 = 0, kg = 0, c = 0, r = 0, s = 0;
    // uniform-tap addressing: see conv_igemm.hip
    unsigned a_voff[LA], a_inv[LA];
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
            const int taps = R_ * S_;
            const unsigned full = taps >= 32 ? ~0u : (1u << taps) - 1u;
            unsigned rep = 0;
            for (int rr = 0; rr < R_; ++rr) rep |= 1u << (rr * S_);
#pragma unroll
            for (int i = 0; i < LA; ++i) {
                const int m = m0 + (i * 4 + wave) * 8 + lrow;
                const int t = div_by(m, qmul, qsh), qo = m - t * Qo_;
                const int img = div_by(t, pmul, psh), po = t - img * Po_;
                const int h0 = po * sh_ - ph_, w0 = qo * sw_ - pw_;
                // taps of this pixel's window inside the image: rows rlo..rhi, columns slo..shi
                int rlo = max(0, -h0), rhi = min(R_ - 1, Hi_ - 1 - h0);
                int slo = max(0, -w0), shi = min(S_ - 1, Wi_ - 1 - w0);
                const bool ok = (m < M_) & (rlo <= rhi) & (slo <= shi);
                rlo = min(rlo, R_ - 1);
                rhi = max(rhi, 0);
                slo = min(slo, S_ - 1);
                const int sspan = max(shi - slo, 0);
                const unsigned hm = (full << (rlo * S_)) & (full >> ((R_ - 1 - rhi) * S_));
                const unsigned wmk = rep * (((2u << sspan) - 1u) << slo);
                a_inv[i] = ok ? ~(hm & wmk) : ~0u;
                a_voff[i] = ok ? (unsigned)(((((img - img0) * Hi_ + h0 + phb) * Wi_) + w0 + pwb) * Ci_ * 4 + kq * 16) : 0u;
            }
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
                const unsigned vo = ((a_inv[l] << up) & kBufferBytes) | a_voff[l];
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
    auto split_store = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int l = 0; l < LPT; ++l) {
            const Split2 a = split2(g[l].x, g[l].y), b = split2(g[l].z, g[l].w);
            unsigned char* q = st + (l < LA ? l * 2 : BM / 16 + (l - LA) * 2) * kBlock16;
            *reinterpret_cast<uint2*>(q) = make_uint2(a.h, b.h);
            *reinterpret_cast<uint2*>(q + 1024) = make_uint2(a.m, b.m);
            *reinterpret_cast<uint2*>(q + 2048) = make_uint2(a.l, b.l);
        }
    };

    // ---------------- compute side ----------------
    f32x4 acc[TM][TN];
    bf16x8 fa[3][TM], fb[3][TN];
    const unsigned char* const fr = lds + fgrp * 256 + ((frow ^ (fgrp << 1)) * 16);
    auto read_a = [&](int plane) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < TM; ++i) fa[plane][i] = *reinterpret_cast<const bf16x8*>(fr + (wm * TM + i) * kBlock16 + plane * 1024);
    };
    auto read_b = [&](int plane) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < TN; ++j) fb[plane][j] = *reinterpret_cast<const bf16x8*>(fr + (BM / 16 + wn * TN + j) * kBlock16 + plane * 1024);
    };
    auto product = [&](int pa, int pb) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[pb][j], fa[pa][i], acc[i][j], 0, 0, 0);
    };
    auto clear_acc = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    };
    // An infinity or a NaN does not survive the split (inf - inf), nor does a value that rounds past the largest bf16: this wave's part of
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
            f32x4* part = reinterpret_cast<f32x4*>(p.partial) + ((size_t)2 * bid + (c_seg == rounds ? 0 : 1)) * (BM * BN / 4);
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j) part[((i * TN + j) * 4 + wave) * 64 + lane] = acc[i][j];
            return;
        }
        // 16 rows at a time through the wave's own LDS slice, so that a store covers whole rows of the wave's part (4 x 256 or 8 x 128 bytes, in
        // lane order) and not 16 bytes of each of 16 rows per 16 lanes: 1x1 over 64 channels at 56x56, batch 256, 270 -> 23x us.
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
        float* const mine = out_lds + wave * (16 * kOutPitch);
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
                if (quads) {
                    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, out[e]), d_rsrc, (int)(col < N_ ? off : kBufferBytes), 0, 0);
                } else {
#pragma unroll
                    for (int v = 0; v < 4; ++v)
                        __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(out[e][v]), d_rsrc, (int)(col + v < N_ ? off : kBufferBytes), v * 4, 0);
                }
            }
        }
        if constexpr (!SCATTER) {
            if (p.stats) {
                // Per column, the sum and the sum of squares of what this wave has just stored over its WTM rows; rows past M are zero (their
                // operands were).  A lane holds TM rows of four columns; the other 15 rows of each 16 are in its row of 16 lanes.
                const int col0 = n0 + wn * WTN + 4 * fgrp;
                f32x4* st4 = reinterpret_cast<f32x4*>(p.stats + ((size_t)(tm * 2 + wm) * N_ + col0) * 2);
                auto row_sum = [&](float x) __attribute__((always_inline)) {
                    x += __uint_as_float(__builtin_amdgcn_mov_dpp(__float_as_uint(x), 0x128 /* row_ror:8 */, 0xF, 0xF, true));
                    x += __uint_as_float(__builtin_amdgcn_mov_dpp(__float_as_uint(x), 0x124, 0xF, 0xF, true));
                    x += __uint_as_float(__builtin_amdgcn_mov_dpp(__float_as_uint(x), 0x122, 0xF, 0xF, true));
                    x += __uint_as_float(__builtin_amdgcn_mov_dpp(__float_as_uint(x), 0x121, 0xF, 0xF, true));
                    return x;
                };
#pragma unroll
                for (int j = 0; j < TN; ++j) {
                    float sum[4], sq[4];
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        float a = 0.f, b = 0.f;
#pragma unroll
                        for (int i = 0; i < TM; ++i) {
                            a += acc[i][j][v];
                            b = fmaf(acc[i][j][v], acc[i][j][v], b);
                        }
                        sum[v] = row_sum(a);
                        sq[v] = row_sum(b);
                    }
                    if (frow == 0) {
                        if (quads) {
                            if (col0 + j * 16 < N_) {
                                st4[j * 8] = f32x4{sum[0], sq[0], sum[1], sq[1]};
                                st4[j * 8 + 1] = f32x4{sum[2], sq[2], sum[3], sq[3]};
                            }
                        } else {
#pragma unroll
                            for (int v = 0; v < 4; ++v)
                                if (col0 + j * 16 + v < N_) {
                                    reinterpret_cast<float*>(st4)[(j * 16 + v) * 2] = sum[v];
                                    reinterpret_cast<float*>(st4)[(j * 16 + v) * 2 + 1] = sq[v];
                                }
                        }
                    }
                }
            }
        }
    };

    // ---------------- the pipeline ----------------
    load_step();                                  // k-step 0 of the sequence
    clear_acc();
    for (int f = 0; f < F; ++f) {
        split_store();
        if (f + 1 < F) load_step();               // stays in flight over the matrix phase
        lds_barrier();
        __builtin_amdgcn_s_setprio(1);
        read_b(0);
        read_a(2);
        read_a(1);
        __builtin_amdgcn_sched_barrier(0);
        product(2, 0);
        read_a(0);
        __builtin_amdgcn_sched_barrier(0);
        product(1, 0);
        read_b(1);
        __builtin_amdgcn_sched_barrier(0);
        product(0, 0);
        __builtin_amdgcn_sched_barrier(0);
        product(1, 1);
        read_b(2);
        __builtin_amdgcn_sched_barrier(0);
        product(0, 1);
        __builtin_amdgcn_sched_barrier(0);
        product(0, 2);
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_setprio(0);
        lds_barrier();                            // every wave has read its last fragments
        if (++c_k == c_k1) {                      // the segment is complete: store it, the next step starts a new one
            epilogue();
            clear_acc();
            ++c_seg;
            segment(c_seg, c_tile, c_k0, c_k1);
            c_k = c_k0;
        }
    }
}

// Adds the parts of every tile that stream-K blocks split between them, in k order, and stores the tile: block (t, y) handles the 16x16
// tile y of each of the four waves of stream-K tile t.  Four parts are fetched at a time.
template <int BM, int BN>
__global__ void __launch_bounds__(256) conv_split_fixup_kernel(const GemmConv p) {
    constexpr int TN = BN / 32;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int nbn = (p.N + BN - 1) / BN;
    const int nkt = (p.Kg + BK - 1) / BK;
    const long long tb = (long long)blockIdx.x * nkt, te = tb + nkt;      // this tile's k-steps in stream-K positions
    auto begin_of = [&](long long j) { return j * p.sk_iters / p.sk_blocks; };
    long long j = tb * p.sk_blocks / p.sk_iters;
    while (j > 0 && begin_of(j) > tb) --j;
    while (begin_of(j + 1) <= tb) ++j;
    if (begin_of(j) <= tb && begin_of(j + 1) >= te) return;              // one block did the whole tile and stored it
    long long j1 = te * p.sk_blocks / p.sk_iters;                        // one past the last block with a part of this tile
    while (j1 > 0 && begin_of(j1 - 1) >= te) --j1;
    while (j1 < p.sk_blocks && begin_of(j1) < te) ++j1;
    const f32x4* part = reinterpret_cast<const f32x4*>(p.partial) + (blockIdx.y * 4 + wave) * 64 + lane;
    constexpr size_t kSlot = BM * BN / 4;
    // the first block's piece is the last of its range unless its range starts here; all others start their ranges in this tile
    f32x4 sum = part[((size_t)2 * j + (begin_of(j) >= tb ? 0 : 1)) * kSlot];
    for (++j; j < j1; j += 4) {
        f32x4 v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) v[u] = part[(size_t)2 * (j + u < j1 ? j + u : j) * kSlot];
#pragma unroll
        for (int u = 0; u < 4; ++u)
            if (j + u < j1) sum += v[u];
    }
    const int tile = p.dp_tiles + blockIdx.x, tm = tile / nbn;
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
    s->sk = sk_plan(s->tiles, s->nkt, s->resident, true, 4);
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
        const unsigned rest = (unsigned)(s.tiles - p.dp_tiles);
        hipLaunchKernelGGL((conv_split_fixup_kernel<128, BN>), dim3(rest, 16 * BN / 128), dim3(256), 0, stream, p);
        if (p.stats) lc_launch_tile_stats(p, 128, BN, p.dp_tiles, rest, stream);
    }
    return lc_end_call();
}

}  // namespace

size_t lc_conv_split_workspace(const GemmConv& p) {
    SplitPlan s;
    if (!split_plan(p, &s)) return 0;
    return (size_t)2 * s.sk.sk_blocks * 128 * s.bn * sizeof(float);
}

lc_status lc_launch_conv_split(GemmConv p, hipStream_t stream) {
    SplitPlan s;
    if (!split_plan(p, &s)) return LC_ERR_UNSUPPORTED;
    if (p.scatter && p.stats) return LC_ERR_UNSUPPORTED;
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
    magic_for(p.Qo, &p.qo_mul, &p.qo_shift);
    magic_for(p.Po, &p.po_mul, &p.po_shift);
    const unsigned grid = p.dp_tiles > 0 ? (unsigned)s.resident : (unsigned)p.sk_blocks;
    const bool whole = p.sk_blocks == 0 || p.sk_iters == (long long)p.sk_blocks * s.nkt;
    return s.bn == 128 ? launch_split_tile<128>(p, s, whole, grid, stream) : launch_split_tile<64>(p, s, whole, grid, stream);
}
