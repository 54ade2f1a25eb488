// bf16 filter gradients with operands straight into LDS.
#include "dma_common.h"

namespace {

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

// One tile of large operands, bound by memory: all blocks work on one narrow stretch of both (and past the caches: nothing reads them again) instead of each on rows of its own.  us, each on its own / so, two
// sets in turn, images of 56x56: 128 to 64, 319 images 74.3 / 64.3, 205 49.8 / 43.5, 160 39.8 / 36.5; 64 to 128, 512 images 110 / 98, 200 to 72 160 / 141, 72 to 160 137 / 124, 128 to 32 88 / 78, 16 to 128 83 / 75.
// From 160 MB on: 128 to 64, 154 MB 38.1 / 37.9, 96 to 64, 128 MB 26.4 / 30.6.  Where the operands fill three fifths of the tile's rows and columns: 72 to 72 82 / 89, 72 to 32 62 / 66, 8 to 96 64 / 65, though 8 to 160
// 99 / 96.  Several tiles read the same rows, and the L2s hold them better in one place: 512 to 128 at 28x28 104 / 108, 512 to 2048 at 7x7 64 / 73.
static bool wgrad_around(const GemmWgrad& p, int bm, int bn) {
    return wgrad_plain(p) && p.K <= bm && p.J <= bn && 5 * (p.K + p.J) >= 3 * (bm + bn) && (double)p.M * (p.K + p.C) * 2 >= 160e6;
}
// 128x128 tiles whose blocks have a compute unit each: eight waves, which hide each other's reads of LDS.  us, four / eight: 3x3 over 512 channels, 37 images of 7x7 24.8 / 22.3, one image of 28x28 14.9 / 13.2,
// 512 to 256, 16 of 14x14 23.4 / 21.7; 1x1 256 to 448, 96 of 21x21 27.3 / 25.9.  Splits of up to 100 stages gain, 1 to 12 % (twenty-six layers, the worst 1.015); longer ones are bound by memory: 196
// stages, 512 to 128, 512 of 28x28 102 / 103, 200 to 72, 256 of 56x56 84 / 96.
static bool wgrad_eight_waves(const GemmWgrad& p) {
    return (long long)((p.K + 127) / 128) * ((p.J + 127) / 128) * p.splits <= device_cu_count() && p.m_per_split <= 128 * 32;
}

const char* lc_wgrad_dma_form(const GemmWgrad& p) {
    const bool eight = p.dma_bm == 128 && p.dma_bn == 128 && wgrad_eight_waves(p);
    return wgrad_around(p, p.dma_bm, p.dma_bn) ? (eight ? " eight waves around" : " around") : eight ? " eight waves" : "";
}

lc_status lc_launch_wgrad_dma(const GemmWgrad& p, hipStream_t stream) {
    if (!aligned16(p.dy) || !aligned16(p.x)) return LC_ERR_ALIGN;
    const bool plain = wgrad_plain(p);
    auto go = [&]<int BM, int BN, int WM, int WN, int NS>() {
        if (wgrad_around(p, BM, BN)) return launch_wgrad_dma<BM, BN, WM, WN, NS, kAround>(p, stream);
        return plain ? launch_wgrad_dma<BM, BN, WM, WN, NS, kPlain>(p, stream) : launch_wgrad_dma<BM, BN, WM, WN, NS, kWindow>(p, stream);
    };
    switch (p.dma_bm * 1000 + p.dma_bn) {
        case 256256: return go.template operator()<256, 256, 2, 4, 4>();
        case 256128: return go.template operator()<256, 128, 4, 2, 5>();
        case 128256: return go.template operator()<128, 256, 2, 4, 5>();
        case 128128:
            if (wgrad_eight_waves(p)) return go.template operator()<128, 128, 2, 4, 5>();
            return go.template operator()<128, 128, 2, 2, 4>();
        case 256064: return go.template operator()<256, 64, 4, 1, 3>();
        case 64256: return go.template operator()<64, 256, 1, 4, 3>();
        case 128064: return go.template operator()<128, 64, 2, 2, 4>();
        case 64128: return go.template operator()<64, 128, 1, 4, 4>();
    }
    return LC_ERR_UNSUPPORTED;
}
