// bf16 forward and backward-data with operands straight into LDS: the question whether a problem is taken, the plan, tiles of up to 128 columns
// (conv_dma.h), and the kernel of the 64-channel 3x3 layers.
#include "conv_dma.h"

namespace {

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

// PAST: the result leaves past the caches (chosen store by store, the layers that don't took 2 % longer: 128 images of 56x56 42.7 us, 43.5 so)
template <bool STATS, bool PAST>
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
            __builtin_amdgcn_raw_buffer_store_b128(out[e], d_rsrc, (int)d_voff, m * ldd_ * 2, PAST ? kNonTemporal : 0);
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

void lc_conv_dma_describe(const GemmConv& p, bool stats, bool form, char* text, size_t size) {
    ConvDmaPlan c;
    static const char* const in[] = {"chunks", "padded", "pieces", "runs", "taps"};
    if (!conv_dma_plan(p, !stats, &c)) snprintf(text, size, "none");
    else
        snprintf(text, size, "conv_dma %dx%d%s %s%s%s", kConvTiles[c.tile].bm, kConvTiles[c.tile].bn, c.tile == kNarrowTwoWaves ? " two waves" : "",
                 in[conv_dma_in(p)], conv_dma_shares(c) ? " shared" : "",
                 !form ? "" : conv_dma_deep(p, c) ? " four stages" : conv_dma_in(p) == kChunks && conv_dma_once(p, kConvTiles[c.tile].bn) ? " once" : "");
}

lc_status lc_launch_conv_dma(const GemmConv& p, hipStream_t stream) {
    ConvDmaPlan c;
    if (!conv_dma_plan(p, p.stats == nullptr, &c)) return LC_ERR_UNSUPPORTED;
    if (p.scatter && p.stats) return LC_ERR_UNSUPPORTED;
    auto go = [&]<int TMA, int TMB, int TN, int WN, int NS = 2>() { return launch_conv_dma<TMA, TMB, TN, WN, NS>(p, c, stream); };
    const bool deep = conv_dma_deep(p, c);
    lc_status st = LC_ERR_UNSUPPORTED;
    switch (c.tile) {
        case kSquare: st = deep ? go.template operator()<4, 4, 2, 4, 4>() : go.template operator()<4, 4, 4, 2>(); break;
        case kNarrow: st = deep ? go.template operator()<4, 4, 2, 2, 4>() : go.template operator()<4, 4, 2, 2>(); break;
        case kNarrowTwoWaves: st = go.template operator()<4, 4, 4, 1>(); break;
        case kSlim: st = go.template operator()<4, 4, 2, 1>(); break;
        default: st = lc_launch_conv_dma_wide(p, c.tile, c.nkt, c.tiles, c.sk.dp_tiles, c.sk.sk_blocks, c.sk.sk_iters, stream);
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
    ConvHeld c;
    if (!conv_held_ok(p, p.stats != nullptr, &c)) return LC_ERR_UNSUPPORTED;
    c.g = p;
    magic_for(p.Wi, &c.w_mul, &c.w_shift);
    magic_for(p.Wi + 2, &c.w2_mul, &c.w2_shift);
    magic_for(c.per_image, &c.t_mul, &c.t_shift);
    const dim3 grid((unsigned)std::min(c.tiles, device_cu_count()));
    auto launch = [&]<bool STATS, bool PAST>() {
        static const bool once =
            hipFuncSetAttribute(reinterpret_cast<const void*>(conv3x3_held_kernel<STATS, PAST>), hipFuncAttributeMaxDynamicSharedMemorySize, lds) == hipSuccess;
        if (once) hipLaunchKernelGGL((conv3x3_held_kernel<STATS, PAST>), grid, dim3(256), lds, stream, c);
        return once;
    };
    const bool launched = p.stats ? (p.stream_d ? launch.template operator()<true, true>() : launch.template operator()<true, false>())
                                  : (p.stream_d ? launch.template operator()<false, true>() : launch.template operator()<false, false>());
    if (!launched) return LC_ERR_LAUNCH;
    return lc_end_call();
}
