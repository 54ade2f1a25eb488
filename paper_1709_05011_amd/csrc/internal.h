// Declarations shared by the translation units of liblarsconv (not part of the C ABI).
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "../../include/larsconv.h"

// Launch bookkeeping (conv_api.hip).  lc_begin_call() drops any stale error another user of the HIP
// runtime left on this thread, so that lc_end_call() reports only what this library's launches caused.
void lc_begin_call();
lc_status lc_end_call();     // LC_OK, or LC_ERR_LAUNCH with the detail text recorded
lc_status lc_fail_call(hipError_t e, const char* what);   // records "what: error" as the detail text, returns LC_ERR_LAUNCH

// fp32 -> bf16, round to nearest even (NaN stays NaN): the conversion instruction of gfx950
__device__ __forceinline__ uint16_t lc_bf16_rne(float x) { return __builtin_bit_cast(uint16_t, (__bf16)x); }
// two at once: lo in bits 0..15, hi in bits 16..31
__device__ __forceinline__ uint32_t lc_bf16x2_rne(float lo, float hi) {
    typedef float lc_f32x2 __attribute__((ext_vector_type(2)));
    typedef __bf16 lc_bf16x2 __attribute__((ext_vector_type(2)));
    const lc_f32x2 v = {lo, hi};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, lc_bf16x2));
}

// 16-byte accesses.  NT: non-temporal, for streams that nothing reads again soon; a line that the caches hold is still found there.
typedef unsigned lc_u32x4 __attribute__((ext_vector_type(4)));
template <bool NT, typename R>
__device__ __forceinline__ R lc_fetch16(const void* p) {
    static_assert(sizeof(R) == 16, "16-byte access");
    if constexpr (NT) return __builtin_bit_cast(R, __builtin_nontemporal_load(static_cast<const lc_u32x4*>(p)));
    else return *static_cast<const R*>(p);
}
template <bool NT, typename R>
__device__ __forceinline__ void lc_put16(void* p, const R& v) {
    static_assert(sizeof(R) == 16, "16-byte access");
    if constexpr (NT) __builtin_nontemporal_store(__builtin_bit_cast(lc_u32x4, v), static_cast<lc_u32x4*>(p));
    else *static_cast<R*>(p) = v;
}

// ---- small device-side utilities (layout.hip) ----
void lc_bf16_to_f32(const void* src, float* dst, size_t count, hipStream_t stream);
void lc_f32_to_bf16(const float* src, void* dst, size_t count, hipStream_t stream);
void lc_fill_f32(float* dst, float value, size_t count, hipStream_t stream);
void lc_fill_u32x4(void* dst, size_t bytes16, hipStream_t stream);   // zero `bytes16` * 16 bytes
void lc_zero_bytes(void* dst, size_t bytes, hipStream_t stream);      // zero an even number of bytes at a 2-byte aligned address
void lc_zero_off_grid(void* dst, int n, int h, int w, size_t pixel_bytes, int sh, int sw, bool past,
                      hipStream_t stream);   // [n][h][w] pixels but those on the stride grid; past: past the caches

// rows x width_bytes bytes from src (row pitch src_pitch bytes) to dst (row pitch dst_pitch); every size a multiple of 2
void lc_copy2d(const void* src, size_t src_pitch, void* dst, size_t dst_pitch, size_t width_bytes, size_t rows, hipStream_t stream);

// NCHW <-> NHWC for activations ([n][c][hw] <-> [n][hw][c]); esize 4 (fp32) or 2 (bf16).
void lc_nchw_to_nhwc(const void* src, void* dst, int n, int c, int hw, int esize, hipStream_t stream);
void lc_nhwc_to_nchw(const void* src, void* dst, int n, int c, int hw, int esize, hipStream_t stream);

// Filter re-ordering.  All take and give fp32 or bf16 by esize.
//  KRSC -> [c][R-1-r][S-1-s][k]  (the filter of the backward-data convolution)
void lc_filter_for_bwd_data(const void* w_krsc, void* out, int k, int c, int r, int s, int esize, hipStream_t stream);
//  the taps r = a, a + sh, ... / s = b, b + sw, ... of it (ra x sb of them) in the same order: one stride phase
void lc_filter_for_bwd_data_phase(const void* w_krsc, void* out, int k, int c, int r, int s, int a, int b, int sh, int sw, int ra,
                                  int sb, int esize, hipStream_t stream);
//  pad the channel dimension (innermost) of an [rows][c] array with zeros to [rows][cpad]
// few-channel stride-2 convolution as a stride-1 convolution over 2x2 pixel blocks (see layout.hip)
void lc_stem_unfold(const void* x, void* u, int n, int c, int h, int w, int q, int hb, int sb, int cu, int eph, int epw, int esize,
                    hipStream_t stream);
void lc_stem_filter(const void* w, void* wu, int k, int r, int s, int c, int rb, int sb, int cu, int eh, int ew, int esize,
                    hipStream_t stream);
void lc_stem_filter_grad(const float* dwu, float* dw, int k, int r, int s, int c, int rb, int cu, int eh, int ew, hipStream_t stream);
void lc_pad_channels(const void* src, void* dst, size_t rows, int c, int cpad, int esize, hipStream_t stream);

// dw[k][j] (j < cols, c index j % cpad < c kept) = sum over splits of part[z][k][cols] in index order.
// sq (may be null): one double per block of the reduction, lc_reduce_splits_blocks(rows_times_cols) of them, the sum of
// the squares of the values that block wrote to dw.
void lc_reduce_splits(const float* part, float* dw, int splits, size_t rows_times_cols, int cpad, int c, double* sq, hipStream_t stream);
size_t lc_reduce_splits_blocks(size_t rows_times_cols);
// sq[b] = sum of x[i]^2 over elements 4096*b .. 4096*b + 4095: lc_sq_partials_blocks(count) doubles
void lc_sq_partials(const float* x, size_t count, double* sq, hipStream_t stream);
size_t lc_sq_partials_blocks(size_t count);

// ---- implicit-GEMM convolution kernels (conv_igemm.hip) ----
// One problem D[m][n] = sum_kg A(m, kg) * B[n][kg] where A is gathered from an NHWC tensor:
// row m = (img, po, qo), column kg = (r, s, ci).
struct GemmConv {
    const void* a;      // gathered tensor [imgs][Hi][Wi][Ci]
    const void* b;      // [N][Kg], Kg = R*S*Ci contiguous
    void* d;            // output rows of ldd elements
    int M, N, Kg;
    int Hi, Wi, Ci;
    int Po, Qo;         // m -> (img, po, qo)
    int R, S;
    int sh, sw;         // position stride:  h = po*sh - ph + r
    int ph, pw;
    int dh, dw;         // > 1: "dilated" read, valid only where h % dh == 0, then h /= dh
    int ldd;
    // scatter epilogue (0 = off): row (img,po,qo) is pixel (po*esh, qo*esw) of an [imgs][Ho][Wo][ldd] tensor;
    // the pixels between the stride grid are the caller's, every value on it is written.
    int scatter, Ho, Wo, esh, esw;
    // stream-K split, filled in by the launcher: whole-tile blocks, blocks sharing the k-steps of the
    // remaining tiles, their total k-steps, and the workspace for partial tiles (2 slots per such block)
    int dp_tiles, sk_blocks;
    long long sk_iters;
    // first k-step of stream-K block j: j * sk_iters / sk_blocks = j * sk_q + j * sk_rem / sk_blocks, the quotient by multiply-high constants
    int sk_q, sk_rem;
    unsigned sk_mul, sk_shift;
    float sk_per_step;  // sk_blocks / sk_iters, about
    float* partial;
    // multiply-high division constants for Qo and Po (filled in by the launcher)
    unsigned qo_mul, qo_shift, po_mul, po_shift;
    int bf16;           // operands a, b and result d are bf16 (sums stay fp32)
    int split;          // fp32 backward-data: products as sums of bf16 products (conv_split.hip)
    // not null (main and slab kernels, no scatter): [lc_conv_gemm_stats_tiles()][N][2] floats -- per half tile of rows and
    // per column, the sum and the sum of squares of the values stored to d (as stored: after rounding to bf16)
    float* stats;
    int copied;         // d is copied to another layout next
    int stream_d;       // d is stored past the caches (lc_stream_out()): set by lc_launch_conv_gemm()
};
// Whether a convolution's result of so many bytes is stored with non-temporal stores.  They do not push the operands out of the caches, and they go to memory in
// order: us, 512 images in bf16, ordinary / so, alternating: 128 to 512 1x1 at 28x28 128 / 86, 256 to 1024 at 14x14 87 / 65, 64 to 256 at 56x56 200 / 195 and its
// backward-data 198 / 187, 3x3 over 128 channels at 28x28 130 / 121 and 134 / 127; also where two stores fill a line between them (64 columns: 256 to 64 at 56x56 193 / 184, 3x3 32 to 64 at
// 56x56 128 / 114).  fp32, 256 images: 128 to 512 at 28x28 230 / 224, its backward-data 174 / 173, 512 to 128 216 / 217 and 199 / 191, 3x3 over 128 435 / 433 and 314 / 318, 16 to 128 1x1 at 56x56
// 107 / 91; most others within 1 %.  A result that the caches hold until the next layer reads it is worth more there: whole bf16 step at 512 images 35.24 ms without, 34.80 from 64 MB,
// 34.73 to 34.79 from 30, 50, 90 or 120 MB; fp32 at 32 images 10.44 with and without.  Results below the line gain as much by themselves (128 to 64 1x1 at 28x28, 51 MB 31 / 27) or nothing (3x3 over 256 at
// 14x14, 51 MB 94.0 / 93.2).  Only where every row is whole lines of 128 bytes: a line that two tiles fill goes to memory twice (64 to 104 1x1 at 56x56 122 / 159, to 200 187 / 309; fp32, 64 to 100 170 / 201).
constexpr double kStreamOutBytes = 64e6;
// A copy that another layout is made of at once is left to the caches as long as the memory-side cache can hold it (NCHW, the pass and its transposes, us: bf16 3x3 over 128, 103 MB 310 / 318 and 313 / 321,
// 512 to 128 562 / 586; fp32 103 and 206 MB no difference; 128 to 512, 411 MB, bf16 603 / 547, fp32 506 / 490).  (Copies of a group's channels gain from 64 MB on: 3x3 over 128 392 / 374 and 398 / 376.)
constexpr double kStreamCopyBytes = 256e6;
inline int lc_stream_out(double bytes, const void* d, size_t row_bytes, double least = kStreamOutBytes) {
    return bytes >= least && row_bytes % 128 == 0 && (reinterpret_cast<uintptr_t>(d) & 127) == 0;
}
// The same for the first layer, as long as its images leave room in the memory-side cache: they are what gains by staying there (bf16, us, ordinary / past the caches, two sets in turn, then five: 64 images
// 39 / 38 and 46 / 38, 128 86 / 67 and 86 / 66, 256 169 / 125 and 161 / 160, 512, 154 MB, 318 / 321 and 315 / 322; fp32 within 1 % from 16 to 256 images; whole steps the same either way).
inline int lc_stream_first_layer(double y_bytes, double x_bytes, const void* y, size_t row_bytes) { return x_bytes <= 128e6 && lc_stream_out(y_bytes, y, row_bytes); }
lc_status lc_launch_conv_gemm(const GemmConv& p, hipStream_t stream);
size_t lc_conv_gemm_stats_tiles(const GemmConv& p);   // row pieces of `stats` for this problem; 0: the kernel that takes it has none
extern "C" int lc_selftest_stream_k(int max_blocks);   // host check of the work split's 32-bit form (0 = all good)
extern "C" int lc_selftest_division(int max_d);   // host check of the multiply-high division constants (0 = all good)
extern "C" long long lc_selftest_lars_launches(int n_chunks, long long longest);   // host check of the update pass's launches (lars.hip)
bool lc_conv_gemm_bf16_native(const GemmConv& p);   // can the bf16 MFMA kernel take this problem (shape and alignment)?
bool lc_conv_gemm_scatter_ok(const GemmConv& p);    // can the main kernel's scatter epilogue take this problem?
// fp32 backward-data on the bf16 matrix pipe (conv_split.hip), and the partial-tile bytes they need
lc_status lc_launch_conv_split(GemmConv p, hipStream_t stream);
size_t lc_conv_split_workspace(const GemmConv& p);
// bf16 operands straight into LDS (conv_dma.hip): whether the kernel takes a problem, partial-tile bytes, row pieces of `stats`
bool lc_conv_dma_ok(const GemmConv& p);
size_t lc_conv_dma_workspace(const GemmConv& p);
size_t lc_conv_dma_stats_tiles(const GemmConv& p);
lc_status lc_launch_conv_dma(const GemmConv& p, hipStream_t stream);
// its tiles of 256 columns, with the plan that conv_dma_plan() made
lc_status lc_launch_conv_dma_wide(const GemmConv& p, int tile, int nkt, long long tiles, int dp_tiles, int sk_blocks, long long sk_iters, hipStream_t stream);
// the kernel (tile, addressing, whether blocks share tiles) that takes a problem, in words
// (`form`: also its form, where the plan has a choice of several that give the same sums)
void lc_conv_dma_describe(const GemmConv& p, bool stats, bool form, char* text, size_t size);
void lc_conv_gemm_describe(const GemmConv& p, bool stats, bool form, char* text, size_t size);
// bf16 3x3 layers from 64 channels to 33 to 64 filters whose filter a wave holds in registers (conv_dma.hip)
bool lc_conv_held_ok(const GemmConv& p, bool stats);
size_t lc_conv_held_stats_tiles(const GemmConv& p);
lc_status lc_launch_conv_held(const GemmConv& p, hipStream_t stream);
// the column sums of the tiles first_tile .. tiles - 1 of bm x bn, read back from p.d (conv_igemm.hip)
void lc_tile_stats(const GemmConv& p, int bm, int bn, int first_tile, long long tiles, hipStream_t stream);
size_t lc_conv_gemm_workspace(const GemmConv& p);   // bytes `partial` must hold for this problem (0 = none)

// ResNet's first layer in fp32 (conv_stem.hip): 7x7, stride 2, padding 3, 3 -> 64 channels, NHWC, P and Q multiples of 16.
struct StemConv {
    const float* x;     // [imgs][H][W][3]
    const float* w;     // [64][7][7][3]
    float* y;           // [imgs][P][Q][64]
    float* stats;       // [pieces][64][2] (sum, sum of squares per piece of 64 pixels) or null
    int imgs, H, W, P, Q;
    int stream_y;       // lc_stream_first_layer(): set by the launcher
};
struct StemConvBf16 {
    const uint16_t* x;  // [imgs][H][W][3]
    const uint16_t* w;  // [64][7][7][3]
    uint16_t* y;        // [imgs][P][Q][64]
    float* stats;       // as StemConv
    int imgs, H, W, P, Q;
    int stream_y;       // as StemConv
};
lc_status lc_launch_conv_stem_bf16(const StemConvBf16& p, hipStream_t stream);
struct StemWgrad {
    const float* x;     // [imgs][H][W][3]
    const float* dy;    // [imgs][P][Q][64]
    float* part;        // [blocks][64][147]: one partial filter gradient per block
    int imgs, H, W, P, Q;
};
struct StemWgradBf16 {
    const uint16_t* x;  // [imgs][H][W][3]
    const uint16_t* dy; // [imgs][P][Q][64]
    float* part;        // as StemWgrad
    int imgs, H, W, P, Q;
};
lc_status lc_launch_conv_stem_wgrad_bf16(const StemWgradBf16& p, int blocks, hipStream_t stream);
int lc_conv_stem_blocks(int imgs, int P, int Q);
lc_status lc_launch_conv_stem_wgrad_f32(const StemWgrad& p, int blocks, hipStream_t stream);
bool lc_conv_stem_f32_ok(int imgs, int c, int h, int w, int k, int r, int s, int sh, int sw, int ph, int pw, int P, int Q);
size_t lc_conv_stem_f32_stats_pieces(int imgs, int P, int Q);
lc_status lc_launch_conv_stem_f32(const StemConv& p, hipStream_t stream);

// Filter gradient: D[k][j] = sum_m dY[m][k] * Xg(m, j), m = (img, p, q), j = (r, s, c); the reduction
// over m is cut into `splits` ranges, split z writing to d + z * K * J.
struct GemmWgrad {
    const void* dy;     // [M][K]
    const void* x;      // [imgs][H][W][C]
    float* d;           // [splits][K][J]
    int M, K, J;
    int H, W, C, P, Q, R, S;
    int sh, sw, ph, pw;
    int splits, m_per_split;
    int bf16;           // dy and x are bf16 (widened on the fly; the sums and d stay fp32)
    int slab;           // 3x3 stride-1 pad-1 bf16 layer for wgrad3x3_slab_kernel: m_per_split counts padded positions
    unsigned q_mul, q_shift, p_mul, p_shift;       // multiply-high division constants for Q and P (filled in by the launcher that needs them)
    int dma_bm, dma_bn; // bf16 layer for wgrad_dma_kernel (wgrad_dma.hip): its tile, chosen by lc_wgrad_splits() (0: another kernel)
};
lc_status lc_launch_wgrad_f32(const GemmWgrad& p, hipStream_t stream);
void lc_wgrad_describe(const GemmWgrad& p, bool form, char* text, size_t size);     // the kernel that takes a planned problem, in words
int lc_wgrad_splits(GemmWgrad* p);   // fixed function of the shape (determinism); chooses the tile of wgrad_dma_kernel where that takes the layer
// bf16 operands straight into LDS (wgrad_dma.hip): tile and number of splits for a shape, false where another kernel takes it; and the launch
bool lc_wgrad_dma_plan(const GemmWgrad& p, int* bm, int* bn, int* splits);
lc_status lc_launch_wgrad_dma(const GemmWgrad& p, hipStream_t stream);
const char* lc_wgrad_dma_form(const GemmWgrad& p);      // which of its forms, in words behind a space, or nothing
int lc_wgrad_dma_sum_rows(const GemmWgrad& p);     // rows that go into one running sum
// fp32 operands on the bf16 matrix pipe (conv_split.hip), output tile bm x bn; and how many of its blocks fit on a compute unit
lc_status lc_launch_wgrad_split(const GemmWgrad& p, int bm, int bn, hipStream_t stream);
int lc_wgrad_split_blocks_per_cu(int bm, int bn);
bool lc_wgrad_slab_ok(int imgs, int H, int W, int C, int K, int R, int S, int sh, int sw, int ph, int pw, int P, int Q, bool bf16);
constexpr int kWgradSlabMinW = 24;     // columns of an image that the slab kernel takes
int lc_wgrad_round_splits(const GemmWgrad& p);     // splits that fill one round of blocks of the kernels that stage operands through registers
int lc_wgrad_slab_splits(int imgs, int H, int W, int C, int K, int* pos_per_split);
