// conv_dma_kernel's tiles of 256 columns (conv_dma.h).
#include "conv_dma.h"

lc_status lc_launch_conv_dma_wide(const GemmConv& p, int tile, int nkt, long long tiles, int dp_tiles, int sk_blocks, long long sk_iters, hipStream_t stream) {
    const ConvDmaPlan c = {tile, nkt, tiles, {dp_tiles, sk_blocks, sk_iters}};
    switch (tile) {
        case kWide: return launch_conv_dma<8, 8, 4, 4, 2>(p, c, stream);
        case kOtherRows: return launch_conv_dma<8, 7, 4, 4, 2>(p, c, stream);
        case kOtherRows + 1: return launch_conv_dma<7, 7, 4, 4, 2>(p, c, stream);
        case kOtherRows + 2: return launch_conv_dma<7, 6, 4, 4, 2>(p, c, stream);
        case kOtherRows + 3: return launch_conv_dma<6, 6, 4, 4, 2>(p, c, stream);
    }
    return LC_ERR_UNSUPPORTED;
}
