// Multi-tap SPARQ convolution as many small workgroups, 128 pixels x 128 channels: every trim variant and output.
#include "sparq_conv_block_kernel.h"

namespace sparq {
sparq_status launch_block_128x128(TrimKind kind, const BlockParams& p, int npix_max, hipStream_t s) {
    return launch_block_tile<Block128x128>(kind, p, npix_max, s);
}
}  // namespace sparq
