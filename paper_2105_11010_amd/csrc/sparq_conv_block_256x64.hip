// Multi-tap SPARQ convolution as many small workgroups, 256 pixels x 64 channels: every trim variant and output.
#include "sparq_conv_block_kernel.h"

namespace sparq {
sparq_status launch_block_256x64(TrimKind kind, const BlockParams& p, int npix_max, hipStream_t s) {
    return launch_block_tile<Block256x64>(kind, p, npix_max, s);
}
}  // namespace sparq
