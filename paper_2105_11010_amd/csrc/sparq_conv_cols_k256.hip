// 1x1 SPARQ convolution with the weights in registers: up to 256 channels, every trim variant and output.
#include "sparq_conv_cols_kernel.h"

namespace sparq {
SPARQ_DECLARE_ROWS(launch_cols_k256) { return launch_cols_kind<ColsCfg<8, 2, 1, 2>>(kind, p, s); }
}  // namespace sparq
