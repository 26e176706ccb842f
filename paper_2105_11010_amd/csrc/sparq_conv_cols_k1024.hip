// 1x1 SPARQ convolution with the weights in registers: up to 1024 channels, every trim variant and output.
#include "sparq_conv_cols_kernel.h"

namespace sparq {
SPARQ_DECLARE_ROWS(launch_cols_k1024) { return launch_cols_kind<ColsCfg<32, 1, 1, 1>>(kind, p, s); }
}  // namespace sparq
