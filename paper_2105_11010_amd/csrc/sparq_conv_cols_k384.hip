// 1x1 SPARQ convolution with the weights in registers: up to 384 channels, every trim variant and output.
#include "sparq_conv_cols_kernel.h"

namespace sparq {
SPARQ_DECLARE_ROWS(launch_cols_k384) { return launch_cols_kind<ColsCfg<12, 2, 1, 2>, ColsCfg<12, 2, 2, 1>>(kind, p, s); }
}  // namespace sparq
