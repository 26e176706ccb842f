// 1x1 SPARQ convolution with the weights in registers: up to 512 channels, every trim variant and output.
#include "sparq_conv_cols_kernel.h"

namespace sparq {
SPARQ_DECLARE_ROWS(launch_cols_k512) { return launch_cols_kind<ColsCfg<16, 2, 1, 1>, ColsCfg<16, 2, 2, 1>, ColsCfg<16, 2, 1, 1>>(kind, p, s); }
}  // namespace sparq
