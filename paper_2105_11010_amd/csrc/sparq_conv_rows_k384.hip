// 1x1 SPARQ convolution with the activations in registers: up to 384 channels, every trim variant and output.
#include "sparq_conv_rows_kernel.h"

namespace sparq {
SPARQ_DECLARE_ROWS(launch_rows_k384) { return launch_rows_kind<RowsCfg<12, 1, true, 2>, RowsCfg<12, 2, false, 2>>(kind, p, s); }
}  // namespace sparq
