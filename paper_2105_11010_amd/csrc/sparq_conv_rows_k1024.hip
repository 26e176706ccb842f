// 1x1 SPARQ convolution with the activations in registers: up to 1024 channels, every trim variant and output.
#include "sparq_conv_rows_kernel.h"

namespace sparq {
SPARQ_DECLARE_ROWS(launch_rows_k1024) { return launch_rows_kind<RowsCfg<32, 1, false, 2>>(kind, p, s); }
}  // namespace sparq
