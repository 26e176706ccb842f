// 1x1 SPARQ convolution with the activations in registers: up to 128 channels, every trim variant and output.
#include "sparq_conv_rows_kernel.h"

namespace sparq {
SPARQ_DECLARE_ROWS(launch_rows_k128) { return launch_rows_kind<RowsCfg<4, 1, true, 4>>(kind, p, s); }
}  // namespace sparq
