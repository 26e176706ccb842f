// 1x1 SPARQ convolution with the activations in registers: up to 64 channels, every trim variant and output.
#include "sparq_conv_rows_kernel.h"

namespace sparq {
SPARQ_DECLARE_ROWS(launch_rows_k64) { return launch_rows_kind<RowsCfg<2, 1, true, 4>>(kind, p, s); }
}  // namespace sparq
