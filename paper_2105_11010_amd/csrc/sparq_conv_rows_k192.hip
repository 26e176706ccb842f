// 1x1 SPARQ convolution with the activations in registers: up to 192 channels, every trim variant and output.
#include "sparq_conv_rows_kernel.h"

namespace sparq {
SPARQ_DECLARE_ROWS(launch_rows_k192) { return launch_rows_kind<RowsCfg<6, 1, true, 3>, RowsCfg<6, 2, true, 2>>(kind, p, s); }
}  // namespace sparq
