// SPARQ matrix product with a long reduction, eight wavefronts per tile: 128 x 512 tiles, every trim variant and output.
#include "sparq_conv_wide_kernel.h"

namespace sparq {
sparq_status launch_wide_512(TrimKind kind, const WideParams& p, hipStream_t s) { return launch_wide_kind<Wide512>(kind, p, s); }
}  // namespace sparq
