// SPARQ matrix product with a long reduction, eight wavefronts per tile: 128 x 256 tiles, every trim variant and output.
#include "sparq_conv_wide_kernel.h"

namespace sparq {
sparq_status launch_wide_256(TrimKind kind, const WideParams& p, hipStream_t s) { return launch_wide_kind<Wide256>(kind, p, s); }
}  // namespace sparq
