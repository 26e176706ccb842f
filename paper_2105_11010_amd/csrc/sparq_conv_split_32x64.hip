// Small-layer SPARQ convolution, reduction split over the wavefronts: 32x64 tiles, every trim variant.
#include "sparq_conv_split_kernel.h"

namespace sparq {
sparq_status launch_split_32x64(TrimKind kind, const SplitParams& p, int npix_max, hipStream_t s) { return launch_split_kind<Split32x64>(kind, p, npix_max, s); }
}  // namespace sparq
