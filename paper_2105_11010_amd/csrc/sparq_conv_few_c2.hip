// SPARQ convolution of layers with two channels: every filter height, stride and output.
#include "sparq_conv_few_kernel.h"

namespace sparq {
sparq_status launch_few_c2(const FewParams& p, hipStream_t s) { return launch_few_channels<2>(p, s); }
}  // namespace sparq
