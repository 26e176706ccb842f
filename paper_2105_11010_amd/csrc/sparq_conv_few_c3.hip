// SPARQ convolution of layers with three channels: every filter height, stride and output.
#include "sparq_conv_few_kernel.h"

namespace sparq {
sparq_status launch_few_c3(const FewParams& p, hipStream_t s) { return launch_few_channels<3>(p, s); }
}  // namespace sparq
