// SPARQ convolution of layers with one channel: every filter height, stride and output.
#include "sparq_conv_few_kernel.h"

namespace sparq {
sparq_status launch_few_c1(const FewParams& p, hipStream_t s) { return launch_few_channels<1>(p, s); }
}  // namespace sparq
