#include "sparq_packed_act_kernel.h"

namespace sparq {
CodecKernel codec_kernel_3bit(bool pack, int sb, int group, bool pair, bool variant) {
    return pack ? codec_kernel_n<3, true>(sb, group, pair, variant) : codec_kernel_n<3, false>(sb, group, pair, variant);
}
}  // namespace sparq
