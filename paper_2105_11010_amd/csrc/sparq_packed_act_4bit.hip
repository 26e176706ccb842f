#include "sparq_packed_act_kernel.h"

namespace sparq {
CodecKernel codec_kernel_4bit(bool pack, int sb, int group, bool pair, bool variant) {
    return pack ? codec_kernel_n<4, true>(sb, group, pair, variant) : codec_kernel_n<4, false>(sb, group, pair, variant);
}
}  // namespace sparq
