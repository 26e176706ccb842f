#include "sparq_packed_act_kernel.h"

namespace sparq {
CodecKernel codec_kernel_2bit(bool pack, int sb, int group, bool pair, bool variant) {
    return pack ? codec_kernel_n<2, true>(sb, group, pair, variant) : codec_kernel_n<2, false>(sb, group, pair, variant);
}
}  // namespace sparq
