// Multi-tap SPARQ convolution as many small workgroups: every trim variant and output.
#include "sparq_conv_block_kernel.h"

namespace sparq {
template <int KIND>
static sparq_status launch_block_out(const BlockParams& p, int npix_max, hipStream_t s) {
    return p.out_u8 ? launch_block_cfg<KIND, true>(p, npix_max, s) : launch_block_cfg<KIND, false>(p, npix_max, s);
}

sparq_status launch_block(TrimKind kind, const BlockParams& p, int npix_max, hipStream_t s) {
    switch (kind) {
        case kTrimNone: return launch_block_out<kTrimNone>(p, npix_max, s);
        case kTrimFloor: return launch_block_out<kTrimFloor>(p, npix_max, s);
        case kTrimFloorPair: return launch_block_out<kTrimFloorPair>(p, npix_max, s);
        case kTrimFloorPairWide: return launch_block_out<kTrimFloorPairWide>(p, npix_max, s);
        case kTrimRound: return launch_block_out<kTrimRound>(p, npix_max, s);
        case kTrimRound4: return launch_block_out<kTrimRound4>(p, npix_max, s);
        case kTrimRoundPairWide: return launch_block_out<kTrimRoundPairWide>(p, npix_max, s);
        case kTrimRoundPair4: return launch_block_out<kTrimRoundPair4>(p, npix_max, s);
        default: return SPARQ_EUNSUPPORTED;
    }
}
}  // namespace sparq
