// Packed storage of trimmed activations: what SPARQ's multiplier consumes (Eq. 4) instead of 8-bit values.
//
// Section 3.1: an n-bit window travels with an identifier of its position; Section 5.1: per n-bit datum a
// ShiftCtrl field and, with vSPARQ, a 1-bit MuxCtrl that names the weight the datum multiplies; Section 6:
// ShiftCtrl may be shared by a number of activations.  A pair of channels (2j, 2j+1) is stored as two data:
//   both values non-zero (or vSPARQ off): their two windows, each steered to its own channel;
//   second value zero, else first value zero (the case order of Eq. 2): the other value's 2n-bit window as a
//   high half (shift t+n) and a low half (shift t), both steered to that value's channel.
// A channel's value is the sum of datum << shift over the data steered to it.
//
// Record layout (32 channels of one row, the last record of a row zero-filled; little-endian 32-bit words):
//   data      n words          datum k in bits [k*n, k*n+n)
//   ShiftCtrl ceil(F*sb/32) w. field f in bits [f*sb, f*sb+sb): rank of the shift among the allowed ones;
//                              sb = bits to number them; F = 32 / group fields (group = 1: one per datum)
//   MuxCtrl   1 word           bit k: datum k goes to the odd channel of its pair (absent with vSPARQ off)
// group > 1 (vSPARQ off only): one shift per group of consecutive channels, the placement bSPARQ picks for the
// group's largest value; every value of the group is trimmed at that shift (floor, or round half up saturating).
//
// One lane handles one record (sparq_packed_act_kernel.h).  The window fields are recomputed from the activation's
// leading one, which selects the same window before and after the trim (rounding saturates inside it).
#include "sparq_packed_act_kernel.h"

namespace sparq {

namespace {

int shift_ctrl_bits(uint32_t S) {
    int bits = 0;
    while ((1 << bits) < __builtin_popcount(S)) ++bits;
    return bits;
}

// Bound by memory: a record per lane, so that the accesses of the moment lie close together (unpacking [65536][4608] 104 -> 98 us,
// packing it without vSPARQ 111 -> 99; up to twice the last-level cache 0.94-1.0 x, so from there on).  Bound by arithmetic (packing with vSPARQ): what a lane sets up is worth several records.
int grid_for(int64_t items, bool streams) {
    int64_t blocks = (items + kPkThreads - 1) / kPkThreads;
    const int64_t cap = streams ? 1 << 19 : 256 * 16;
    if (blocks > cap) blocks = cap;
    return (int)(blocks < 1 ? 1 : blocks);
}

// Record size in 32-bit words; 0: this mode / group has no packed form.
int record_words(const sparq_mode* mode, int group) {
    if (!mode_valid(mode) || mode->window_bits == 8) return 0;
    if (group < 1 || group > kRecChannels || kRecChannels % group != 0 || (group > 1 && mode->pair)) return 0;
    const int sb = shift_ctrl_bits(mode->shift_mask);
    return mode->window_bits + (kRecChannels / group * sb + 31) / 32 + (mode->pair ? 1 : 0);
}

sparq_status launch_codec(bool pack, const void* bytes, const void* packed, int64_t rows, int C, const sparq_mode* mode,
                          int group, hipStream_t s) {
    if (rows == 0) return SPARQ_OK;
    const int n = mode->window_bits, sb = shift_ctrl_bits(mode->shift_mask);
    const auto pick = n == 4 ? codec_kernel_4bit : n == 3 ? codec_kernel_3bit : codec_kernel_2bit;
    CodecParams p{};
    p.bytes = static_cast<uint8_t*>(const_cast<void*>(bytes));
    p.packed = static_cast<uint32_t*>(const_cast<void*>(packed));
    p.C = C;
    p.nrec = (C + kRecChannels - 1) / kRecChannels;
    p.records = rows * p.nrec;
    p.total = rows * C;
    p.div_nrec = make_fastdiv((uint32_t)p.nrec);
    p.L = make_pack_luts(n, mode->shift_mask);
    const bool turn = C % kRecChannels == 0 && aligned(bytes, 4) && p.total + p.records * record_words(mode, group) * 4 >= kStreamedBytes;
    const CodecKernel kernel = pick(pack, sb, group, mode->pair != 0, pack ? mode->round_nearest != 0 : turn);
    if (!kernel) return SPARQ_EUNSUPPORTED;
    const bool streams = (!pack || !mode->pair) && p.total + p.records * record_words(mode, group) * 4 >= 2 * (int64_t)kStreamedBytes;
    kernel<<<grid_for(p.records, streams), kPkThreads, 0, s>>>(p);
    return launch_status();
}

}  // namespace

sparq_status launch_unpack_act(const void* packed, uint8_t* y, int64_t rows, int C, const sparq_mode* mode, int group,
                               hipStream_t s) {
    return launch_codec(false, y, packed, rows, C, mode, group, s);
}

}  // namespace sparq

using namespace sparq;

extern "C" size_t sparq_packed_act_bytes(int64_t rows, int32_t C, const sparq_mode* mode, int32_t group) {
    const int words = record_words(mode, group);
    if (words == 0 || rows < 0 || C <= 0) return 0;
    return (size_t)rows * (size_t)((C + kRecChannels - 1) / kRecChannels) * (size_t)words * 4;
}

extern "C" sparq_status sparq_pack_act(const uint8_t* x, void* packed, size_t packed_bytes, int64_t rows, int32_t C,
                                       const sparq_mode* mode, int32_t group, void* stream) {
    if (rows < 0 || C <= 0 || record_words(mode, group) == 0) return SPARQ_EINVAL;
    if (rows == 0) return SPARQ_OK;                      // nothing to do (the pointers are not looked at)
    if (!x || !packed || !aligned(packed, 4)) return SPARQ_EINVAL;
    if (packed_bytes < sparq_packed_act_bytes(rows, C, mode, group)) return SPARQ_EWORKSPACE;
    return launch_codec(true, x, packed, rows, C, mode, group, static_cast<hipStream_t>(stream));
}

extern "C" sparq_status sparq_unpack_act(const void* packed, size_t packed_bytes, uint8_t* y, int64_t rows, int32_t C,
                                         const sparq_mode* mode, int32_t group, void* stream) {
    if (rows < 0 || C <= 0 || record_words(mode, group) == 0) return SPARQ_EINVAL;
    if (rows == 0) return SPARQ_OK;
    if (!packed || !y || !aligned(packed, 4)) return SPARQ_EINVAL;
    if (packed_bytes < sparq_packed_act_bytes(rows, C, mode, group)) return SPARQ_EWORKSPACE;
    return launch_codec(false, y, packed, rows, C, mode, group, static_cast<hipStream_t>(stream));
}
