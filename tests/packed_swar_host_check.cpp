// Host build of the packed-storage codec's record arithmetic (its intrinsics emulated), so that it can be compared
// with the oracle over the whole input domain without a GPU.  Compiled on the fly by tests/test_packed_swar_host.py.
#include "../paper_2105_11010_amd/csrc/sparq_packed_swar.h"

#include <string.h>

using namespace sparq;

namespace {
template <int N, int SB, int G, bool PAIR>
void run(const PackLuts& L, bool round, const unsigned char* x, long records, unsigned* packed, unsigned char* y) {
    constexpr int W = codec_words(N, SB, G, PAIR);
    for (long r = 0; r < records; ++r) {
        uint32_t w[8], rec[W], back[8];
        memcpy(w, x + 32 * r, 32);
        if (round) pack_record<N, SB, G, PAIR, true>(w, L, rec);
        else pack_record<N, SB, G, PAIR, false>(w, L, rec);
        memcpy(packed + W * r, rec, sizeof(rec));
        unpack_record<N, SB, G, PAIR>(rec, L, back);
        memcpy(y + 32 * r, back, 32);
    }
}
template <int N, int SB>
int run_group(int group, bool pair, const PackLuts& L, bool round, const unsigned char* x, long records, unsigned* packed, unsigned char* y) {
    if (pair) { run<N, SB, 1, true>(L, round, x, records, packed, y); return 0; }
    switch (group) {
        case 1: run<N, SB, 1, false>(L, round, x, records, packed, y); return 0;
        case 2: run<N, SB, 2, false>(L, round, x, records, packed, y); return 0;
        case 4: run<N, SB, 4, false>(L, round, x, records, packed, y); return 0;
        case 8: run<N, SB, 8, false>(L, round, x, records, packed, y); return 0;
        case 16: run<N, SB, 16, false>(L, round, x, records, packed, y); return 0;
        case 32: run<N, SB, 32, false>(L, round, x, records, packed, y); return 0;
    }
    return 1;
}
}  // namespace

// records * 32 channels in x; their records (sb ShiftCtrl bits) in packed, the values these encode in y.
extern "C" int codec_records(int n, unsigned S, int round, int pair, int group, int sb, const unsigned char* x, long records,
                             unsigned* packed, unsigned char* y) {
    const PackLuts L = make_pack_luts(n, S);
#define CASE(NN, SS) if (n == NN && sb == SS) return run_group<NN, SS>(group, pair != 0, L, round != 0, x, records, packed, y);
    CASE(4, 1) CASE(4, 2) CASE(4, 3) CASE(3, 1) CASE(3, 2) CASE(3, 3) CASE(2, 1) CASE(2, 2) CASE(2, 3)
#undef CASE
    return 1;
}
