// Host build of the GPU library's packed-byte trim (its intrinsics emulated), so the
// bit manipulation can be compared with the oracle over the whole input domain
// without a GPU.  Compiled on the fly by tests/test_swar_host.py.
#include "../paper_2105_11010_amd/csrc/sparq_swar.h"

// out[4 * (a * 256 + b) + i] = byte i of trim4({a, b, b, a}) -- pairs (a,b) and (b,a).
extern "C" void swar_all_pairs(int n, unsigned S, int round_nearest, int pair, unsigned char* out) {
    const sparq::TrimLuts L = sparq::make_luts(n, S);
    for (unsigned a = 0; a < 256; ++a)
        for (unsigned b = 0; b < 256; ++b) {
            const uint32_t x = a | (b << 8) | (b << 16) | (a << 24);
            const uint32_t y = sparq::trim4_any(x, L, round_nearest != 0, pair != 0);
            for (int i = 0; i < 4; ++i) out[4 * (a * 256 + b) + i] = (unsigned char)(y >> (8 * i));
        }
}

// 2:4 groups of four: words[k] trimmed in partition j, in its byte order; out[0][j][k] from one pair of trims, out[1][j][k] by
// a trim of the reordered word.
extern "C" void swar_partitions(int n, unsigned S, int round_nearest, const uint32_t* words, int count, uint32_t* out) {
    using namespace sparq;
    const TrimLuts L = make_luts(n, S);
    for (int k = 0; k < count; ++k) {
        const uint32_t x = words[k];
        const auto beside = [&](uint32_t pm) {
            if (n == 4) return round_nearest ? trim4_round_n4_beside<true>(x, pm, L) : trim4_beside<false, true, false>(x, pm, L);
            return round_nearest ? trim4_beside<true, true, true>(x, pm, L) : trim4_beside<false, true, true>(x, pm, L);
        };
        const uint32_t full = beside(0xFFFFFFFFu), alone = beside(0u);
        for (int j = 0; j < 3; ++j) {
            out[j * count + k] = sparse24_choose(full, alone, sparse24_partner_flags(j), sparse24_pair_order(j));
            out[(3 + j) * count + k] = trim4_any(perm(0, x, sparse24_pair_order(j)), L, round_nearest != 0, true);
        }
    }
}
