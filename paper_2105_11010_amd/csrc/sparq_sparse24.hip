// 2:4 structured weight sparsity (Section 4, sparse tensor core; Section 5.3): the expansion that makes the
// pair-dependent trim an ordinary contraction, and the operand formats of the dense and the sparse matrix
// instruction for it.
//
// Of every four adjacent weights along the input channels an output channel keeps two, stored with their
// coordinates; the coordinates pick two of the four activations, and the picked two form that output channel's
// vSPARQ pair (Eq. 2).  The trim of an activation therefore depends on WHICH other activation the output channel
// picks with it -- but only through one bit: whether that partner is zero.  With
//     A(i|j) = x_i trimmed as the pair rule trims it beside x_j,
// a group of four input channels has twelve such values, in three words of two pairs each:
//     G_0 = A(0|1) A(1|0) A(2|3) A(3|2)    G_1 = A(0|2) A(2|0) A(1|3) A(3|1)    G_2 = A(0|3) A(3|0) A(1|2) A(2|1)
// -- G_j is the ordinary trim of the group's bytes brought into another order.  Whatever two positions an output
// channel keeps, both its values sit in one of the three words, so its two weights go to their two places there and
// zeros everywhere else: the plain-8-bit contraction over 3C channels is exactly the sparse, pair-trimmed dot product.
// (Three bytes per channel are also the least: the twelve values are independent of each other.)  Every expanded
// aligned group of four again holds two non-zeros or none, so the weights also go, as kept bytes plus positions, to
// the sparse matrix instruction (the SP form of the input-patch kernel).
// Blocked order (sparse24_blocked: C a multiple of 16 that wastes at most a fifth on whole 64-channel blocks): a block
// of 64 channels becomes three blocks of 64, all its G_0, all its G_1, all its G_2.  Then the SP kernel's staging
// wavefronts read the tensor itself and trim each block three times, in three byte orders, and no expanded tensor is
// written at all.  Otherwise the three words of a group follow each other.  Zero channels fill the pixel up to a multiple
// of 16, of 1x1 layers to whole units of the input-patch kernel (sparse24_channels).
// With vSPARQ off (or a plain 8-bit layer) nothing depends on the partner: the problem is the layer itself.
#include "sparq_common.h"
#include "sparq_fastdiv.h"

namespace sparq {

namespace {

constexpr int kSpThreads = 256;
typedef unsigned int v4u __attribute__((ext_vector_type(4)));
typedef v4u v4u_w __attribute__((aligned(4)));

int sp_grid(int64_t items) {
    int64_t blocks = (items + kSpThreads - 1) / kSpThreads;
    if (blocks > 256 * 16) blocks = 256 * 16;
    return (int)(blocks < 1 ? 1 : blocks);
}

// Word of the expanded pixel (or weight row) that holds G_j of group `grp`.
__device__ __forceinline__ int expanded_word(int grp, int j, bool blocked) {
    return blocked ? (grp >> 4) * 48 + j * 16 + (grp & 15) : 3 * grp + j;
}

// One lane per 16 bytes of an expanded pixel, so that every store instruction writes whole lines; the channels they come from are 16
// neighbouring ones (blocked order) or those of two neighbouring groups, read three times from L1.  Bound by memory: 401408 pixels of 160
// channels 88 -> 67 us (4.8 TB/s), of 12 16.5 -> 12.6 (a lane per group of channels with three four-byte stores and a 64-bit division before).
// groups: of four channels of x; chunks: 16-byte pieces of an expanded pixel (what lies past the groups' words: zeros).
template <int KIND, bool BLOCKED>
__global__ __launch_bounds__(kSpThreads) void expand_act_kernel(const uint32_t* __restrict__ x, uint4* __restrict__ xe,
                                                                 int64_t items, int groups, int chunks,
                                                                 FastDiv div_chunks, TrimLuts L) {
    const int64_t stride = (int64_t)gridDim.x * kSpThreads;
    for (int64_t i = (int64_t)blockIdx.x * kSpThreads + threadIdx.x; i < items; i += stride) {
        const int64_t pix = items < (1ll << 31) ? (int64_t)fastdiv((uint32_t)i, div_chunks) : i / chunks;
        const int q = (int)(i - pix * chunks);
        const uint32_t* src = x + pix * groups;
        uint32_t o[4] = {0, 0, 0, 0};
        if (BLOCKED) {
            const int blk = q / 12, part = q - 12 * blk, g0 = 16 * blk + 4 * (part & 3);     // (past groups: nothing)
            const uint32_t order = sparse24_pair_order(part >> 2);
            if (g0 < groups) {                               // C is a multiple of 16: all four groups exist
                const v4u_w v = *reinterpret_cast<const v4u_w*>(src + g0);
#pragma unroll
                for (int k = 0; k < 4; ++k) o[k] = trim4_kind<KIND>(perm(0, v[k], order), L);
            }
        } else {
            const int g0 = 4 * q / 3, j0 = 4 * q - 3 * g0;   // word 4q is G_j0 of group g0
            const uint32_t a = g0 < groups ? src[g0] : 0u, b = g0 + 1 < groups ? src[g0 + 1] : 0u;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const int j = j0 + k;
                o[k] = trim4_kind<KIND>(perm(0, j < 3 ? a : b, sparse24_pair_order(j < 3 ? j : j - 3)), L);
            }
        }
        xe[i] = make_uint4(o[0], o[1], o[2], o[3]);
    }
}

template <int KIND>
void launch_expand_act(bool blocked, const uint8_t* x, uint8_t* xe, int64_t items, int groups, int chunks, const TrimLuts& L, hipStream_t s) {
    const auto kernel = blocked ? expand_act_kernel<KIND, true> : expand_act_kernel<KIND, false>;
    kernel<<<sp_grid(items), kSpThreads, 0, s>>>(reinterpret_cast<const uint32_t*>(x), reinterpret_cast<uint4*>(xe), items, groups,
                                                 chunks, make_fastdiv((uint32_t)chunks), L);
}

// One lane per (output channel, tap, group): two kept weights and their coordinates -> a dense group.
// EXPAND: three words, the weights at the places of their pair (words_out per tap, groups past `groups` are zeros);
// otherwise the four bytes of the decompressed group.
template <bool EXPAND>
__global__ __launch_bounds__(kSpThreads) void expand_weights_kernel(const int8_t* __restrict__ vals, const uint8_t* __restrict__ idx,
                                                                     uint32_t* __restrict__ dense, int64_t items, int groups,
                                                                     int groups_out, int words_out, int blocked) {
    const int64_t stride = (int64_t)gridDim.x * kSpThreads;
    for (int64_t i = (int64_t)blockIdx.x * kSpThreads + threadIdx.x; i < items; i += stride) {
        const int64_t tap = i / groups_out;
        const int grp = (int)(i - tap * groups_out);
        uint32_t w0 = 0, w1 = 0;
        int i0 = 0, i1 = 0;
        if (grp < groups) {
            const int64_t s = tap * groups + grp;
            w0 = (uint8_t)vals[2 * s]; w1 = (uint8_t)vals[2 * s + 1];
            i0 = idx[2 * s] & 3; i1 = idx[2 * s + 1] & 3;                         // (coordinates are a precondition; masked for safety)
        }
        if (EXPAND) {
            uint32_t* dst = dense + tap * words_out;
            const int word = (i0 ^ i1) - 1;                                       // which of G_0..G_2 holds the pair
            // place of channel i inside G_j: nibble i of the table
            const uint32_t place = word == 0 ? 0x3210u : word == 1 ? 0x3120u : 0x1320u;
            const uint32_t o = (w0 << (8 * ((place >> (4 * i0)) & 3))) | (w1 << (8 * ((place >> (4 * i1)) & 3)));
#pragma unroll
            for (int j = 0; j < 3; ++j) dst[expanded_word(grp, j, blocked != 0)] = j == word ? o : 0u;
            for (int k = 3 * groups_out + grp; k < words_out; k += groups_out) dst[k] = 0u;
        } else {
            dense[i] = (w0 << (8 * i0)) | (w1 << (8 * i1));
        }
    }
}

// Operands of the sparse matrix instruction from dense weights w[N][taps][C] that hold at most two non-zeros in
// every aligned group of four channels (the expanded groups above do, and so do decompressed 2:4 weights).
// One lane per (64-index reduction step, half h, output channel n < Np): the 32 weights w[n][step*64 + 32h ..]
// -- taps padded to Cq channels, as in the dense packed tiles -- become 16 kept bytes (two per group of four, in
// position order) and one word of positions (bits [4g+1:4g] and [4g+3:4g+2] for group g, first < second, which
// is the layout v_smfmac_i32_32x32x64_i8 reads from lane (n % 32, h)).  Groups with fewer than two non-zeros keep
// zeros at unused positions.  vals[step][h][Np][16], pos[step][h][Np].
__global__ __launch_bounds__(kSpThreads) void pack_sparse_operand_kernel(const int8_t* __restrict__ w, uint4* __restrict__ vals,
                                                                          uint32_t* __restrict__ pos, int N, int Np, int taps,
                                                                          int C, int Cq, int64_t items) {
    const int64_t stride = (int64_t)gridDim.x * kSpThreads;
    const int steps_tap = Cq / 64;
    for (int64_t it = (int64_t)blockIdx.x * kSpThreads + threadIdx.x; it < items; it += stride) {
        const int n = (int)(it % Np);
        const int64_t sh = it / Np;
        const int h = (int)(sh & 1);
        const int64_t step = sh >> 1;
        const int tap = (int)(step / steps_tap);
        const int c0 = (int)(step % steps_tap) * 64 + 32 * h;
        uint32_t out[4] = {0, 0, 0, 0}, word = 0;
#pragma unroll
        for (int g = 0; g < 8; ++g) {
            const int c = c0 + 4 * g;
            uint32_t v = 0;
            if (n < N && c < C) v = *reinterpret_cast<const uint32_t*>(w + ((int64_t)n * taps + tap) * C + c);   // C % 4 == 0
            int p0 = -1, p1 = -1;
#pragma unroll
            for (int k = 0; k < 4; ++k)
                if ((v >> (8 * k)) & 255u) { if (p0 < 0) p0 = k; else if (p1 < 0) p1 = k; }
            if (p0 < 0) { p0 = 0; p1 = 1; }
            else if (p1 < 0) { if (p0 == 3) { p1 = 3; p0 = 2; } else p1 = 3; }
            const uint32_t b0 = (v >> (8 * p0)) & 255u, b1 = (v >> (8 * p1)) & 255u;
            const int e = 2 * g;
            out[e >> 2] |= (b0 << (8 * (e & 3))) | (b1 << (8 * ((e + 1) & 3)));
            word |= (uint32_t)(p0 | (p1 << 2)) << (4 * g);
        }
        vals[it] = make_uint4(out[0], out[1], out[2], out[3]);
        pos[it] = word;
    }
}

}  // namespace

sparq_status launch_sparse24_pack_operand(const int8_t* dense, uint8_t* vals, uint32_t* pos, int N, int Np, int taps, int C,
                                          int Cq, hipStream_t s) {
    const int64_t items = (int64_t)taps * (Cq / 64) * 2 * Np;
    if (items == 0) return SPARQ_OK;
    pack_sparse_operand_kernel<<<sp_grid(items), kSpThreads, 0, s>>>(dense, reinterpret_cast<uint4*>(vals), pos, N, Np, taps, C, Cq, items);
    return launch_status();
}

sparq_status launch_sparse24_expand_act(const uint8_t* x, uint8_t* xe, int64_t pixels, int C, int Ce, const sparq_mode* mode,
                                        hipStream_t s) {
    const bool blocked = sparse24_blocked(C);
    const int chunks = Ce / 16;
    const int64_t items = pixels * chunks;
    if (items == 0) return SPARQ_OK;
    const TrimLuts L = make_luts(mode->window_bits, mode->shift_mask);
    switch (trim_kind(mode)) {
        case kTrimFloorPair: launch_expand_act<kTrimFloorPair>(blocked, x, xe, items, C / 4, chunks, L, s); break;
        case kTrimFloorPairWide: launch_expand_act<kTrimFloorPairWide>(blocked, x, xe, items, C / 4, chunks, L, s); break;
        case kTrimRoundPairWide: launch_expand_act<kTrimRoundPairWide>(blocked, x, xe, items, C / 4, chunks, L, s); break;
        case kTrimRoundPair4: launch_expand_act<kTrimRoundPair4>(blocked, x, xe, items, C / 4, chunks, L, s); break;
        default: return SPARQ_EINVAL;                        // (only modes that pair are expanded)
    }
    return launch_status();
}

sparq_status launch_sparse24_expand_weights(const int8_t* vals, const uint8_t* idx, int8_t* dense, int64_t rows, int C, int Ce,
                                            hipStream_t s) {
    const bool expand = Ce != C;                             // (at least three expanded channels per channel)
    const bool blocked = expand && sparse24_blocked(C);
    const int groups_out = blocked ? (int)round_up(C, 64) / 4 : C / 4;
    const int64_t items = rows * groups_out;
    if (items == 0) return SPARQ_OK;
    uint32_t* d = reinterpret_cast<uint32_t*>(dense);
    if (expand)
        expand_weights_kernel<true><<<sp_grid(items), kSpThreads, 0, s>>>(vals, idx, d, items, C / 4, groups_out,
                                                                         Ce / 4, blocked ? 1 : 0);
    else
        expand_weights_kernel<false><<<sp_grid(items), kSpThreads, 0, s>>>(vals, idx, d, items, C / 4, groups_out, C / 4, 0);
    return launch_status();
}

}  // namespace sparq
