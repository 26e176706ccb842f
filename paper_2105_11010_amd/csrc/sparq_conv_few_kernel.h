// Fused SPARQ convolution for gfx950, layers of at most four channels (a network's first convolution).
//
// The reduction of one filter row is a run of neighbouring pixels: with every pixel as one word of four channels, the
// KW pixels of a row that an output needs are at most eight words from a multiple of four on, i.e. the 32 reduction
// indices of one matrix instruction.  A workgroup stages the input pixels of its tile in LDS as such words (trimmed, one
// barrier), keeps the weights of all filter rows in registers, and every fragment is one 16-byte LDS read at a multiple of
// the pixel's word: no copy of the input with padded channels, no multiplications for channels padded to 16.
// Weights: output class 0 of the pixel-folded layout (ConvGeom::fold), whose super-pixel taps 0 and 1 are exactly
// those eight words.
// Workgroups are persistent, two per CU: while a tile is multiplied the next one's pixels are on their way.
// Bound by memory (four-byte results: 5.3 TB/s) or, for bytes, by vector issue (55 % of the cycles by the counters, matrix pipeline 31;
// three instructions per result beside 14 matrix instructions per 32 pixels) and the staging (38 % of a wavefront's life in waits).  7x7/2, 224 x 224 x 3 -> 64, us, pixel-folded gather kernel with its padded copy -> now:
// 256 images, bytes 182 -> 79 (memory alone 49), fp32 204 -> 156; 32 images 30 -> 17, fp32 30 -> 23; one image 9.0 -> 5.0.
// 64 shapes of 32 to 384 outputs: 1.59 x.  Tried: one tile per workgroup (124, and 85 at best with its largest tile: the weights and
// constants are 120 registers to fill); three workgroups per CU (spills, 94); fragments of a strided layer as one 16-byte LDS read at
// 8-byte alignment instead of two of 8 bytes (124 against 85).
#pragma once
#include "sparq_conv_patch_kernel.h"
#include "sparq_fastdiv.h"

namespace sparq {

struct FewParams {
    const uint8_t* x;        // activations, NHWC
    const uint8_t* wpk;      // packed weight tiles (pixel-folded)
    const int32_t* colsum;   // sum_k w[n][k], Np entries
    int32_t* acc;            // [M][N] or null
    const float* scale;      // [N] or null
    float* out;              // [M][N] or null
    uint8_t* out_u8;         // [M][N] requantised output or null (then it is the only output; N a multiple of 16)
    uint32_t x_bytes, w_bytes;
    int M, N, Np;
    int B, H, W, Wo, Ho, KH, sh, sw, ph;
    int Hv;                  // virtual rows of an image: H + 2 ph
    int tm;                  // output pixels of a tile, a multiple of 128
    int tiles;
    int patch_bytes;         // LDS of one patch, of which there are two
    int taps_row;            // super-pixel taps of a filter row that class 0 uses: 1 or 2
    int taps_pitch;          // super-pixel taps of a filter row in the packed weights
    int group0;              // first group of four pixels that output column 0 needs, relative to the image (<= 0)
    int steps;               // matrix instructions along the reduction
    int kind;                // TrimKind
    FastDiv div_wo, div_ho, div_hv;
    TrimLuts luts;
};

constexpr int kFewThreads = 256, kFewTN = 64, kFewTurnPitch = kFewTN + 16;
constexpr int kFewLds = kLdsPerCu / 2;                          // of a workgroup: two share a CU
constexpr int kFewTurnBytes = 4 * 32 * kFewTurnPitch;        // a wavefront's 32 result rows on their way to whole lines

typedef v4i v4i_a4 __attribute__((aligned(4)));
typedef v4i v4i_a8 __attribute__((aligned(8)));

// Four pixels of C channels, one word each.
template <int C>
__device__ __forceinline__ v4u few_load(__amdgpu_buffer_rsrc_t rsrc, uint32_t off) {
    if constexpr (C == 4) {
        return __builtin_amdgcn_raw_buffer_load_b128(rsrc, (int)off, 0, 0);
    } else if constexpr (C == 3) {
        const auto w = __builtin_amdgcn_raw_buffer_load_b96(rsrc, (int)off, 0, 0);
        return v4u{(uint32_t)w[0], (uint32_t)w[1], (uint32_t)w[2], 0u};
    } else if constexpr (C == 2) {
        const auto w = __builtin_amdgcn_raw_buffer_load_b64(rsrc, (int)off, 0, 0);
        return v4u{(uint32_t)w[0], (uint32_t)w[1], 0u, 0u};
    } else {
        return v4u{(uint32_t)__builtin_amdgcn_raw_buffer_load_b32(rsrc, (int)off, 0, 0), 0u, 0u, 0u};
    }
}
template <int C>
__device__ __forceinline__ v4u few_spread(v4u w) {
    if constexpr (C == 3) return v4u{w[0] & 0xFFFFFFu, perm(w[1], w[0], 0x0C050403u), perm(w[2], w[1], 0x0C040302u), w[2] >> 8};
    else if constexpr (C == 2) return v4u{w[0] & 0xFFFFu, w[0] >> 16, w[1] & 0xFFFFu, w[1] >> 16};
    else if constexpr (C == 1) return v4u{w[0] & 0xFFu, (w[0] >> 8) & 0xFFu, (w[0] >> 16) & 0xFFu, w[0] >> 24};
    else return w;
}

struct FewOrigin { int v, col, row; };                       // virtual row, column (pixels right of output column 0's first), output row
__device__ __forceinline__ FewOrigin few_origin(const FewParams& p, int m) {
    const int r = (int)fastdiv((uint32_t)m, p.div_wo), ox = m - r * p.Wo;
    const int b = (int)fastdiv((uint32_t)r, p.div_ho), oy = r - b * p.Ho;
    return {b * p.Hv + oy * p.sh, ox * p.sw, r};
}

// EVEN: the stride along a row is 2 or 4, so that a fragment starts on 8 bytes.
template <int STEPS, int C, bool U8, bool EVEN>
__global__ __launch_bounds__(kFewThreads, 2) void conv_few_kernel(const FewParams p) {
    constexpr int FN = kFewTN / 32, CH = 4;                  // column fragments; patch chunks in flight per lane
    extern __shared__ __attribute__((aligned(16))) uint8_t lds[];            // [result rows of the four wavefronts | patch]
    const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, lhi = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n0 = (int)blockIdx.y * kFewTN;
    const __amdgpu_buffer_rsrc_t xrsrc =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t*>(p.x), 0, (int)p.x_bytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t wrsrc =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t*>(p.wpk), 0, (int)p.w_bytes, 0x00020000);

    // ---- a tile's input: rows x groups of four pixels ----
    struct Tile { int m0, rows, v0, g0, groups, chunks; float rcp_groups; };
    auto tile_at = [&](int tile) __attribute__((always_inline)) {
        Tile t;
        t.m0 = tile * p.tm;
        t.rows = p.M - t.m0 < p.tm ? p.M - t.m0 : p.tm;
        const FewOrigin first = few_origin(p, t.m0), last = few_origin(p, t.m0 + t.rows - 1);
        const bool one_row = first.row == last.row;
        t.v0 = first.v;
        t.g0 = one_row ? first.col >> 2 : 0;
        t.groups = (((one_row ? last.col : (p.Wo - 1) * p.sw) + 4 * p.taps_row - 1) >> 2) - t.g0 + 1;
        t.chunks = (last.v - first.v + p.KH) * t.groups;
        t.rcp_groups = 1.0f / (float)t.groups;
        return t;
    };
    v4u a_reg[CH];
    auto load_chunk = [&](const Tile& t, int i, int e) __attribute__((always_inline)) {
        int grp;
        const int vr = t.v0 + div_rcp(e, t.groups, t.rcp_groups, &grp);
        const int b = (int)fastdiv((uint32_t)vr, p.div_hv);
        const int iy = vr - b * p.Hv - p.ph, gx = t.g0 + grp + p.group0;
        const bool ok = (e < t.chunks) & (b < p.B) & ((unsigned)iy < (unsigned)p.H) & ((unsigned)gx < (unsigned)(p.W >> 2));
        const uint32_t off = (uint32_t)(((b * p.H + iy) * p.W + 4 * gx) * C);
        a_reg[i] = few_load<C>(xrsrc, ok ? off : kPatchInvalidOffset);
    };
    auto load_first = [&](const Tile& t) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < CH; ++i) load_chunk(t, i, tid + i * kFewThreads);
    };
    int tile = (int)blockIdx.x;
    Tile t = tile_at(tile);
    load_first(t);

    // ---- weights of all filter rows, per-channel constants ----
    v4i b[STEPS][FN];
#pragma unroll
    for (int j = 0; j < STEPS; ++j) {
        const int u = 2 * j + lhi, kh = u >> (p.taps_row - 1), tap = kh * p.taps_pitch + (u & (p.taps_row - 1));
#pragma unroll
        for (int k = 0; k < FN; ++k)
            b[j][k] = __builtin_bit_cast(v4i, __builtin_amdgcn_raw_buffer_load_b128(
                wrsrc, kh < p.KH ? (tap * p.Np + n0 + 32 * k + l32) * kChunk : (int)kPatchInvalidOffset, 0, 0));
    }
    typedef float v4f __attribute__((ext_vector_type(4)));
    v16i c0[FN];                                             // accumulators' initial value
    v4f fac[FN][4];
    int32_t corr[FN];
    float sc[FN];
    if constexpr (U8) {
        const __amdgpu_buffer_rsrc_t frsrc =
            __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(p.scale), 0, p.N * 4, 0x00020000);
#pragma unroll
        for (int k = 0; k < FN; ++k)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int n = n0 + 32 * k + 8 * q + 4 * lhi;
                const v4i s = *reinterpret_cast<const v4i*>(p.colsum + n);   // Np entries
                fac[k][q] = __builtin_bit_cast(v4f, __builtin_amdgcn_raw_buffer_load_b128(frsrc, n * 4, 0, 0));   // (past N: 0)
#pragma unroll
                for (int e = 0; e < 4; ++e) c0[k][4 * q + e] = s[e] * 128;
            }
    } else {
        const float* scale_or_dummy = p.out ? p.scale : reinterpret_cast<const float*>(p.colsum);
#pragma unroll
        for (int k = 0; k < FN; ++k) {
            const int n = n0 + 32 * k + l32, nc = n < p.N ? n : 0;
            corr[k] = p.colsum[nc] * 128;
            sc[k] = scale_or_dummy[nc];
#pragma unroll
            for (int v = 0; v < 16; ++v) c0[k][v] = 0;
        }
    }

    // ---- a patch into LDS ----
    auto stage_kind = [&](const Tile& t, uint8_t* patch, auto kind_) __attribute__((always_inline)) {
        for (int e0 = 0; e0 < t.chunks; e0 += CH * kFewThreads) {
#pragma unroll
            for (int i = 0; i < CH; ++i) {
                const int at = e0 + i * kFewThreads;
                if (at + wave * 64 < t.chunks) {             // uniform
                    v4u v = few_spread<C>(a_reg[i]);
#pragma unroll
                    for (int j = 0; j < 4; ++j) v[j] = trim4_kind<decltype(kind_)::value>(v[j], p.luts) ^ 0x80808080u;
                    if (at + tid < t.chunks) *reinterpret_cast<v4u*>(patch + (at + tid) * kChunk) = v;
                    if (at + CH * kFewThreads + wave * 64 < t.chunks) load_chunk(t, i, at + CH * kFewThreads + tid);
                }
            }
        }
    };
    auto stage = [&](const Tile& t, uint8_t* patch) __attribute__((always_inline)) {
#define SPARQ_FEW_STAGE(K) case K: stage_kind(t, patch, std::integral_constant<int, K>{}); break
        switch (p.kind) {
            SPARQ_FEW_STAGE(kTrimFloor);
            SPARQ_FEW_STAGE(kTrimFloorPair);
            SPARQ_FEW_STAGE(kTrimFloorPairWide);
            SPARQ_FEW_STAGE(kTrimRound);
            SPARQ_FEW_STAGE(kTrimRoundPairWide);
            SPARQ_FEW_STAGE(kTrimRound4);
            SPARQ_FEW_STAGE(kTrimRoundPair4);
            default: stage_kind(t, patch, std::integral_constant<int, kTrimNone>{}); break;
        }
#undef SPARQ_FEW_STAGE
    };
    uint8_t* patch = lds + (U8 ? kFewTurnBytes : 0);
    uint8_t* other = patch + p.patch_bytes;

    // ---- tiles: while one is multiplied, the next one's input is on its way ----
    for (;;) {
        stage(t, patch);
        __syncthreads();
        const int next = tile + (int)gridDim.x;
        Tile tn = t;
        if (next < p.tiles) {
            tn = tile_at(next);
            load_first(tn);
        }
        const int m0 = t.m0, rows = t.rows, g0 = t.g0;
        const int row_bytes = t.groups * kChunk;
        const int step_bytes = p.taps_row == 2 ? row_bytes : 2 * row_bytes;
        const int half = lhi * (p.taps_row == 2 ? kChunk : row_bytes);
        const size_t base = (size_t)m0 * p.N;
        for (int r0 = wave * 32; r0 < rows; r0 += 128) {
            const int m = r0 + l32 < rows ? m0 + r0 + l32 : m0 + rows - 1;
            const FewOrigin o = few_origin(p, m);
            const uint8_t* src = patch + (o.v - t.v0) * row_bytes + (o.col - 4 * g0) * 4 + half;
            int hi8 = 8;                                         // (opaque: the compiler would merge the halves into one slow misaligned read)
            if constexpr (EVEN) asm("" : "+v"(hi8));
            v4i a[STEPS];
#pragma unroll
            for (int j = 0; j < STEPS; ++j) {
                // (weights past the filter's last row are zero: any place inside the patch)
                const int off = (j < p.steps ? j : 0) * step_bytes;
                if constexpr (EVEN) {
                    typedef int v2i __attribute__((ext_vector_type(2)));
                    const v2i lo = *reinterpret_cast<const v2i*>(src + off), hi = *reinterpret_cast<const v2i*>(src + hi8 + off);
                    a[j] = v4i{lo[0], lo[1], hi[0], hi[1]};
                } else {
                    a[j] = *reinterpret_cast<const v4i_a4*>(src + off);
                }
            }
            v16i c[FN];
#pragma unroll
            for (int k = 0; k < FN; ++k) c[k] = c0[k];
#pragma unroll
            for (int j = 0; j < STEPS; ++j)
#pragma unroll
                for (int k = 0; k < FN; ++k)
                    c[k] = U8 ? __builtin_amdgcn_mfma_i32_32x32x32_i8(b[j][k], a[j], c[k], 0, 0, 0)
                              : __builtin_amdgcn_mfma_i32_32x32x32_i8(a[j], b[j][k], c[k], 0, 0, 0);
            if constexpr (U8) {
                uint8_t* const turn = lds + wave * 32 * kFewTurnPitch;
#pragma unroll
                for (int k = 0; k < FN; ++k) {
                    uint32_t w[4];
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        uint32_t r = __builtin_amdgcn_cvt_pk_u8_f32(__fmul_rn((float)c[k][4 * q], fac[k][q][0]), 0, 0);
                        r = __builtin_amdgcn_cvt_pk_u8_f32(__fmul_rn((float)c[k][4 * q + 1], fac[k][q][1]), 1, r);
                        r = __builtin_amdgcn_cvt_pk_u8_f32(__fmul_rn((float)c[k][4 * q + 2], fac[k][q][2]), 2, r);
                        w[q] = __builtin_amdgcn_cvt_pk_u8_f32(__fmul_rn((float)c[k][4 * q + 3], fac[k][q][3]), 3, r);
                    }
                    const auto s02 = __builtin_amdgcn_permlane32_swap(w[0], w[2], false, false);
                    const auto s13 = __builtin_amdgcn_permlane32_swap(w[1], w[3], false, false);
                    *reinterpret_cast<v4u*>(turn + l32 * kFewTurnPitch + k * 32 + 16 * lhi) = v4u{s02[0], s02[1], s13[0], s13[1]};
                }
                wavefront_lds_fence();
                const __amdgpu_buffer_rsrc_t orsrc =
                    __builtin_amdgcn_make_buffer_rsrc((void*)(p.out_u8 + base), 0, rows * p.N, 0x00020000);
                const int col = n0 + 16 * (lane & 3);
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const int row = 16 * h + (lane >> 2);
                    const v4u v = *reinterpret_cast<const v4u*>(turn + row * kFewTurnPitch + 16 * (lane & 3));
                    __builtin_amdgcn_raw_buffer_store_b128(v, orsrc, col < p.N ? (r0 + row) * p.N + col : (int)kPatchInvalidOffset, 0, 0);
                }
                wavefront_lds_fence();
            } else {
                const int pitch = p.N * 4, bytes = rows * pitch;
                const __amdgpu_buffer_rsrc_t arsrc =
                    __builtin_amdgcn_make_buffer_rsrc(p.acc ? (void*)(p.acc + base) : nullptr, 0, p.acc ? bytes : 0, 0x00020000);
                const __amdgpu_buffer_rsrc_t orsrc =
                    __builtin_amdgcn_make_buffer_rsrc(p.out ? (void*)(p.out + base) : nullptr, 0, p.out ? bytes : 0, 0x00020000);
                auto store = [&](auto acc_, auto out_) __attribute__((always_inline)) {
#pragma unroll
                    for (int v = 0; v < 16; ++v)
#pragma unroll
                        for (int k = 0; k < FN; ++k) {
                            const int n = n0 + 32 * k + l32, row = r0 + 8 * (v / 4) + 4 * lhi + v % 4;
                            const int off = n < p.N ? row * pitch + n * 4 : (int)kPatchInvalidOffset;
                            const int32_t r = c[k][v] + corr[k];
                            if constexpr (decltype(acc_)::value) __builtin_amdgcn_raw_buffer_store_b32(r, arsrc, off, 0, kResultStorePolicy);
                            if constexpr (decltype(out_)::value)
                                __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(int, __fmul_rn((float)r, sc[k])), orsrc, off, 0, kResultStorePolicy);
                        }
                };
                if (p.acc && p.out) store(std::true_type{}, std::true_type{});
                else if (p.out) store(std::false_type{}, std::true_type{});
                else store(std::true_type{}, std::false_type{});
            }
        }
        if (next >= p.tiles) break;
        tile = next;
        t = tn;
        uint8_t* const swap = patch;
        patch = other;
        other = swap;
    }
}

// Everything a launch needs of a pixel-folded layer; steps == 0: not for this kernel.
struct FewGeom { int taps_row, steps, tm, patch_bytes; };

// LDS of a tile of tm pixels: closed-form bound of its rows x groups (plus the row that the upper half of an odd last step
// reads beside zero weights).
inline int64_t few_patch_bytes(const ConvGeom& g, int taps_row, int tm) {
    int64_t d = (tm - 2) / g.Wo + 1;                         // output rows a tile spans, less one
    const int64_t rows_total = (int64_t)g.B * g.Ho;
    if (d > rows_total - 1) d = rows_total - 1;
    const int64_t hv = g.H + 2 * (int64_t)g.ph, gap = hv - (int64_t)g.Ho * g.sh > 0 ? hv - (int64_t)g.Ho * g.sh : 0;
    const int64_t crossings = (d + g.Ho - 1) / g.Ho < g.B - 1 ? (d + g.Ho - 1) / g.Ho : g.B - 1;
    const int64_t rows = d * g.sh + g.KH + crossings * gap + 1;
    const int64_t full = (((int64_t)(g.Wo - 1) * g.sw + 4 * taps_row - 1) >> 2) + 1;
    const int64_t single = (((int64_t)(tm - 1) * g.sw + 4 * taps_row + 2) >> 2) + 1;     // (starts anywhere inside its first group)
    return rows * (d > 0 ? full : single < full ? single : full) * kChunk;
}

// A tile's results are addressed in 32 bits, and kPatchInvalidOffset has to lie beyond them for a column past N to be dropped (as it
// has to lie beyond the weights for a row past the filter's last to read zeros).
inline bool few_addressable(int N, bool bytes, int tm) { return (int64_t)tm * N * (bytes ? 1 : 4) < 0x7FFFFFFF; }

inline FewGeom few_geom(const ConvGeom& g, bool bytes, int cus) {
    FewGeom f{};
    if (!g.fold || (bytes && g.N % 16)) return f;
    const int words = g.KW - g.pw - 4 * g.fold_kw_min;       // from a row's first word to its last tap's
    f.taps_row = (words + 3) / 4;
    const int steps = (g.KH * f.taps_row + 1) / 2;
    if (f.taps_row > 2 || steps > 8) return f;
    if (g.M > (1 << 30) || ((int64_t)g.B * g.H + 2 * (int64_t)g.B * g.ph) > (1 << 30) || g.N > (1 << 20) || (size_t)g.Kp * g.Np >= kPatchInvalidOffset) return f;
    // Four-byte results of many outputs beside a short reduction are bound by their stores, which the gather kernel's wider tiles make
    // in longer runs (3x3, 1.6 M pixels -> 192 / 256 / 384: 246 against 239 us, 316 against 295, 478 against 442; -> 128 167 against 173),
    // and up to 32 of them leave half of a 64-column tile empty (5x5, 262144 pixels -> 32: 15.1 against 13.4).
    if (!bytes && ((g.N > 128 && steps <= 3 && g.M * g.N * 4 >= kStreamedBytes) || (g.N <= 32 && steps > 3 && g.M > 64 * 1024))) return f;
    // Its folded rows of fold_p * N results are also whole 64-byte lines where the layer's own rows are not (`whole`), which counts for
    // more than its copy from 32 to 128 MiB of results on; where neither are, its longer runs do from 128 MiB on; and of few outputs it works out
    // four pixels' side by side where this kernel leaves nearly all of its columns empty.  1160 timed layers of 1 to 384 outputs, 20000 to 3 M
    // pixels: 248 of them go back to it by these lines, on which this kernel took 1.28 x its time (7x7, 259000 pixels -> 300 181 against
    // 76 us; 5x3, 752928 -> 108 203 against 86; 1x7, 631120 -> 5 28.6 against 17.0; 3x3, 196800 -> 14 even).
    if (!bytes && g.sw == 1 && g.M > 176 * 1024 && g.N <= (g.N % 4 ? 16 : 32)) return f;
    if (!bytes && g.N % 16 != 0 && g.sw < 4) {
        const bool whole = g.fold_p * g.N % 16 == 0;
        if ((whole || g.N > 64) && g.M * g.N * 4 >= ((int64_t)(!whole || g.N <= 64 ? 128 : g.sw == 1 ? 32 : 48) << 20)) return f;
    }
    const int64_t columns = (g.N + kFewTN - 1) / kFewTN;
    // The larger the tile, the fewer of its input rows belong to two tiles; smaller ones only while there are not 1.5 of them per CU
    // (three channels, 7x7, bytes: 3.2 M pixels 129 / 96 / 80 / 76 us at 128 / 256 / 512 / 1024 pixels, 12544 pixels 5.0 / 5.7 / 7.0 /
    // 10), or, for four-byte results, whose stores want many tiles in flight, 12 (401408 pixels 22 / 22 / 25 / 24; 3.2 M 175 / 167 / 159 / 144).
    for (int tm = 1024; tm >= 128; tm /= 2) {
        const int64_t patch_bytes = few_patch_bytes(g, f.taps_row, tm);
        if (!few_addressable(g.N, bytes, tm)) continue;
        if (2 * patch_bytes + (bytes ? kFewTurnBytes : 0) > kFewLds) continue;
        f.tm = tm;
        f.patch_bytes = (int)patch_bytes;
        f.steps = steps;
        if ((g.M + tm - 1) / tm * columns * 2 >= (bytes ? 3ll : 24ll) * cus) break;
    }
    return f;
}

template <int STEPS, int C, bool U8, bool EVEN>
sparq_status launch_few_cfg(const FewParams& p, hipStream_t s) {
    if (!few_addressable(p.N, U8, p.tm) || p.w_bytes >= kPatchInvalidOffset) return SPARQ_EUNSUPPORTED;
    const int columns = (p.N + kFewTN - 1) / kFewTN, slots = 2 * device_cu_count() / columns;
    const dim3 grid((unsigned)(p.tiles < slots ? p.tiles : slots > 0 ? slots : 1), (unsigned)columns);
    const int lds_bytes = (U8 ? kFewTurnBytes : 0) + 2 * p.patch_bytes;
    auto kern = conv_few_kernel<STEPS, C, U8, EVEN>;
    // largest dynamic LDS size enabled so far, per device (relaxed atomics: concurrent callers at worst repeat the call)
    static std::atomic<int> lds_set_dev[kMaxDevices];
    const int slot = current_device_slot();
    if (lds_bytes > lds_set_dev[slot].load(std::memory_order_relaxed) || slot == kMaxDevices - 1) {
        if (hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, lds_bytes) != hipSuccess)
            return SPARQ_ELAUNCH;
        lds_set_dev[slot].store(lds_bytes, std::memory_order_relaxed);
    }
    kern<<<grid, kFewThreads, lds_bytes, s>>>(p);
    return launch_status();
}
template <int STEPS, int C>
sparq_status launch_few_steps(const FewParams& p, hipStream_t s) {
    if (p.out_u8) return p.sw > 1 ? launch_few_cfg<STEPS, C, true, true>(p, s) : launch_few_cfg<STEPS, C, true, false>(p, s);
    return p.sw > 1 ? launch_few_cfg<STEPS, C, false, true>(p, s) : launch_few_cfg<STEPS, C, false, false>(p, s);
}
// (filters of 3, 5 and 7 rows with up to eight words a row; others run the next larger one beside zero weights)
template <int C>
sparq_status launch_few_channels(const FewParams& p, hipStream_t s) {
    if (p.steps <= 3) return launch_few_steps<3, C>(p, s);
    if (p.steps <= 5) return launch_few_steps<5, C>(p, s);
    if (p.steps <= 7) return launch_few_steps<7, C>(p, s);
    return launch_few_steps<8, C>(p, s);
}

sparq_status launch_few_c1(const FewParams& p, hipStream_t s);
sparq_status launch_few_c2(const FewParams& p, hipStream_t s);
sparq_status launch_few_c3(const FewParams& p, hipStream_t s);
sparq_status launch_few_c4(const FewParams& p, hipStream_t s);

}  // namespace sparq
