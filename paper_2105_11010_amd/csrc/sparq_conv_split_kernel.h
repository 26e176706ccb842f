// Fused SPARQ convolution for gfx950, small layers: a tile's reduction split over the wavefronts of one workgroup.
//
// A layer with few output tiles is bound by the length of its chain: in the input-patch kernel a tile walks its
// reduction unit by unit behind a barrier each, with four matrix wavefronts, on as many CUs as there are 128 x 64
// tiles (eight for a 7 x 7 image with 512 channels).  Here a tile is 32 or 64 output pixels x 32 or 64 channels, the
// patch of ALL input channels is staged in LDS at once (one barrier), the eight wavefronts share out the
// 32-index reduction steps, each reads its own weights straight from L2 (requested before the patch is staged;
// every weight byte enters a workgroup once), and the eight partial tiles are added up through LDS.  The sums leave LDS
// four channels at a time, so every output form is a vector store.
// Bound by latency: launch, patch from memory, one barrier, the steps, the sum, the stores (a launch that does nothing takes about
// 3 us), so what counts is how many instructions stand before the first request and between two matrix instructions: the
// tile's geometry is integer arithmetic in scalar registers, a lane's chunk of the patch two or three divisions by constants, the fragments'
// offset is carried along, and every wait for weights is for the oldest request only.  Launches replayed back to back as a graph, us,
// first form (pixels numbered through with float divisions, a loop that could end half way) -> now: 56 x 56 x 64 -> 64 3x3, one image,
// 5.4 -> 4.2; 14 x 14 x 256 -> 256 6.1 -> 5.0; 7 x 7 x 512 -> 512 7.2 -> 6.1 (32 images 13.6 -> 11.9); 1x1 7 x 7 x 2048 -> 512 9.0 -> 6.9
// (the tile kernels before it: 7.3 / 9.1 / 13.6 / 15.4, one call after the other).  1100 drawn layers 1.25 x on the first form, two below
// 0.95 x.  Twice the weights requested ahead: 0.6 us slower (the longer code is fetched once per launch).
#pragma once
#include "sparq_conv_patch_kernel.h"
#include "sparq_fastdiv.h"

namespace sparq {

struct SplitParams {
    const uint8_t* x;        // activations, NHWC, C a multiple of 4
    const uint8_t* wpk;      // packed weight tiles
    const int32_t* colsum;   // sum_k w[n][k], Np entries
    int32_t* acc;            // [M][N] or null
    const float* scale;      // [N] or null
    float* out;              // [M][N] or null
    uint8_t* out_u8;         // [M][N] requantised output or null (then it is the only output)
    int trim_out;            // out_u8 with N % 4 == 0 only: trim the requantised bytes with this launch's own mode
    int trim_in;             // 0: x is taken as it is
    uint32_t x_bytes, w_bytes;
    int N, Np, C;
    int planes;              // 16-channel planes of the patch: channels of a tap in the packed weights / 16
    int plane_stride;        // bytes between planes in LDS
    int steps;               // 32-index reduction steps
    int steps_tap;           // ... per filter tap
    int tiles_n;
    FastDiv div_planes, div_steps_tap, div_kw, div_wo, div_ho, div_hv, div_tiles_n;
    PatchGeom g;             // tm = the tile's output pixels
    TrimLuts luts;
};

constexpr int kSplitWaves = 8, kSplitThreads = 64 * kSplitWaves;

// FM x FN fragments of 32 x 32 per tile, every wavefront holds all of them; AHEAD: weight steps requested ahead.
template <int FM, int FN, int AHEAD>
struct SplitCfg {
    static constexpr int kFM = FM, kFN = FN, kAhead = AHEAD;
    static constexpr int kTM = 32 * FM, kTN = 32 * FN;
    static constexpr int kRowPitch = kTN * 4 + 16;           // LDS row of a partial tile, padded against bank conflicts
    static constexpr int kPartialBytes = kTM * kRowPitch;
    static constexpr int kQuads = kTM * kTN / 4;             // groups of four channels the epilogue hands out
};

inline int split_plane_stride(int npix_max) { return (int)round_up((int64_t)npix_max * kChunk, 256) + kChunk; }

// ONE_ROW: the input is one row (1x1 layers: PatchGeom's long row, of pixels of a strided layer where rm_wo is set).
template <class Cfg, int KIND, bool ONE_ROW>
__global__ __launch_bounds__(kSplitThreads, 2) void conv_split_kernel(const SplitParams p) {
    constexpr int FM = Cfg::kFM, FN = Cfg::kFN, D = Cfg::kAhead, TM = Cfg::kTM, TN = Cfg::kTN;
    constexpr int CH = 4;                                    // patch chunks in flight per lane
    typedef float v4f __attribute__((ext_vector_type(4)));
    extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
    const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, lhi = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const PatchGeom& g = p.g;
    const int tile_m = (int)fastdiv(blockIdx.x, p.div_tiles_n), tile_n = (int)blockIdx.x - tile_m * p.tiles_n;
    const int m0 = tile_m * TM, n0 = tile_n * TN;
    const __amdgpu_buffer_rsrc_t xrsrc =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t*>(p.x), 0, (int)p.x_bytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t wrsrc =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t*>(p.wpk), 0, (int)p.w_bytes, 0x00020000);

    // ---- the tile's patch (as tile_patch; in integers, so that it stays in scalar registers) ----
    const auto origin = [&](int m, int* row, int* x) __attribute__((always_inline)) {
        const int r = (int)fastdiv((uint32_t)m, p.div_wo), b = (int)fastdiv((uint32_t)r, p.div_ho);
        *row = r;
        *x = (m - r * g.Wo) * g.sw - g.pw;
        return b * g.Hv + (r - b * g.Ho) * g.sh;             // virtual row
    };
    int row0, row1, x0, x1;
    const int v0 = origin(m0, &row0, &x0), v1 = origin(m0 + TM < g.M ? m0 + TM - 1 : g.M - 1, &row1, &x1);
    const int xlo = row0 == row1 ? x0 : -g.pw;
    const int pwt = row0 == row1 ? x1 - x0 + g.KW : (g.Wo - 1) * g.sw + g.KW;
    const int nrows = v1 - v0 + g.KH;

    // ---- the patch: its 16-byte chunks numbered through, those of a row next to each other in memory; a wavefront takes 64 of them at a
    //      time, every eighth such piece.  A lane's address is two divisions by launch constants, one by the row's chunks and a few
    //      adds (while it was pixels that were numbered through, 250 instructions before the first request and 100 for each
    //      further one).  Row by row, with what depends on the row in scalar registers, each row's last piece is asked for whole: 1-3 %
    //      slower on the networks' layers, and 6.5 -> 21.3 us where rows are short (2 x 2 x 148 -> 608 7x1/2, 57 images) ----
    const int row_chunks = pwt * p.planes, chunks = nrows * row_chunks;
    const float rcp_row = ONE_ROW ? 0.0f : 1.0f / (float)row_chunks;
    int l_piece = wave;                                      // the piece requested next
    v4u a_reg[CH];
    int a_at[CH];                                            // where the chunk goes in LDS, -1: nowhere
    auto load_chunk = [&](int i) __attribute__((always_inline)) {
        const int at = l_piece * 64 + lane;
        const bool inside = at < chunks;
        PatchChunk k;
        int pix;
        bool ok = inside;
        if constexpr (ONE_ROW) {
            k = patch_chunk(at, p.planes, p.div_planes);
            pix = xlo + k.px;
            ok &= (unsigned)pix < (unsigned)g.W;
            if (g.rm_wo) pix = remap_pixel(g, ok ? pix : 0);
        } else {
            k = patch_chunk(at, row_chunks, rcp_row, p.planes, p.div_planes);
            const int vr = v0 + k.row, b = (int)fastdiv((uint32_t)vr, p.div_hv), iy = vr - b * g.Hv - g.ph, ix = xlo + k.px;
            ok &= (b < g.B) & ((unsigned)iy < (unsigned)g.H) & ((unsigned)ix < (unsigned)g.W);
            pix = (b * g.H + iy) * g.W + ix;
        }
        ok &= k.plane * kChunk < p.C;                        // a tap's channel padding reads as zero
        a_reg[i] = __builtin_amdgcn_raw_buffer_load_b128(xrsrc, ok ? pix * p.C + k.plane * kChunk : (int)kPatchInvalidOffset, 0, 0);
        a_at[i] = inside ? k.plane * p.plane_stride + (k.row * pwt + k.px) * kChunk : -1;
        l_piece += kSplitWaves;
    };
    auto stage_chunk = [&](int i) __attribute__((always_inline)) {
        v4u v = a_reg[i];
        if (KIND != kTrimNone && p.trim_in) {
#pragma unroll
            for (int j = 0; j < 4; ++j) v[j] = trim4_kind<KIND>(v[j], p.luts);
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) v[j] ^= 0x80808080u;
        if (a_at[i] >= 0) *reinterpret_cast<v4u*>(lds + a_at[i]) = v;
    };
    // first patch chunks, then the first weights: the patch waits for its own requests only.  (Requests under a uniform
    // condition: `left` counts the pieces of this wavefront.)
    const int total = patch_pieces(chunks);
    int left = total > wave ? (total - wave + kSplitWaves - 1) / kSplitWaves : 0;
#pragma unroll
    for (int i = 0; i < CH; ++i)
        if (i < left) load_chunk(i);

    // ---- this wavefront's share of the reduction steps ----
    const int h0 = p.steps * wave / kSplitWaves, h1 = p.steps * (wave + 1) / kSplitWaves;
    const int wlane = (lhi * p.Np + n0 + l32) * kChunk;
    v4i b_reg[D][FN];
    const int w_step = 2 * p.Np * kChunk, w_last = (h1 - 1) * w_step;
    int w_off = h0 * w_step;                                 // the step requested next
#pragma unroll
    for (int k = 0; k < D; ++k) {
        // past the share: outside the buffer (by the lane's part of the offset), not fetched
        const int voff = h0 + k < h1 ? wlane : (int)kPatchInvalidOffset, soff = h0 + k < h1 ? w_off : 0;
#pragma unroll
        for (int j = 0; j < FN; ++j)
            b_reg[k][j] = __builtin_bit_cast(v4i, __builtin_amdgcn_raw_buffer_load_b128(wrsrc, voff + j * 32 * kChunk, soff, 0));
        w_off += w_step;
    }
    auto load_b = [&](v4i (&b)[FN]) __attribute__((always_inline)) {
        const int soff = w_off < w_last ? w_off : w_last;    // past the share: the last step's once more, from L1
#pragma unroll
        for (int j = 0; j < FN; ++j)
            b[j] = __builtin_bit_cast(v4i, __builtin_amdgcn_raw_buffer_load_b128(wrsrc, wlane + j * 32 * kChunk, soff, 0));
        w_off += w_step;
    };

    // per-channel constants of the epilogue: group q of this lane is channels n0 + 4 * (q % (TN / 4)) .. + 3 for every q
    static_assert(kSplitThreads % (TN / 4) == 0, "a lane's groups share their channels");
    const int en = n0 + 4 * (tid % (TN / 4));
    const bool scaled = p.out || p.out_u8;
    const __amdgpu_buffer_rsrc_t frsrc =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(p.scale), 0, scaled ? p.N * 4 : 0, 0x00020000);     // (past N: 0)
    const v4i colsum4 = *reinterpret_cast<const v4i*>(p.colsum + en);        // Np entries
    const v4u scale4 = __builtin_amdgcn_raw_buffer_load_b128(frsrc, en * 4, 0, 0);
    __builtin_amdgcn_sched_barrier(0);

    // where the fragments of the first step lie: worked out while the requests are on their way
    int32_t fbase[FM];
#pragma unroll
    for (int i = 0; i < FM; ++i) {
        int m = m0 + i * 32 + l32, row, x;
        m = m < g.M ? m : g.M - 1;
        const int v = origin(m, &row, &x);
        fbase[i] = ((v - v0) * pwt + (x - xlo)) * kChunk + lhi * p.plane_stride;
    }
    const int tap0 = (int)fastdiv((uint32_t)h0, p.div_steps_tap);
    const int kh0 = (int)fastdiv((uint32_t)tap0, p.div_kw), kw0 = tap0 - kh0 * g.KW, c0 = h0 - tap0 * p.steps_tap;
    // patch offset of the step whose fragments are read next, steps left in its tap and taps left in its row.  (One step past the last
    // the offset is a row further: other planes of the patch, not used.)
    const int c_step = 2 * p.plane_stride, tap_step = kChunk - p.steps_tap * c_step, row_step = (pwt - g.KW) * kChunk;
    int f_off = c0 * c_step + (kh0 * pwt + kw0) * kChunk, f_c = p.steps_tap - c0, f_kw = g.KW - kw0;
#pragma unroll
    for (int i = 0; i < FM; ++i) asm volatile("" : "+v"(fbase[i]));

    // ---- the whole patch into LDS (the first round apart: in the loop a wait could not tell the patch from the weights) ----
    auto stage_round = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < CH; ++i)
            if (i < left) {                                  // uniform
                stage_chunk(i);
                if (i + CH < left) load_chunk(i);
            }
        left -= CH;
    };
    stage_round();
    while (left > 0) stage_round();
    __syncthreads();

    // ---- multiply ----
    v16i c[FM][FN];
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) c[i][j][v] = 0;
    v4i af[2][FM];
    auto load_frags = [&](v4i (&a)[FM]) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < FM; ++i) a[i] = *reinterpret_cast<const v4i*>(lds + fbase[i] + f_off);
        f_off += c_step;
        if (--f_c == 0) {
            f_c = p.steps_tap;
            f_off += tap_step;
            if (--f_kw == 0) {
                f_kw = g.KW;
                f_off += row_step;
            }
        }
    };
    load_frags(af[0]);
    static_assert(D % 2 == 0, "fragment slots alternate");
    // weights as the row operand: a lane ends up with channels 8 * (v / 4) + 4 * lhi + v % 4 of pixel l32
    auto multiply = [&](int k) __attribute__((always_inline)) {
        load_frags(af[(k + 1) & 1]);
#pragma unroll
        for (int i = 0; i < FM; ++i)
#pragma unroll
            for (int j = 0; j < FN; ++j) c[i][j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(b_reg[k][j], af[k & 1][i], c[i][j], 0, 0, 0);
    };
    // whole rounds of D steps, then the rest apart: a round left half way would meet the loop's start with its requests in
    // another order, and the compiler would wait there for all of them
    int h = h0;
    for (; h + D <= h1; h += D) {
#pragma unroll
        for (int k = 0; k < D; ++k) {
            multiply(k);
            load_b(b_reg[k]);
        }
    }
    const int rest = h1 - h;
#pragma unroll
    for (int k = 0; k < D - 1; ++k) {
        if (k >= rest) break;                                // uniform
        multiply(k);
    }
    __syncthreads();                                         // the patch is not read any more

    // ---- add the eight partial tiles up ----
    uint8_t* mine = lds + wave * Cfg::kPartialBytes + l32 * Cfg::kRowPitch + 16 * lhi;
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const v4i r = {c[i][j][4 * q], c[i][j][4 * q + 1], c[i][j][4 * q + 2], c[i][j][4 * q + 3]};
                *reinterpret_cast<v4i*>(mine + i * 32 * Cfg::kRowPitch + (j * 32 + 8 * q) * 4) = r;
            }
    __syncthreads();
#pragma unroll
    for (int q0 = 0; q0 < Cfg::kQuads; q0 += kSplitThreads) {
        const int q = q0 + tid;
        if (q >= Cfg::kQuads) break;
        const int row = q / (TN / 4);
        const uint8_t* src = lds + row * Cfg::kRowPitch + (tid % (TN / 4)) * 16;
        v4i r = *reinterpret_cast<const v4i*>(src);
#pragma unroll
        for (int w = 1; w < kSplitWaves; ++w) r += *reinterpret_cast<const v4i*>(src + w * Cfg::kPartialBytes);
#pragma unroll
        for (int e = 0; e < 4; ++e) r[e] += colsum4[e] * 128;
        const int m = m0 + row;
        if (m >= g.M || en >= p.N) continue;
        const size_t at = (size_t)m * p.N + en;
        const bool whole = (p.N & 3) == 0;                   // then the four channels are inside N together and aligned
        if (p.out_u8) {
            const auto sc = __builtin_bit_cast(v4f, scale4);
            uint32_t w = requant_u8(r[0], sc[0]) | (requant_u8(r[1], sc[1]) << 8) | (requant_u8(r[2], sc[2]) << 16) |
                         (requant_u8(r[3], sc[3]) << 24);
            if (whole) {
                if (KIND != kTrimNone && p.trim_out) w = trim4_kind<KIND>(w, p.luts);
                *reinterpret_cast<uint32_t*>(p.out_u8 + at) = w;
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (en + e < p.N) p.out_u8[at + e] = (uint8_t)(w >> (8 * e));
            }
            continue;
        }
        if (p.acc) {
            if (whole) {
                *reinterpret_cast<v4i*>(p.acc + at) = r;
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (en + e < p.N) p.acc[at + e] = r[e];
            }
        }
        if (p.out) {
            const auto sc = __builtin_bit_cast(v4f, scale4);
            v4f f;
#pragma unroll
            for (int e = 0; e < 4; ++e) f[e] = __fmul_rn((float)r[e], sc[e]);
            if (whole) {
                *reinterpret_cast<v4f*>(p.out + at) = f;
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (en + e < p.N) p.out[at + e] = f[e];
            }
        }
    }
}

// LDS of a launch: the patch, then the partial tiles in the same place.
template <class Cfg>
int split_lds_bytes(int npix_max, int planes) {
    const int64_t patch = (int64_t)planes * split_plane_stride(npix_max), partials = (int64_t)kSplitWaves * Cfg::kPartialBytes;
    const int64_t need = patch > partials ? patch : partials;
    return need > kLdsPerCu ? -1 : (int)need;
}

// `p` carries everything except plane_stride and tiles_n; npix_max bounds TilePatch::npix.
template <class Cfg, int KIND, bool ONE_ROW>
sparq_status launch_split_rows(const SplitParams& p, int npix_max, hipStream_t s) {
    SplitParams q = p;
    q.plane_stride = split_plane_stride(npix_max);
    const int lds_bytes = split_lds_bytes<Cfg>(npix_max, p.planes);
    if (lds_bytes < 0 || p.g.tm != Cfg::kTM) return SPARQ_EUNSUPPORTED;
    q.tiles_n = (p.N + Cfg::kTN - 1) / Cfg::kTN;
    q.div_tiles_n = make_fastdiv((uint32_t)q.tiles_n);
    const int64_t tiles = (int64_t)((p.g.M + Cfg::kTM - 1) / Cfg::kTM) * q.tiles_n;
    if (tiles > 0x7FFFFFFF) return SPARQ_EUNSUPPORTED;
    auto kern = conv_split_kernel<Cfg, KIND, ONE_ROW>;
    // largest dynamic LDS size enabled so far, per device (relaxed atomics: concurrent callers at worst repeat the call)
    static std::atomic<int> lds_set_dev[kMaxDevices];
    const int slot = current_device_slot();
    if (lds_bytes > lds_set_dev[slot].load(std::memory_order_relaxed) || slot == kMaxDevices - 1) {
        if (hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize,
                                lds_bytes) != hipSuccess)
            return SPARQ_ELAUNCH;
        lds_set_dev[slot].store(lds_bytes, std::memory_order_relaxed);
    }
    kern<<<(unsigned)tiles, kSplitThreads, lds_bytes, s>>>(q);
    return launch_status();
}

template <class Cfg, int KIND>
sparq_status launch_split_cfg(const SplitParams& p, int npix_max, hipStream_t s) {
    const bool one_row = p.g.B == 1 && p.g.H == 1 && p.g.ph == 0;
    return one_row ? launch_split_rows<Cfg, KIND, true>(p, npix_max, s) : launch_split_rows<Cfg, KIND, false>(p, npix_max, s);
}

template <class Cfg>
sparq_status launch_split_kind(TrimKind kind, const SplitParams& p, int npix_max, hipStream_t s) {
    switch (kind) {
        case kTrimNone: return launch_split_cfg<Cfg, kTrimNone>(p, npix_max, s);
        case kTrimFloor: return launch_split_cfg<Cfg, kTrimFloor>(p, npix_max, s);
        case kTrimFloorPair: return launch_split_cfg<Cfg, kTrimFloorPair>(p, npix_max, s);
        case kTrimFloorPairWide: return launch_split_cfg<Cfg, kTrimFloorPairWide>(p, npix_max, s);
        case kTrimRound: return launch_split_cfg<Cfg, kTrimRound>(p, npix_max, s);
        case kTrimRound4: return launch_split_cfg<Cfg, kTrimRound4>(p, npix_max, s);
        case kTrimRoundPairWide: return launch_split_cfg<Cfg, kTrimRoundPairWide>(p, npix_max, s);
        case kTrimRoundPair4: return launch_split_cfg<Cfg, kTrimRoundPair4>(p, npix_max, s);
        default: return SPARQ_EUNSUPPORTED;
    }
}

typedef SplitCfg<1, 1, 8> Split32x32;
typedef SplitCfg<1, 2, 6> Split32x64;
typedef SplitCfg<2, 2, 4> Split64x64;
typedef sparq_status (*SplitLauncher)(TrimKind, const SplitParams&, int, hipStream_t);
sparq_status launch_split_32x32(TrimKind kind, const SplitParams& p, int npix_max, hipStream_t s);
sparq_status launch_split_32x64(TrimKind kind, const SplitParams& p, int npix_max, hipStream_t s);
sparq_status launch_split_64x64(TrimKind kind, const SplitParams& p, int npix_max, hipStream_t s);

}  // namespace sparq
