// Fused SPARQ convolution for gfx950, small layers: a tile's reduction split over the wavefronts of one workgroup.
//
// A layer with few output tiles is bound by the length of its chain: in the input-patch kernel a tile walks its
// reduction unit by unit behind a barrier each, with four matrix wavefronts, on as many CUs as there are 128 x 64
// tiles (eight for a 7 x 7 image with 512 channels).  Here a tile is 32 or 64 output pixels x 32 or 64 channels, the
// patch of ALL input channels is staged in LDS at once (one barrier), the eight wavefronts share out the
// 32-index reduction steps, each reads its own weights straight from L2 (requested before the patch is staged;
// every weight byte enters a workgroup once), and the eight partial tiles are added up through LDS.  The sums leave LDS
// four channels at a time, so every output form is a vector store.
// Bound by latency: launch, patch from memory, one barrier, the steps, the sum, the stores (5.2 us with nothing to reduce,
// of which a launch that does nothing takes about 3).  Back to back on one stream, before -> now: 56 x 56 x 64 -> 64 3x3,
// one image, 7.3 -> 5.5 us; 14 x 14 x 256 -> 256 9.1 -> 5.9; 7 x 7 x 512 -> 512 13.6 -> 6.8 (32 images 15.4 -> 12.9).
#pragma once
#include "sparq_conv_patch_kernel.h"
#include "sparq_fastdiv.h"

namespace sparq {

struct SplitParams {
    const uint8_t* x;        // activations, NHWC, C a multiple of 16
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
    FastDiv div_planes, div_steps_tap, div_kw;
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

template <class Cfg, int KIND>
__global__ __launch_bounds__(kSplitThreads, 2) void conv_split_kernel(const SplitParams p) {
    constexpr int FM = Cfg::kFM, FN = Cfg::kFN, D = Cfg::kAhead, TM = Cfg::kTM, TN = Cfg::kTN;
    constexpr int CH = 4;                                    // patch chunks in flight per lane
    extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
    const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, lhi = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const PatchGeom& g = p.g;
    const int tile_m = (int)blockIdx.x / p.tiles_n, tile_n = (int)blockIdx.x - tile_m * p.tiles_n;
    const int m0 = tile_m * TM, n0 = tile_n * TN;
    const __amdgpu_buffer_rsrc_t xrsrc =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t*>(p.x), 0, (int)p.x_bytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t wrsrc =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t*>(p.wpk), 0, (int)p.w_bytes, 0x00020000);

    const TilePatch t = tile_patch(g, m0);
    const int chunks = t.npix * p.planes;
    v4u a_reg[CH];
    auto load_chunk = [&](int i, int e) __attribute__((always_inline)) {
        const int pix = (int)fastdiv((uint32_t)e, p.div_planes);
        const int ch = (e - pix * p.planes) * kChunk;
        uint32_t off = patch_pixel_offset_u32(g, t, pix, p.C, kPatchInvalidOffset);
        off = ch < p.C ? off : kPatchInvalidOffset;          // a tap's channel padding reads as zero
        off += off != kPatchInvalidOffset ? (uint32_t)ch : 0u;
        a_reg[i] = __builtin_amdgcn_raw_buffer_load_b128(xrsrc, (int)off, 0, 0);
    };
    auto stage_chunk = [&](int i, int e) __attribute__((always_inline)) {
        v4u v = a_reg[i];
        if (KIND != kTrimNone && p.trim_in) {
#pragma unroll
            for (int j = 0; j < 4; ++j) v[j] = trim4_kind<KIND>(v[j], p.luts);
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) v[j] ^= 0x80808080u;
        const int pix = (int)fastdiv((uint32_t)e, p.div_planes);
        if (e < chunks) *reinterpret_cast<v4u*>(lds + (e - pix * p.planes) * p.plane_stride + pix * kChunk) = v;
    };
    // first patch chunks, then the first weights: the patch waits for its own requests only
#pragma unroll
    for (int i = 0; i < CH; ++i) load_chunk(i, tid + i * kSplitThreads);

    // ---- this wavefront's share of the reduction steps ----
    const int h0 = p.steps * wave / kSplitWaves, h1 = p.steps * (wave + 1) / kSplitWaves;
    const int wlane = (lhi * p.Np + n0 + l32) * kChunk;
    v4i b_reg[D][FN];
    auto load_b = [&](v4i (&b)[FN], int h) __attribute__((always_inline)) {
        // past the share: outside the buffer (by the lane's part of the offset), not fetched
        const int voff = h < h1 ? wlane : (int)kPatchInvalidOffset, soff = h < h1 ? h * 2 * p.Np * kChunk : 0;
#pragma unroll
        for (int j = 0; j < FN; ++j)
            b[j] = __builtin_bit_cast(v4i, __builtin_amdgcn_raw_buffer_load_b128(wrsrc, voff + j * 32 * kChunk, soff, 0));
    };
#pragma unroll
    for (int k = 0; k < D; ++k) load_b(b_reg[k], h0 + k);

    // per-channel constants of the epilogue: group q of this lane is channels n0 + 4 * (q % (TN / 4)) .. + 3 for every q
    static_assert(kSplitThreads % (TN / 4) == 0, "a lane's groups share their channels");
    const int en = n0 + 4 * (tid % (TN / 4));
    int32_t corr[4];
    float sc[4];
    const float* scale_or_dummy = (p.out || p.out_u8) ? p.scale : reinterpret_cast<const float*>(p.colsum);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const int nc = en + e < p.N ? en + e : 0;
        corr[e] = p.colsum[nc] * 128;
        sc[e] = scale_or_dummy[nc];
    }
    __builtin_amdgcn_sched_barrier(0);

    // ---- the whole patch into LDS ----
    for (int e0 = 0; e0 < chunks; e0 += CH * kSplitThreads) {
#pragma unroll
        for (int i = 0; i < CH; ++i)
            if (e0 + i * kSplitThreads + wave * 64 < chunks) {       // uniform
                stage_chunk(i, e0 + tid + i * kSplitThreads);
                const int next = e0 + (CH + i) * kSplitThreads;
                if (next + wave * 64 < chunks) load_chunk(i, next + tid);
            }
    }
    __syncthreads();

    // ---- multiply ----
    int32_t fbase[FM];
#pragma unroll
    for (int i = 0; i < FM; ++i) {
        int m = m0 + i * 32 + l32;
        m = m < g.M ? m : g.M - 1;
        fbase[i] = patch_pixel_of_output(g, t, m) * kChunk + lhi * p.plane_stride;
    }
    const int tap0 = (int)fastdiv((uint32_t)h0, p.div_steps_tap);
    int f_c = h0 - tap0 * p.steps_tap;
    int f_kh = (int)fastdiv((uint32_t)tap0, p.div_kw);
    int f_kw = tap0 - f_kh * g.KW;
    auto frag_offset = [&]() __attribute__((always_inline)) {
        return f_c * 2 * p.plane_stride + (f_kh * t.pwt + f_kw) * kChunk;
    };
    auto advance = [&]() __attribute__((always_inline)) {
        if (++f_c == p.steps_tap) {
            f_c = 0;
            if (++f_kw == g.KW) {
                f_kw = 0;
                if (++f_kh == g.KH) f_kh = 0;                // past the last step: any place inside the patch
            }
        }
    };
    v16i c[FM][FN];
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) c[i][j][v] = 0;
    v4i af[2][FM];
    auto load_frags = [&](v4i (&a)[FM]) __attribute__((always_inline)) {
        const int off = frag_offset();
#pragma unroll
        for (int i = 0; i < FM; ++i) a[i] = *reinterpret_cast<const v4i*>(lds + fbase[i] + off);
        advance();
    };
    load_frags(af[0]);
    static_assert(D % 2 == 0, "fragment slots alternate");
    for (int h = h0; h < h1; h += D) {
#pragma unroll
        for (int k = 0; k < D; ++k) {
            if (k && h + k >= h1) break;                     // uniform
            load_frags(af[(k + 1) & 1]);
            // weights as the row operand: a lane ends up with channels 8 * (v / 4) + 4 * lhi + v % 4 of pixel l32
#pragma unroll
            for (int i = 0; i < FM; ++i)
#pragma unroll
                for (int j = 0; j < FN; ++j)
                    c[i][j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(b_reg[k][j], af[k & 1][i], c[i][j], 0, 0, 0);
            load_b(b_reg[k], h + k + D);
        }
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
        for (int e = 0; e < 4; ++e) r[e] += corr[e];
        const int m = m0 + row;
        if (m >= g.M || en >= p.N) continue;
        const size_t at = (size_t)m * p.N + en;
        const bool whole = (p.N & 3) == 0;                   // then the four channels are inside N together and aligned
        if (p.out_u8) {
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
            typedef float v4f __attribute__((ext_vector_type(4)));
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
template <class Cfg, int KIND>
sparq_status launch_split_cfg(const SplitParams& p, int npix_max, hipStream_t s) {
    SplitParams q = p;
    q.plane_stride = split_plane_stride(npix_max);
    const int lds_bytes = split_lds_bytes<Cfg>(npix_max, p.planes);
    if (lds_bytes < 0 || p.g.tm != Cfg::kTM) return SPARQ_EUNSUPPORTED;
    q.tiles_n = (p.N + Cfg::kTN - 1) / Cfg::kTN;
    const int64_t tiles = (int64_t)((p.g.M + Cfg::kTM - 1) / Cfg::kTM) * q.tiles_n;
    if (tiles > 0x7FFFFFFF) return SPARQ_EUNSUPPORTED;
    auto kern = conv_split_kernel<Cfg, KIND>;
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
