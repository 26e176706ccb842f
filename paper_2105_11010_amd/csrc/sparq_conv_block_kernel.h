// Fused SPARQ convolution for gfx950, filters of several taps on narrow layers: many small workgroups.
//
// In the persistent tile kernel (sparq_conv_patch_kernel.h) one workgroup per CU, or two, overlap their own phases by
// software pipelining; on layers of few channels its matrix wavefronts wait at the tile's barrier and then work through
// long epilogues alone.  Here a workgroup does one tile in plain phases -- stage 64 channels of the patch, multiply all taps,
// next 64 channels, results out -- and four of them share a CU, so that one stages while another multiplies and a third
// stores.  A tile is 256 pixels x 64 channels: of a 56-pixel-wide 3x3 layer 256 pixels need 1.6 patch pixels each, 128 need
// 2.6, and the trim of the patch is the largest item of such a layer.  128 pixels x 128 channels trim a patch once per 128 outputs
// instead: ahead beyond 64 of them, except where rows are wide (35 x 35 x 64 -> 96 3x3, batch 128, bytes 21.1 -> 19.1 us; the tile
// kernel 23.5).  A patch pixel's address is worked out once per tile, into
// LDS.  Requantised results: weights as the row operand (see sparq_conv_rows_kernel.h), rows leave through LDS.
// Bound by vector issue (66 % of the cycles by the counters, the matrix pipeline 30) and the phases' waits (40 % of a wavefront's
// life): 56 x 56 x 64 -> 64 3x3, batch 256, bytes: 78 -> 52 us (memory alone 21, the
// matrix instructions 18); three workgroups per CU with twice the weights requested ahead: 63; 128 pixels per tile: 77.  Waits that count
// exactly -- no request under a condition, none of the staging's left when the taps begin, fragments and weights asked for where it is
// written -- are 8 to 15 % of that (before 57; 35 x 35 x 96 3x3/2, batch 128, fp32 23.9 -> 20.3, 17 x 17 x 192 7x1 25.5 -> 23.5); the first
// requests ahead of the accumulators' constants, which keeps the weights' registers through the staging: 4 % slower.
#pragma once
#include "sparq_conv_patch_kernel.h"

namespace sparq {

struct BlockParams {
    const uint8_t* x;        // activations, NHWC, C a multiple of 4
    const uint8_t* wpk;      // packed weight tiles
    const int32_t* colsum;   // sum_k w[n][k], Np entries
    int32_t* acc;            // [M][N] or null
    const float* scale;      // [N] or null
    float* out;              // [M][N] or null
    uint8_t* out_u8;         // [M][N] requantised output or null (then it is the only output; N a multiple of 16)
    int trim_out;            // trim the requantised bytes with this launch's own mode
    int trim_in;             // 0: x is taken as it is
    uint32_t x_bytes, w_bytes;
    int N, Np, C;
    int ncb;                 // 64-channel blocks of a tap in the packed weights
    int plane_stride;        // bytes between the four 16-channel planes of the patch in LDS
    int tiles, tiles_n, tiles_xcd;
    PatchGeom g;             // tm = the tile's output pixels
    TrimLuts luts;
};

// WM x WN = 4 wavefronts, each 32 FM pixels x 32 FN channels.
template <int WM, int WN>
struct BlockCfg {
    static constexpr int kWM = WM, kWN = WN, kFM = 2, kFN = 2, kOcc = 4;         // four workgroups per CU: 128 registers
    static constexpr int kThreads = 256, kTM = 32 * kFM * WM, kTN = 32 * kFN * WN;
    static constexpr int kRowPitch = kTN + 16;               // LDS row of a pixel's result bytes
    static constexpr int kAhead = 2;                         // weight steps requested ahead
    static_assert(WM * WN == 4, "one wavefront per SIMD and workgroup");
};
typedef BlockCfg<4, 1> Block256x64;
typedef BlockCfg<2, 2> Block128x128;

template <class Cfg, int KIND, bool U8>
__global__ __launch_bounds__(Cfg::kThreads, Cfg::kOcc) void conv_block_kernel(const BlockParams p) {
    constexpr int FM = Cfg::kFM, FN = Cfg::kFN, TM = Cfg::kTM, TN = Cfg::kTN, NT = Cfg::kThreads, D = Cfg::kAhead;
    constexpr int CH = 3;                                    // patch chunks in flight per lane (4: 1 % slower)
    extern __shared__ __attribute__((aligned(16))) uint8_t lds[];            // [patch | pixel offsets], then result rows
    // every eighth workgroup runs on the same XCD: neighbouring tiles, which share patch rows and weights, go to one
    const int tile = ((int)blockIdx.x & 7) * p.tiles_xcd + ((int)blockIdx.x >> 3);
    if (tile >= p.tiles) return;
    const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, lhi = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), wm = wave % Cfg::kWM, wn = wave / Cfg::kWM;
    const PatchGeom& g = p.g;
    const int tile_m = tile / p.tiles_n, tile_n = tile - tile_m * p.tiles_n;
    const int m0 = tile_m * TM, n0t = tile_n * TN, n0 = n0t + wn * 32 * FN;      // the wavefront's channels
    const __amdgpu_buffer_rsrc_t xrsrc =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t*>(p.x), 0, (int)p.x_bytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t wrsrc =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t*>(p.wpk), 0, (int)p.w_bytes, 0x00020000);

    const TilePatch t = tile_patch(g, m0);
    uint32_t* const loff = reinterpret_cast<uint32_t*>(lds + 4 * p.plane_stride);
    for (int pix = tid; pix < t.npix; pix += NT) loff[pix] = patch_pixel_offset_u32<false>(g, t, pix, p.C, kPatchInvalidOffset);

    v16i c[FM][FN];
    int32_t corr[FN];
    float sc[FN];
    const float* scale_or_dummy = p.out ? p.scale : reinterpret_cast<const float*>(p.colsum);
#pragma unroll
    for (int j = 0; j < FN; ++j) {
        if constexpr (U8) {                                  // 128 * sum_k w[n][k] as the accumulators' initial value
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const v4i k = *reinterpret_cast<const v4i*>(p.colsum + n0 + 32 * j + 8 * q + 4 * lhi);   // Np entries
#pragma unroll
                for (int i = 0; i < FM; ++i)
#pragma unroll
                    for (int e = 0; e < 4; ++e) c[i][j][4 * q + e] = k[e] * 128;
            }
        } else {
            const int n = n0 + 32 * j + l32, nc = n < p.N ? n : 0;
            corr[j] = p.colsum[nc] * 128;
            sc[j] = scale_or_dummy[nc];
#pragma unroll
            for (int i = 0; i < FM; ++i)
#pragma unroll
                for (int v = 0; v < 16; ++v) c[i][j][v] = 0;
        }
    }
    int32_t fbase[FM];
#pragma unroll
    for (int i = 0; i < FM; ++i) {
        int m = m0 + (wm * FM + i) * 32 + l32;
        m = m < g.M ? m : g.M - 1;
        fbase[i] = patch_pixel_of_output(g, t, m) * kChunk + lhi * p.plane_stride;
    }
    const int wlane = (lhi * p.Np + n0 + l32) * kChunk;
    const int w_step = 2 * p.Np * kChunk;                    // bytes of a 32-index step of all channels
    const int steps = 2 * g.KH * g.KW;                       // per 64-channel block
    __syncthreads();

    const int plane = tid & 3;
    const int chunks = t.npix * 4;
    v4u a_reg[CH];
    for (int cb = 0; cb < p.ncb; ++cb) {
        // ---- the block's weights start, its patch goes to LDS ----
        v4i b[D][FN];
        int b_tap = 0, b_half = 0;                           // the step requested next
        auto load_b = [&](v4i (&dst)[FN]) __attribute__((always_inline)) {
            const int soff = ((b_tap * p.ncb + cb) * 2 + b_half) * w_step;
#pragma unroll
            for (int j = 0; j < FN; ++j)
                dst[j] = __builtin_bit_cast(v4i, __builtin_amdgcn_raw_buffer_load_b128(wrsrc, wlane + j * 32 * kChunk, soff, 0));
            b_tap += b_half;
            b_half ^= 1;
            if (2 * b_tap == steps) b_tap = 0;               // past the last: a read that is not used
        };
        // A request past the patch reads 0 without touching memory: under a condition it would cost the exact wait counts, and every chunk
        // a full latency.
        const uint32_t ch = (uint32_t)(cb * 64 + plane * kChunk);
        const bool live = (int)ch < p.C;
        auto load_chunk = [&](int i, int e) __attribute__((always_inline)) {
            const uint32_t off = loff[e < chunks ? e >> 2 : 0] + ch;
            a_reg[i] = __builtin_amdgcn_raw_buffer_load_b128(xrsrc, e < chunks && live ? (int)off : (int)kPatchInvalidOffset, 0, 0);
        };
#pragma unroll
        for (int i = 0; i < CH; ++i) load_chunk(i, tid + i * NT);
#pragma unroll
        for (int k = 0; k < D; ++k) load_b(b[k]);
        __builtin_amdgcn_sched_barrier(0);
        for (int e0 = 0; e0 < chunks; e0 += CH * NT) {
#pragma unroll
            for (int i = 0; i < CH; ++i) {
                const int e = e0 + i * NT + tid;
                if (e0 + i * NT + wave * 64 < chunks) {      // uniform
                    v4u v = a_reg[i];
                    if (KIND != kTrimNone && p.trim_in) {
#pragma unroll
                        for (int j = 0; j < 4; ++j) v[j] = trim4_kind<KIND>(v[j], p.luts);
                    }
#pragma unroll
                    for (int j = 0; j < 4; ++j) v[j] ^= 0x80808080u;
                    if (e < chunks) *reinterpret_cast<v4u*>(lds + plane * p.plane_stride + (e >> 2) * kChunk) = v;
                }
                load_chunk(i, e + CH * NT);
            }
        }
        // the last requests (past the patch) end here: their registers serve the loop below, which would wait for its weights with them
#pragma unroll
        for (int i = 0; i < CH; ++i) asm volatile("" ::"v"(a_reg[i]));
        __syncthreads();

        // ---- all taps ----
        int f_half = 0, f_kh = 0, f_kw = 0;
        v4i af[2][FM];
        auto load_frags = [&](v4i (&a)[FM]) __attribute__((always_inline)) {
            const int off = f_half * 2 * p.plane_stride + (f_kh * t.pwt + f_kw) * kChunk;
#pragma unroll
            for (int i = 0; i < FM; ++i) a[i] = *reinterpret_cast<const v4i*>(lds + fbase[i] + off);
            f_kw += f_half;
            f_half ^= 1;
            if (f_kw == g.KW) {
                f_kw = 0;
                if (++f_kh == g.KH) f_kh = 0;                // past the last step: any place inside the patch
            }
        };
        load_frags(af[0]);
        for (int h = 0; h < steps; h += D) {                 // (two steps a tap)
#pragma unroll
            for (int k = 0; k < D; ++k) {
                load_frags(af[(k + 1) & 1]);
                __builtin_amdgcn_sched_barrier(0);           // (the compiler puts reads and requests right in front of their use)
#pragma unroll
                for (int i = 0; i < FM; ++i)
#pragma unroll
                    for (int j = 0; j < FN; ++j)
                        c[i][j] = U8 ? __builtin_amdgcn_mfma_i32_32x32x32_i8(b[k][j], af[k & 1][i], c[i][j], 0, 0, 0)
                                     : __builtin_amdgcn_mfma_i32_32x32x32_i8(af[k & 1][i], b[k][j], c[i][j], 0, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
                load_b(b[k]);
            }
        }
        __syncthreads();                                     // the patch has been read
    }

    // ---- results ----
    const int rows = g.M - m0 < TM ? g.M - m0 : TM;
    const size_t base = (size_t)m0 * p.N;
    if constexpr (U8) {
        const __amdgpu_buffer_rsrc_t frsrc =
            __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(p.scale), 0, p.N * 4, 0x00020000);
#pragma unroll
        for (int j = 0; j < FN; ++j) {
            typedef float v4f __attribute__((ext_vector_type(4)));
            v4f fac[4];
#pragma unroll
            for (int q = 0; q < 4; ++q)                      // (past N: 0)
                fac[q] = __builtin_bit_cast(v4f, __builtin_amdgcn_raw_buffer_load_b128(frsrc, (n0 + 32 * j + 8 * q + 4 * lhi) * 4, 0, 0));
#pragma unroll
            for (int i = 0; i < FM; ++i) {
                uint32_t w[4];
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    uint32_t r = __builtin_amdgcn_cvt_pk_u8_f32(__fmul_rn((float)c[i][j][4 * q], fac[q][0]), 0, 0);
                    r = __builtin_amdgcn_cvt_pk_u8_f32(__fmul_rn((float)c[i][j][4 * q + 1], fac[q][1]), 1, r);
                    r = __builtin_amdgcn_cvt_pk_u8_f32(__fmul_rn((float)c[i][j][4 * q + 2], fac[q][2]), 2, r);
                    w[q] = __builtin_amdgcn_cvt_pk_u8_f32(__fmul_rn((float)c[i][j][4 * q + 3], fac[q][3]), 3, r);
                }
                if (KIND != kTrimNone && p.trim_out) {
#pragma unroll
                    for (int q = 0; q < 4; ++q) w[q] = trim4_kind<KIND>(w[q], p.luts);
                }
                const auto s02 = __builtin_amdgcn_permlane32_swap(w[0], w[2], false, false);
                const auto s13 = __builtin_amdgcn_permlane32_swap(w[1], w[3], false, false);
                *reinterpret_cast<v4u*>(lds + ((wm * FM + i) * 32 + l32) * Cfg::kRowPitch + (wn * FN + j) * 32 + 16 * lhi) =
                    v4u{s02[0], s02[1], s13[0], s13[1]};
            }
        }
        __syncthreads();
        const __amdgpu_buffer_rsrc_t orsrc =
            __builtin_amdgcn_make_buffer_rsrc((void*)(p.out_u8 + base), 0, rows * p.N, 0x00020000);
        constexpr int LPR = TN / 16, RPR = NT / LPR;         // lanes per row, rows per round
        const int col = n0t + 16 * (tid % LPR);
#pragma unroll
        for (int r = 0; r < TM / RPR; ++r) {
            const int row = r * RPR + tid / LPR;
            const v4u o = *reinterpret_cast<const v4u*>(lds + row * Cfg::kRowPitch + 16 * (tid % LPR));
            __builtin_amdgcn_raw_buffer_store_b128(o, orsrc, col < p.N ? row * p.N + col : (int)kPatchInvalidOffset, 0, 0);
        }
    } else {
        const int pitch = p.N * 4, bytes = rows * pitch;
        const __amdgpu_buffer_rsrc_t arsrc =
            __builtin_amdgcn_make_buffer_rsrc(p.acc ? (void*)(p.acc + base) : nullptr, 0, p.acc ? bytes : 0, 0x00020000);
        const __amdgpu_buffer_rsrc_t orsrc =
            __builtin_amdgcn_make_buffer_rsrc(p.out ? (void*)(p.out + base) : nullptr, 0, p.out ? bytes : 0, 0x00020000);
        auto store = [&](auto acc_, auto out_) __attribute__((always_inline)) {
#pragma unroll
            for (int i = 0; i < FM; ++i)
#pragma unroll
                for (int v = 0; v < 16; ++v)
#pragma unroll
                    for (int j = 0; j < FN; ++j) {
                        const int n = n0 + 32 * j + l32;
                        const int row = (wm * FM + i) * 32 + 8 * (v / 4) + 4 * lhi + v % 4;
                        const int off = n < p.N ? row * pitch + n * 4 : (int)kPatchInvalidOffset;
                        const int32_t r = c[i][j][v] + corr[j];
                        if constexpr (decltype(acc_)::value) __builtin_amdgcn_raw_buffer_store_b32(r, arsrc, off, 0, kResultStorePolicy);
                        if constexpr (decltype(out_)::value)
                            __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(int, __fmul_rn((float)r, sc[j])), orsrc, off, 0, kResultStorePolicy);
                    }
        };
        if (p.acc && p.out) store(std::true_type{}, std::true_type{});
        else if (p.out) store(std::false_type{}, std::true_type{});
        else store(std::true_type{}, std::false_type{});
    }
}

// LDS of a launch: the patch and its pixel offsets, or the result rows in the same place.
template <class Cfg>
int block_lds_bytes(int npix_max) {
    const int64_t patch = 4ll * patch_plane_stride(npix_max, 4) + round_up(4ll * npix_max, 16), rows = (int64_t)Cfg::kTM * Cfg::kRowPitch;
    const int64_t need = patch > rows ? patch : rows;
    return need > kLdsPerCu ? -1 : (int)need;
}

template <class Cfg>
int64_t block_tiles(int64_t M, int64_t N) {
    return (M + Cfg::kTM - 1) / Cfg::kTM * ((N + Cfg::kTN - 1) / Cfg::kTN);
}
// What the kernel can be launched for: LDS (64 KB: what a launch may use without asking), 32-bit offsets inside a tile of
// results, tile numbers.  The rule that picks this form asks the same, so that other layers go on to the other kernels.
template <class Cfg>
bool block_launchable(int64_t M, int64_t N, int npix_max) {
    const int lds_bytes = block_lds_bytes<Cfg>(npix_max);
    return lds_bytes >= 0 && lds_bytes <= 64 * 1024 && N * 4 * Cfg::kTM < 0x7FFFFFFF && block_tiles<Cfg>(M, N) <= 0x0FFFFFFF;
}

// `p` carries everything except plane_stride and the tile counts; npix_max bounds TilePatch::npix.
template <class Cfg, int KIND, bool U8>
sparq_status launch_block_cfg(const BlockParams& p, int npix_max, hipStream_t s) {
    BlockParams q = p;
    q.plane_stride = patch_plane_stride(npix_max, 4);
    const int lds_bytes = block_lds_bytes<Cfg>(npix_max);
    q.tiles_n = (p.N + Cfg::kTN - 1) / Cfg::kTN;
    if (p.g.tm != Cfg::kTM || p.g.rm_wo || q.tiles_n * Cfg::kTN > p.Np || !block_launchable<Cfg>(p.g.M, p.N, npix_max)) return SPARQ_EUNSUPPORTED;
    q.tiles = (int)block_tiles<Cfg>(p.g.M, p.N);
    q.tiles_xcd = (q.tiles + 7) / 8;
    conv_block_kernel<Cfg, KIND, U8><<<(unsigned)(8 * q.tiles_xcd), Cfg::kThreads, lds_bytes, s>>>(q);
    return launch_status();
}

template <class Cfg>
sparq_status launch_block_tile(TrimKind kind, const BlockParams& p, int npix_max, hipStream_t s) {
    const auto go = [&](auto kind_) {
        constexpr int K = decltype(kind_)::value;
        return p.out_u8 ? launch_block_cfg<Cfg, K, true>(p, npix_max, s) : launch_block_cfg<Cfg, K, false>(p, npix_max, s);
    };
    switch (kind) {
        case kTrimNone: return go(int_c<kTrimNone>{});
        case kTrimFloor: return go(int_c<kTrimFloor>{});
        case kTrimFloorPair: return go(int_c<kTrimFloorPair>{});
        case kTrimFloorPairWide: return go(int_c<kTrimFloorPairWide>{});
        case kTrimRound: return go(int_c<kTrimRound>{});
        case kTrimRound4: return go(int_c<kTrimRound4>{});
        case kTrimRoundPairWide: return go(int_c<kTrimRoundPairWide>{});
        case kTrimRoundPair4: return go(int_c<kTrimRoundPair4>{});
        default: return SPARQ_EUNSUPPORTED;
    }
}
typedef sparq_status (*BlockLauncher)(TrimKind, const BlockParams&, int npix_max, hipStream_t);
sparq_status launch_block_256x64(TrimKind kind, const BlockParams& p, int npix_max, hipStream_t s);
sparq_status launch_block_128x128(TrimKind kind, const BlockParams& p, int npix_max, hipStream_t s);

}  // namespace sparq
