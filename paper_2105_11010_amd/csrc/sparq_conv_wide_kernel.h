// Fused SPARQ matrix product for gfx950: 1x1 filters with a long reduction, eight wavefronts per tile.
//
// Every activation of such a layer is used once per output channel and nothing else, so its trim (about 20 vector
// instructions per four activations) runs beside the matrix instructions of the same SIMD and has to be shared by as many
// output channels as possible: tiles of 128 pixels x 512 (or 256) channels.  The gather kernel's 128 x 512 tile has one
// wavefront per SIMD, which holds 128 x 128 results and stands still at every wait; here two wavefronts per SIMD hold
// 128 x 64 results each, and one trims or waits while the other multiplies.
// A step is 64 channels: 512 lanes stage one 16-byte chunk each (8 KB, one of four LDS buffers), requested four steps and
// written two steps ahead of its use; weights come from L2 two steps ahead; one barrier per step.  The steps of a
// workgroup's tiles form one pipeline: the next tile's chunks and weights are on their way while results leave.
// The trim goes between the matrix instructions in quarters of a step, by hand: left to the scheduler it bunches (65536 x
// 4608 x 512, int32: 188 us, this way 172; the gather kernel 197; bytes 154 against 233).  Bound by the step's traffic beside the
// matrix pipeline (without any trim 144): 32 KB of weights through L1 and 64 KB of fragments through LDS per 1024 cycles
// of matrix instructions, and by the result stores, which both tiles of a CU wait for (18 us of int32 results).  Counters: matrix pipeline busy 56 %
// of the cycles, vector issue 48, LDS 23, a quarter of a wavefront's life in waits.
#pragma once
#include "sparq_conv_patch_kernel.h"

namespace sparq {

struct WideParams {
    const uint8_t* x;        // activations, NHWC, C a multiple of 4
    const uint8_t* wpk;      // packed weight tiles
    const int32_t* colsum;   // sum_k w[n][k], Np entries
    int32_t* acc;            // [M][N] or null
    const float* scale;      // [N] or null
    float* out;              // [M][N] or null
    uint8_t* out_u8;         // [M][N] requantised output or null (then it is the only output; N a multiple of 16)
    int trim_out;            // trim the requantised bytes with this launch's own mode
    int trim_in;             // always 1 (a branch in the step would part its instructions)
    uint32_t x_bytes, w_bytes;
    int M, N, Np, C;
    int steps;               // 64-channel steps
    int steps4;              // ... rounded up to a multiple of four (the ring's length); the extra ones multiply zeros
    int tiles, tiles_n, tiles_xcd;
    PatchGeom g;             // the long row's pixel remap for strided layers
    TrimLuts luts;
};

constexpr int kWideThreads = 512;
constexpr int kWidePitch = 64 + 16;                // LDS row of 64 result bytes

// WM x WN = 8 wavefronts of 32 FM pixels x 64 channels.
template <int WM, int WN, int FM>
struct WideCfg {
    static constexpr int kWM = WM, kWN = WN, kFM = FM, kTM = 32 * FM * WM, kTN = 64 * WN;
    static constexpr int kPlane = kTM * kChunk + 64;         // bytes between the 16-channel planes of a step's buffer
    static constexpr int kBuf = 4 * kPlane;
    static constexpr int kLds = 4 * kBuf + 8 * 32 * kWidePitch;
    static_assert(WM * WN == 8 && kTM == 128, "512 lanes stage one chunk each");
};

template <class Cfg, int KIND, bool U8>
__global__ __launch_bounds__(kWideThreads, 2) void conv_wide_kernel(const WideParams p) {
    constexpr int FM = Cfg::kFM, FN = 2, TM = Cfg::kTM, TN = Cfg::kTN;
    extern __shared__ __attribute__((aligned(16))) uint8_t lds[];            // [4 step buffers][result rows per wavefront]
    const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, lhi = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave % Cfg::kWM, wn = wave / Cfg::kWM;
    // every eighth workgroup runs on the same XCD: an XCD's tiles are neighbours, sharing pixels or weights in its L2
    const int xcd = (int)blockIdx.x & 7, tile_step = (int)gridDim.x >> 3;
    const int tile_end = (xcd + 1) * p.tiles_xcd < p.tiles ? (xcd + 1) * p.tiles_xcd : p.tiles;
    int tile = xcd * p.tiles_xcd + ((int)blockIdx.x >> 3);
    if (tile >= tile_end) return;
    const __amdgpu_buffer_rsrc_t xrsrc =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t*>(p.x), 0, (int)p.x_bytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t wrsrc =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t*>(p.wpk), 0, (int)p.w_bytes, 0x00020000);

    // ---- activations: lane's chunk is plane tid & 3 of row tid >> 2 ----
    const int plane = tid & 3, srow = tid >> 2;
    uint8_t* const stage_at = lds + plane * Cfg::kPlane + srow * kChunk;
    v4u raw[4];
    // byte offset of the lane's row of a tile (past the last tile or row: outside the tensor, reads 0)
    auto row_offset = [&](int of_tile) __attribute__((always_inline)) -> uint32_t {
        const int m = of_tile / p.tiles_n * TM + srow;
        const bool live = of_tile < tile_end && m < p.M;
        int pix = m;
        if (p.g.rm_wo) pix = remap_pixel(p.g, live ? m : 0);
        return live ? (uint32_t)(pix * p.C) : kPatchInvalidOffset;
    };
    uint32_t x_now = row_offset(tile), x_next = 0;
    int w_now = tile % p.tiles_n * TN * kChunk, w_next = 0;  // byte offset of a tile's channels in a half step's weights
    // step u of this tile, u - steps4 of the next (the requests run ahead by less than a tile)
    auto load_x = [&](v4u& dst, int u) __attribute__((always_inline)) {
        const bool over = u >= p.steps4;                     // uniform
        const int ch = (over ? u - p.steps4 : u) * 64 + plane * kChunk;
        const uint32_t off = ch < p.C ? (over ? x_next : x_now) + (uint32_t)ch : kPatchInvalidOffset;
        dst = __builtin_amdgcn_raw_buffer_load_b128(xrsrc, (int)off, 0, 0);
    };
    auto stage = [&](v4u v, int buf) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < 4; ++j) v[j] = trim4_kind<KIND>(v[j], p.luts) ^ 0x80808080u;
        *reinterpret_cast<v4u*>(stage_at + buf * Cfg::kBuf) = v;
    };

    // ---- weights ----
    const int wlane = (lhi * p.Np + wn * 64 + l32) * kChunk;
    const int w_half = 2 * p.Np * kChunk;                    // bytes of a 32-index half step of all channels
    v4i b[2][2][FN];
    auto load_b = [&](v4i (&dst)[2][FN], int u, int h) __attribute__((always_inline)) {      // half h of the step
        const bool over = u >= p.steps4;                     // uniform
        const int step = over ? u - p.steps4 : u;
        const bool live = step < p.steps;                    // the padding steps read 0 (nothing is fetched)
        const int voff = live ? wlane : (int)kPatchInvalidOffset;
        const int soff = live ? (step * 2 + h) * w_half + (over ? w_next : w_now) : 0;
#pragma unroll
        for (int j = 0; j < FN; ++j)
            dst[h][j] = __builtin_bit_cast(v4i, __builtin_amdgcn_raw_buffer_load_b128(wrsrc, voff + j * 32 * kChunk, soff, 0));
    };

    // ---- fragments: half h of the buffer's step ----
    const uint8_t* const frag_at = lds + lhi * Cfg::kPlane + (wm * 32 * FM + l32) * kChunk;
    v4i af[2][FM];
    auto load_frags = [&](v4i (&a)[FM], int buf, int h) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < FM; ++i)
            a[i] = *reinterpret_cast<const v4i*>(frag_at + buf * Cfg::kBuf + h * 2 * Cfg::kPlane + i * 32 * kChunk);
    };

#pragma unroll
    for (int k = 0; k < 4; ++k) load_x(raw[k], k);
#pragma unroll
    for (int k = 0; k < 4; ++k) load_b(b[k / 2], k / 2, k & 1);
    stage(raw[0], 0);
    load_x(raw[0], 4);
    stage(raw[1], 1);
    load_x(raw[1], 5);
    __syncthreads();
    load_frags(af[0], 0, 0);

    v16i c[FM][FN];
    const float* scale_or_dummy = p.out ? p.scale : reinterpret_cast<const float*>(p.colsum);
    for (; tile < tile_end; tile += tile_step) {
        x_next = row_offset(tile + tile_step);
        w_next = (tile + tile_step < tile_end ? tile + tile_step : tile) % p.tiles_n * TN * kChunk;
#pragma unroll
        for (int i = 0; i < FM; ++i)
#pragma unroll
            for (int j = 0; j < FN; ++j)
#pragma unroll
                for (int v = 0; v < 16; ++v) c[i][j][v] = 0;
        for (int s = 0; s < p.steps4; s += 4) {
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                // Four regions of a quarter of the step's matrix instructions and one word of the trim each, interleaved
                // by hand (both wavefronts of a SIMD are in the same step, so a stretch without matrix instructions is
                // one for both; over the whole step the compiler bunches them).
                constexpr int QM = FM / 2;                   // pixel fragments per quarter
                v4u st = raw[(k + 2) & 3];
                auto quarter = [&](auto w_) __attribute__((always_inline)) {
                    constexpr int w = decltype(w_)::value, h = w / 2;
                    if constexpr (w == 0) load_frags(af[1], k, 1);
                    if constexpr (w == 2) {
                        load_frags(af[0], (k + 1) & 3, 0);
                        load_b(b[k & 1], s + k + 2, 0);
                    }
#pragma unroll
                    for (int i = (w & 1) * QM; i < (w & 1) * QM + QM; ++i)
#pragma unroll
                        for (int j = 0; j < FN; ++j)
                            c[i][j] = U8 ? __builtin_amdgcn_mfma_i32_32x32x32_i8(b[k & 1][h][j], af[h][i], c[i][j], 0, 0, 0)
                                         : __builtin_amdgcn_mfma_i32_32x32x32_i8(af[h][i], b[k & 1][h][j], c[i][j], 0, 0, 0);
                    st[w] = trim4_kind<KIND>(st[w], p.luts) ^ 0x80808080u;
#pragma unroll
                    for (int q = 0; q < QM * FN; ++q) {
                        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);               // a matrix instruction
                        __builtin_amdgcn_sched_group_barrier(0x002, (KIND == kTrimNone ? 4 : 24) / (QM * FN), 0);   // a part of the trim
                        if constexpr (!(w & 1)) __builtin_amdgcn_sched_group_barrier(0x100, (FM + QM * FN - 1) / (QM * FN), 0);   // fragment reads
                        if constexpr (w == 2) __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);    // a request
                    }
                    __builtin_amdgcn_sched_barrier(0);
                };
                quarter(int_c<0>{});
                quarter(int_c<1>{});
                quarter(int_c<2>{});
                quarter(int_c<3>{});
                *reinterpret_cast<v4u*>(stage_at + ((k + 2) & 3) * Cfg::kBuf) = st;
                load_b(b[k & 1], s + k + 2, 1);
                load_x(raw[(k + 2) & 3], s + k + 6);
                __syncthreads();
            }
        }

        // ---- results ----
        const int tile_m = tile / p.tiles_n, nw = (tile - tile_m * p.tiles_n) * TN + wn * 64;
        const int m0 = tile_m * TM, rows = p.M - m0 < TM ? p.M - m0 : TM;
        const size_t base = (size_t)m0 * p.N;
        if constexpr (U8) {
            typedef float v4f __attribute__((ext_vector_type(4)));
            const __amdgpu_buffer_rsrc_t frsrc =
                __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(p.scale), 0, p.N * 4, 0x00020000);
            const __amdgpu_buffer_rsrc_t orsrc =
                __builtin_amdgcn_make_buffer_rsrc((void*)(p.out_u8 + base), 0, rows * p.N, 0x00020000);
            uint8_t* const turn = lds + 4 * Cfg::kBuf + wave * 32 * kWidePitch;      // the wavefront's own: no barrier
            const int col = nw + 16 * (lane & 3);
#pragma unroll
            for (int i = 0; i < FM; ++i) {
#pragma unroll
                for (int j = 0; j < FN; ++j) {
                    // (read again for every fragment, from L1: held for the tile they would push the loop's registers out)
                    int n_lane = nw + 32 * j + 4 * lhi;
                    asm volatile("" : "+v"(n_lane));
                    v4i corr[4];
                    v4f fac[4];
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        corr[q] = *reinterpret_cast<const v4i*>(p.colsum + n_lane + 8 * q);          // (Np entries)
                        fac[q] = __builtin_bit_cast(v4f, __builtin_amdgcn_raw_buffer_load_b128(frsrc, (n_lane + 8 * q) * 4, 0, 0));   // (past N: 0)
                    }
                    uint32_t w[4];
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        int32_t r[4];
#pragma unroll
                        for (int e = 0; e < 4; ++e) r[e] = c[i][j][4 * q + e] + corr[q][e] * 128;
                        uint32_t t = __builtin_amdgcn_cvt_pk_u8_f32(__fmul_rn((float)r[0], fac[q][0]), 0, 0);
                        t = __builtin_amdgcn_cvt_pk_u8_f32(__fmul_rn((float)r[1], fac[q][1]), 1, t);
                        t = __builtin_amdgcn_cvt_pk_u8_f32(__fmul_rn((float)r[2], fac[q][2]), 2, t);
                        w[q] = __builtin_amdgcn_cvt_pk_u8_f32(__fmul_rn((float)r[3], fac[q][3]), 3, t);
                    }
                    if (KIND != kTrimNone && p.trim_out) {
#pragma unroll
                        for (int q = 0; q < 4; ++q) w[q] = trim4_kind<KIND>(w[q], p.luts);
                    }
                    const auto s02 = __builtin_amdgcn_permlane32_swap(w[0], w[2], false, false);
                    const auto s13 = __builtin_amdgcn_permlane32_swap(w[1], w[3], false, false);
                    *reinterpret_cast<v4u*>(turn + l32 * kWidePitch + 32 * j + 16 * lhi) = v4u{s02[0], s02[1], s13[0], s13[1]};
                }
                wavefront_lds_fence();
#pragma unroll
                for (int r = 0; r < 2; ++r) {
                    const int row = 16 * r + (lane >> 2);
                    const v4u o = *reinterpret_cast<const v4u*>(turn + row * kWidePitch + 16 * (lane & 3));
                    const int off = col < p.N ? ((wm * FM + i) * 32 + row) * p.N + col : (int)kPatchInvalidOffset;
                    __builtin_amdgcn_raw_buffer_store_b128(o, orsrc, off, 0, 0);
                }
                wavefront_lds_fence();
            }
        } else {
            const int pitch = p.N * 4, bytes = rows * pitch;
            const __amdgpu_buffer_rsrc_t arsrc =
                __builtin_amdgcn_make_buffer_rsrc(p.acc ? (void*)(p.acc + base) : nullptr, 0, p.acc ? bytes : 0, 0x00020000);
            const __amdgpu_buffer_rsrc_t orsrc =
                __builtin_amdgcn_make_buffer_rsrc(p.out ? (void*)(p.out + base) : nullptr, 0, p.out ? bytes : 0, 0x00020000);
            int32_t corr[FN];
            float sc[FN];
            uint32_t lane_off[FN];
#pragma unroll
            for (int j = 0; j < FN; ++j) {
                const int n = nw + 32 * j + l32, nc = n < p.N ? n : 0;
                corr[j] = p.colsum[nc] * 128;
                sc[j] = scale_or_dummy[nc];
                lane_off[j] = n < p.N ? (uint32_t)((wm * FM * 32 + 4 * lhi) * pitch + n * 4) : kPatchInvalidOffset;
            }
            auto store = [&](auto acc_, auto out_) __attribute__((always_inline)) {
#pragma unroll
                for (int i = 0; i < FM; ++i)
#pragma unroll
                    for (int v = 0; v < 16; ++v)
#pragma unroll
                        for (int j = 0; j < FN; ++j) {
                            const int32_t r = c[i][j][v] + corr[j];
                            const int off = (int)(lane_off[j] + (uint32_t)((i * 32 + 8 * (v / 4) + v % 4) * pitch));
                            if constexpr (decltype(acc_)::value) __builtin_amdgcn_raw_buffer_store_b32(r, arsrc, off, 0, kResultStorePolicy);
                            if constexpr (decltype(out_)::value)
                                __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(int, __fmul_rn((float)r, sc[j])), orsrc, off, 0, kResultStorePolicy);
                        }
            };
            if (p.acc && p.out) store(std::true_type{}, std::true_type{});
            else if (p.out) store(std::false_type{}, std::true_type{});
            else store(std::true_type{}, std::false_type{});
        }
        x_now = x_next;
        w_now = w_next;
    }
}

// `p` carries everything except steps4 and the tile counts.
template <class Cfg, int KIND, bool U8>
sparq_status launch_wide_cfg(const WideParams& p, hipStream_t s) {
    WideParams q = p;
    q.steps4 = (p.steps + 3) & ~3;
    q.tiles_n = (p.N + Cfg::kTN - 1) / Cfg::kTN;
    // the requests run six steps ahead, at most into the next tile
    if (q.steps4 < 8 || !p.trim_in || q.tiles_n * Cfg::kTN > p.Np || (int64_t)p.N * 4 * Cfg::kTM >= 0x7FFFFFFF) return SPARQ_EUNSUPPORTED;
    const int64_t tiles = ((int64_t)p.M + Cfg::kTM - 1) / Cfg::kTM * q.tiles_n;
    if (tiles > 0x0FFFFFFF) return SPARQ_EUNSUPPORTED;
    q.tiles = (int)tiles;
    q.tiles_xcd = (q.tiles + 7) / 8;
    auto kern = conv_wide_kernel<Cfg, KIND, U8>;
    static_assert(Cfg::kLds <= 64 * 1024, "what a launch may use without asking");
    // one workgroup per CU (its registers fill it); a multiple of eight: the same number for every XCD
    const int cus = device_cu_count() & ~7;
    const int grid = 8 * q.tiles_xcd < cus ? 8 * q.tiles_xcd : cus < 8 ? 8 : cus;
    kern<<<(unsigned)grid, kWideThreads, Cfg::kLds, s>>>(q);
    return launch_status();
}

template <class Cfg, int KIND>
sparq_status launch_wide_out(const WideParams& p, hipStream_t s) {
    return p.out_u8 ? launch_wide_cfg<Cfg, KIND, true>(p, s) : launch_wide_cfg<Cfg, KIND, false>(p, s);
}

template <class Cfg>
sparq_status launch_wide_kind(TrimKind kind, const WideParams& p, hipStream_t s) {
    switch (kind) {
        case kTrimNone: return launch_wide_out<Cfg, kTrimNone>(p, s);
        case kTrimFloor: return launch_wide_out<Cfg, kTrimFloor>(p, s);
        case kTrimFloorPair: return launch_wide_out<Cfg, kTrimFloorPair>(p, s);
        case kTrimFloorPairWide: return launch_wide_out<Cfg, kTrimFloorPairWide>(p, s);
        case kTrimRound: return launch_wide_out<Cfg, kTrimRound>(p, s);
        case kTrimRound4: return launch_wide_out<Cfg, kTrimRound4>(p, s);
        case kTrimRoundPairWide: return launch_wide_out<Cfg, kTrimRoundPairWide>(p, s);
        case kTrimRoundPair4: return launch_wide_out<Cfg, kTrimRoundPair4>(p, s);
        default: return SPARQ_EUNSUPPORTED;
    }
}

typedef WideCfg<1, 8, 4> Wide512;
typedef WideCfg<2, 4, 2> Wide256;
typedef sparq_status (*WideLauncher)(TrimKind, const WideParams&, hipStream_t);
sparq_status launch_wide_512(TrimKind kind, const WideParams& p, hipStream_t s);
sparq_status launch_wide_256(TrimKind kind, const WideParams& p, hipStream_t s);

}  // namespace sparq
