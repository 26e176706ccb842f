// Fused SPARQ convolution for gfx950, 1x1 filters (and plain matrix products) with a short reduction: activations
// stay in registers.
//
// A 1x1 layer moves a byte or four per result and multiplies little, so what it spends outside the matrix
// instructions decides.  Here a wavefront takes 32 or 64 output pixels, loads their channels straight in fragment
// order (lane = pixel, 16 channels per load), trims them once, and keeps all K of them in registers while it walks the
// output channels 32 at a time: no LDS patch, no barrier, no tile boundary, and other wavefronts of the SIMD work while
// one waits.  The next pixels are requested before the walk starts.
// Requantised results: the weights are the row operand, so a lane holds four times four consecutive channels of one
// pixel.  The offset 128 * sum_k w[n][k] is the accumulators' initial value, the conversion packs the bytes of a word, and
// two half-wave swaps make 16 consecutive bytes of them: 52 vector instructions per 16 results (100 in the tile kernels,
// which transpose lane quads); they leave through a wavefront's own LDS rows, 128 bytes of a pixel at a time (as 32-byte
// pieces straight from the registers 64 -> 256 channels took 118 us, this way 58).  int32 / fp32 results: the activations
// are the row operand and a store writes whole runs.
// Up to 128 channels bound by memory (64 -> 256, 802816 pixels, bytes: 106 -> 58 us, 4.4 TB/s; 128 -> 512, 200704 pixels:
// 60 -> 35); from 256 channels on by the trim's vector instructions and the weights from L2 (256 -> 64, 802816 pixels:
// 80 -> 69, 56 without a trim; 256 -> 1024, 50176 pixels: 42 -> 29; 512 -> 1024: 69 -> 47).  Counters, bytes: with 64 channels 55 % of
// a wavefront's life in waits, with 256 25 % and vector issue at 45 to 53 % of the cycles.
#pragma once
#include "sparq_conv_patch_kernel.h"

namespace sparq {

typedef float v4f_rows __attribute__((ext_vector_type(4)));

struct RowsParams {
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
    int M, N, Np, C;
    int steps;               // 32-index reduction steps, at most KS
    int items_n;             // shares the output channels are split into
    int item_blocks;         // 32-channel blocks per share
    int items;               // groups of pixels x shares
    PatchGeom g;             // the long row's pixel remap for strided layers
    TrimLuts luts;
};

constexpr int kRowsThreads = 256;
constexpr int kRowsPitch = 128 + 16;               // LDS row of 128 result bytes, padded against bank conflicts

// KS 32-index steps of activations in registers, FM fragments of 32 pixels per wavefront, PF: the next pixels are requested
// while the current ones are multiplied, OCC wavefronts per SIMD.
template <int KS, int FM, bool PF, int OCC>
struct RowsCfg {
    static constexpr int kKS = KS, kFM = FM, kOcc = OCC, kRM = 32 * FM;
    static constexpr bool kPF = PF;
    static constexpr int kRing = KS % 8 == 0 ? 8 : KS % 6 == 0 ? 6 : KS % 5 == 0 ? 5 : KS;     // weight steps requested ahead; divides KS
    static_assert(KS % kRing == 0, "ring slots are fixed per step");
};

template <class Cfg, int KIND, bool U8>
__global__ __launch_bounds__(kRowsThreads, Cfg::kOcc) void conv_rows_kernel(const RowsParams p) {
    constexpr int KS = Cfg::kKS, FM = Cfg::kFM, RM = Cfg::kRM, D = Cfg::kRing;
    constexpr bool PF = Cfg::kPF;
    // U8: a wavefront's bytes on their way out, then [corr | factor] of all channels
    extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
    const int lane = threadIdx.x & 63, l32 = lane & 31, lhi = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int nr = (p.N + 31) & ~31;
    int32_t* lcorr = reinterpret_cast<int32_t*>(lds + (kRowsThreads / 64) * RM * kRowsPitch);
    float* lfac = reinterpret_cast<float*>(lcorr) + nr;
    // turned through LDS (the wavefront's own area, no barrier): a lane writes 16 bytes of its pixel per block and reads
    // 16 bytes of the row its group of eight lanes stores
    uint8_t* const turn = lds + wave * RM * kRowsPitch;
    uint8_t* const turn_w = turn + l32 * kRowsPitch + 16 * lhi;
    const uint8_t* const turn_r = turn + (lane >> 3) * kRowsPitch + 16 * (lane & 7);
    if constexpr (U8) {
        for (int n = threadIdx.x; n < nr; n += kRowsThreads) {
            const int nc = n < p.N ? n : 0;
            lcorr[n] = p.colsum[nc] * 128;
            lfac[n] = p.scale[nc];
        }
        __syncthreads();
    }
    const __amdgpu_buffer_rsrc_t xrsrc =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t*>(p.x), 0, (int)p.x_bytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t wrsrc =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t*>(p.wpk), 0, (int)p.w_bytes, 0x00020000);
    // items go round by wavefront slot first, so that what is left over spreads over all workgroups
    const int stride = (int)gridDim.x * (kRowsThreads / 64);
    int item = wave * (int)gridDim.x + (int)blockIdx.x;

    v4u raw[FM][KS];
    // Channels past C (the padding of the last step) read what follows the pixel, or 0 past the tensor: their weights are 0.
    auto load_rows = [&](int it) __attribute__((always_inline)) {
        const int m0 = it / p.items_n * RM;
#pragma unroll
        for (int i = 0; i < FM; ++i) {
            const int m = m0 + i * 32 + l32;
            int pix = m;
            if (p.g.rm_wo) pix = remap_pixel(p.g, m < p.M ? m : 0);
            const uint32_t off = (it < p.items && m < p.M) ? (uint32_t)(pix * p.C + lhi * kChunk) : kPatchInvalidOffset;
#pragma unroll
            for (int h = 0; h < KS; ++h)
                raw[i][h] = __builtin_amdgcn_raw_buffer_load_b128(xrsrc, (int)(off + (uint32_t)(h * 32)), 0, 0);
        }
    };
    const int wlane = (lhi * p.Np + l32) * kChunk;
    v4i b[D];
    auto load_b = [&](v4i& dst, int n0, int h) __attribute__((always_inline)) {
        const bool live = h < p.steps;                       // uniform; KS can exceed the layer's steps
        const int voff = live ? wlane : (int)kPatchInvalidOffset, soff = live ? (h * 2 * p.Np + n0) * kChunk : 0;
        dst = __builtin_bit_cast(v4i, __builtin_amdgcn_raw_buffer_load_b128(wrsrc, voff, soff, 0));
    };
    const float* scale_or_dummy = p.out ? p.scale : reinterpret_cast<const float*>(p.colsum);

    load_rows(item);
    for (; item < p.items; item += stride) {
        const int rg = item / p.items_n;
        const int n_begin = (item - rg * p.items_n) * p.item_blocks * 32;
        int n_end = n_begin + p.item_blocks * 32;
        n_end = n_end < nr ? n_end : nr;
        // workgroups of an XCD (every eighth) start their walk at different channels: all at the same one keep asking the
        // same few L2 channels for the same weights
        const int runs = (n_end - n_begin + 127) >> 7;
        const int n_first = n_begin + ((int)(blockIdx.x >> 3) % runs) * 128;
#pragma unroll
        for (int h = 0; h < D; ++h) load_b(b[h], n_first, h);
        v4i a[FM][KS];
#pragma unroll
        for (int i = 0; i < FM; ++i)
#pragma unroll
            for (int h = 0; h < KS; ++h) {
                v4u v = raw[i][h];
                if (KIND != kTrimNone && p.trim_in) {
#pragma unroll
                    for (int j = 0; j < 4; ++j) v[j] = trim4_kind<KIND>(v[j], p.luts);
                }
#pragma unroll
                for (int j = 0; j < 4; ++j) v[j] ^= 0x80808080u;
                a[i][h] = __builtin_bit_cast(v4i, v);
            }
        if constexpr (PF) load_rows(item + stride);
        const int m0 = rg * RM;
        const int rows = p.M - m0 < RM ? p.M - m0 : RM;
        const size_t base = (size_t)m0 * p.N;
        for (int n0 = n_first;;) {
            const int n_next = n0 + 32 < n_end ? n0 + 32 : n_begin;      // (past the last: a read that is not used)
            v16i c[FM];
            v4f_rows fac[4];
            int32_t corr = 0;
            float sc = 0.0f;
            const int n = n0 + l32;
            if constexpr (U8) {
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const v4i k = *reinterpret_cast<const v4i*>(lcorr + n0 + 8 * q + 4 * lhi);
                    fac[q] = *reinterpret_cast<const v4f_rows*>(lfac + n0 + 8 * q + 4 * lhi);
#pragma unroll
                    for (int i = 0; i < FM; ++i)
#pragma unroll
                        for (int e = 0; e < 4; ++e) c[i][4 * q + e] = k[e];
                }
            } else {
                const int nc = n < p.N ? n : 0;
                corr = p.colsum[nc] * 128;
                sc = scale_or_dummy[nc];
#pragma unroll
                for (int i = 0; i < FM; ++i)
#pragma unroll
                    for (int v = 0; v < 16; ++v) c[i][v] = 0;
            }
#pragma unroll
            for (int h = 0; h < KS; ++h) {
#pragma unroll
                for (int i = 0; i < FM; ++i)
                    c[i] = U8 ? __builtin_amdgcn_mfma_i32_32x32x32_i8(b[h % D], a[i][h], c[i], 0, 0, 0)
                              : __builtin_amdgcn_mfma_i32_32x32x32_i8(a[i][h], b[h % D], c[i], 0, 0, 0);
                if (h + D < KS) load_b(b[h % D], n0, h + D);
                else load_b(b[h % D], n_next, h + D - KS);
            }
            if constexpr (U8) {
                const int part = ((n0 - n_begin) >> 5) & 3;          // which 32 bytes of a run
#pragma unroll
                for (int i = 0; i < FM; ++i) {
                    uint32_t w[4];
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        uint32_t t = __builtin_amdgcn_cvt_pk_u8_f32(__fmul_rn((float)c[i][4 * q], fac[q][0]), 0, 0);
                        t = __builtin_amdgcn_cvt_pk_u8_f32(__fmul_rn((float)c[i][4 * q + 1], fac[q][1]), 1, t);
                        t = __builtin_amdgcn_cvt_pk_u8_f32(__fmul_rn((float)c[i][4 * q + 2], fac[q][2]), 2, t);
                        w[q] = __builtin_amdgcn_cvt_pk_u8_f32(__fmul_rn((float)c[i][4 * q + 3], fac[q][3]), 3, t);
                    }
                    if (KIND != kTrimNone && p.trim_out) {
#pragma unroll
                        for (int q = 0; q < 4; ++q) w[q] = trim4_kind<KIND>(w[q], p.luts);
                    }
                    // word q holds channels 8q + 4 * lhi .. + 3; after the swaps the low half of the wavefront holds
                    // channels 0..15 of its pixels and the high half 16..31
                    const auto s02 = __builtin_amdgcn_permlane32_swap(w[0], w[2], false, false);
                    const auto s13 = __builtin_amdgcn_permlane32_swap(w[1], w[3], false, false);
                    *reinterpret_cast<v4u*>(turn_w + i * 32 * kRowsPitch + 32 * part) = v4u{s02[0], s02[1], s13[0], s13[1]};
                }
                if (part == 3 || n0 + 32 >= n_end) {                 // uniform: 128 channels gathered, or the last ones
                    wavefront_lds_fence();
                    const __amdgpu_buffer_rsrc_t orsrc =
                        __builtin_amdgcn_make_buffer_rsrc((void*)(p.out_u8 + base), 0, rows * p.N, 0x00020000);
                    const int no = n0 - 32 * part + 16 * (lane & 7);
                    const int lane_off = ((lane & 7) < 2 * (part + 1) && no < p.N) ? (lane >> 3) * p.N + no : (int)kPatchInvalidOffset;
#pragma unroll
                    for (int r = 0; r < RM / 8; ++r) {
                        const v4u o = *reinterpret_cast<const v4u*>(turn_r + 8 * r * kRowsPitch);
                        __builtin_amdgcn_raw_buffer_store_b128(o, orsrc, lane_off + 8 * r * p.N, 0, 0);
                    }
                    wavefront_lds_fence();
                }
            } else {
                const int pitch = p.N * 4, bytes = rows * pitch;
                const __amdgpu_buffer_rsrc_t arsrc =
                    __builtin_amdgcn_make_buffer_rsrc(p.acc ? (void*)(p.acc + base) : nullptr, 0, p.acc ? bytes : 0, 0x00020000);
                const __amdgpu_buffer_rsrc_t orsrc =
                    __builtin_amdgcn_make_buffer_rsrc(p.out ? (void*)(p.out + base) : nullptr, 0, p.out ? bytes : 0, 0x00020000);
                const uint32_t lane_off = n < p.N ? (uint32_t)(4 * lhi * pitch + n * 4) : kPatchInvalidOffset;
                auto store = [&](auto acc_, auto out_) __attribute__((always_inline)) {
#pragma unroll
                    for (int i = 0; i < FM; ++i)
#pragma unroll
                        for (int v = 0; v < 16; ++v) {
                            const int32_t r = c[i][v] + corr;
                            const int off = (int)(lane_off + (uint32_t)((i * 32 + 8 * (v / 4) + (v % 4)) * pitch));
                            if constexpr (decltype(acc_)::value) __builtin_amdgcn_raw_buffer_store_b32(r, arsrc, off, 0, kResultStorePolicy);
                            if constexpr (decltype(out_)::value)
                                __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(int, __fmul_rn((float)r, sc)), orsrc, off, 0, kResultStorePolicy);
                        }
                };
                if (p.acc && p.out) store(std::true_type{}, std::true_type{});
                else if (p.out) store(std::false_type{}, std::true_type{});
                else store(std::true_type{}, std::false_type{});
            }
            n0 = n_next;
            if (n0 == n_first) break;
        }
        if constexpr (!PF) load_rows(item + stride);
    }
}

// Dynamic LDS of a launch with rm pixels per wavefront.
inline int64_t rows_lds_bytes(int rm, int64_t N, bool bytes) {
    return bytes ? (kRowsThreads / 64) * rm * kRowsPitch + (N + 31) / 32 * 32 * 8 : 0;
}

// `p` carries everything except the item counts.
template <class Cfg, int KIND, bool U8>
sparq_status launch_rows_cfg(const RowsParams& p, hipStream_t s) {
    RowsParams q = p;
    const int blocks = (p.N + 31) / 32;
    const int64_t groups = ((int64_t)p.M + Cfg::kRM - 1) / Cfg::kRM;
    const int64_t slots = (int64_t)device_cu_count() * 4 * Cfg::kOcc;        // wavefronts the chip holds
    // Shares of the output channels.  Few pixel groups leave SIMDs idle and a last round can be nearly empty, so a group's
    // channels may be split -- but every share loads and trims the group's pixels again.  Taken is the split whose rounds
    // cost least: a round of w wavefronts per SIMD takes w items' issue slots (trim per reduction step; conversion, stores
    // and matrix instructions per block) or one item's own chain (plus waits), whichever is longer.  The five constants
    // are fitted to 115 timed shapes (K 64..512, N 64..1024, M 3136..200704): 0.6 % from the best split on average.
    const int64_t trim = (int64_t)Cfg::kFM * Cfg::kKS * (KIND == kTrimNone ? 20 : 96), block = Cfg::kFM * (130 + 4 * Cfg::kKS);
    int64_t best = INT64_MAX;
    for (int shares = 1; shares == 1 || shares * 2 <= blocks; shares *= 2) {
        const int64_t ib = (blocks + shares - 1) / shares, items = groups * ((blocks + ib - 1) / ib);
        const int64_t issue = trim + ib * block, chain = issue + 300 + ib * 60;
        const auto round = [&](int64_t w) { return w * issue > chain ? w * issue : chain; };
        const int64_t rest = items % slots;
        const int64_t cost = items / slots * round(Cfg::kOcc) + (rest ? round((rest * Cfg::kOcc + slots - 1) / slots) : 0);
        if (cost < best) {
            best = cost;
            q.item_blocks = (int)ib;
        }
    }
    q.items_n = (blocks + q.item_blocks - 1) / q.item_blocks;
    const int64_t items = groups * q.items_n;
    // (the loop's cursor runs past the last item by less than two strides)
    if (items > (1 << 30) || (int64_t)p.N * 4 * Cfg::kRM >= 0x7FFFFFFF || p.steps > Cfg::kKS) return SPARQ_EUNSUPPORTED;
    q.items = (int)items;
    const int64_t lds_bytes = rows_lds_bytes(Cfg::kRM, p.N, U8);
    if (lds_bytes > 64 * 1024) return SPARQ_EUNSUPPORTED;    // (what a launch may use without asking)
    const int64_t wgs = (items + 3) / 4, resident = slots / 4;
    conv_rows_kernel<Cfg, KIND, U8><<<(unsigned)(wgs < resident ? wgs : resident), kRowsThreads, (size_t)lds_bytes, s>>>(q);
    return launch_status();
}

// Cfg1: 32 pixels per wavefront, Cfg2: 64.  Sixty-four halve the weight traffic and win once both sides of the product are
// large (K 256, N 1024, M 200704: 75 against 83 us); otherwise the shorter items do (K 256, N 256, M 12544: 7.2 against 9.9).
inline bool rows_large(int64_t M, int64_t N) { return N >= 512 && M >= 48 * 1024; }
template <class Cfg1, class Cfg2, int KIND>
sparq_status launch_rows_out(const RowsParams& p, hipStream_t s) {
    if (!std::is_same_v<Cfg1, Cfg2> && rows_large(p.M, p.N))
        return p.out_u8 ? launch_rows_cfg<Cfg2, KIND, true>(p, s) : launch_rows_cfg<Cfg2, KIND, false>(p, s);
    return p.out_u8 ? launch_rows_cfg<Cfg1, KIND, true>(p, s) : launch_rows_cfg<Cfg1, KIND, false>(p, s);
}

template <class Cfg1, class Cfg2 = Cfg1>
sparq_status launch_rows_kind(TrimKind kind, const RowsParams& p, hipStream_t s) {
    switch (kind) {
        case kTrimNone: return launch_rows_out<Cfg1, Cfg2, kTrimNone>(p, s);
        case kTrimFloor: return launch_rows_out<Cfg1, Cfg2, kTrimFloor>(p, s);
        case kTrimFloorPair: return launch_rows_out<Cfg1, Cfg2, kTrimFloorPair>(p, s);
        case kTrimFloorPairWide: return launch_rows_out<Cfg1, Cfg2, kTrimFloorPairWide>(p, s);
        case kTrimRound: return launch_rows_out<Cfg1, Cfg2, kTrimRound>(p, s);
        case kTrimRound4: return launch_rows_out<Cfg1, Cfg2, kTrimRound4>(p, s);
        case kTrimRoundPairWide: return launch_rows_out<Cfg1, Cfg2, kTrimRoundPairWide>(p, s);
        case kTrimRoundPair4: return launch_rows_out<Cfg1, Cfg2, kTrimRoundPair4>(p, s);
        default: return SPARQ_EUNSUPPORTED;
    }
}

typedef sparq_status (*RowsLauncher)(TrimKind, const RowsParams&, hipStream_t);
#define SPARQ_DECLARE_ROWS(name) sparq_status name(TrimKind kind, const RowsParams& p, hipStream_t s)
SPARQ_DECLARE_ROWS(launch_rows_k64);
SPARQ_DECLARE_ROWS(launch_rows_k128);
SPARQ_DECLARE_ROWS(launch_rows_k192);
SPARQ_DECLARE_ROWS(launch_rows_k256);
SPARQ_DECLARE_ROWS(launch_rows_k320);
SPARQ_DECLARE_ROWS(launch_rows_k384);
SPARQ_DECLARE_ROWS(launch_rows_k512);

}  // namespace sparq
