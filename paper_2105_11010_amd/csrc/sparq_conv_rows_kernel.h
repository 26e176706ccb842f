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
// Many pixels and few enough weights: one workgroup per CU holds all of them in LDS, and memory is what bounds the layer (launch_rows_held,
// where the figures are).  Otherwise the weights come from L2, and with 256 channels and more they and the trim's vector instructions
// bound it; wide layers of 256 channels and more hold the weights instead (sparq_conv_cols_kernel.h).  By the counters, bytes, weights in LDS: 64 channels
// vector issue 67 % of the cycles, the matrix pipeline 13, waits 35 % of a wavefront's life; 256 channels 59, 12 and 20.
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

// KS 32-index steps of activations in registers, FM fragments of 32 pixels per wavefront, PF: the next pixels are requested
// while the current ones are multiplied, OCC wavefronts per SIMD.
template <int KS, int FM, bool PF, int OCC, bool WL = false, int RUN = 128>
struct RowsCfg {
    static constexpr int kKS = KS, kFM = FM, kOcc = OCC, kRM = 32 * FM, kRun = RUN, kPitch = RUN + 16;
    static constexpr bool kPF = PF, kWL = WL;
    static constexpr int kThreads = WL ? 256 * OCC : kRowsThreads;
    // weight steps requested ahead; divides KS
    static constexpr int kRing = WL ? (KS % 4 == 0 ? 4 : KS % 5 == 0 ? 5 : KS % 3 == 0 ? 3 : KS) : KS % 8 == 0 ? 8 : KS % 6 == 0 ? 6 : KS % 5 == 0 ? 5 : KS;
    static_assert(KS % kRing == 0, "ring slots are fixed per step");
};

template <class Cfg, int KIND, bool U8>
__global__ __launch_bounds__(Cfg::kThreads, Cfg::kOcc) void conv_rows_kernel(const RowsParams p) {
    constexpr int KS = Cfg::kKS, FM = Cfg::kFM, RM = Cfg::kRM, D = Cfg::kRing;
    constexpr bool PF = Cfg::kPF, WL = Cfg::kWL;
    constexpr int NT = Cfg::kThreads, PITCH = Cfg::kPitch, LPR = Cfg::kRun / 16, RPR = 64 / LPR;       // lanes per row, rows per store
    // U8: a wavefront's bytes on their way out, then [corr | factor] of all channels
    extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
    const int lane = threadIdx.x & 63, l32 = lane & 31, lhi = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int nr = (p.N + 31) & ~31;
    int32_t* lcorr = reinterpret_cast<int32_t*>(lds + (NT / 64) * RM * PITCH);
    float* lfac = reinterpret_cast<float*>(lcorr) + nr;
    // turned through LDS (the wavefront's own area, no barrier): a lane writes 16 bytes of its pixel per block and reads
    // 16 bytes of the row its group of eight lanes stores
    uint8_t* const turn = lds + wave * RM * PITCH;
    uint8_t* const turn_w = turn + l32 * PITCH + 16 * lhi;
    const uint8_t* const turn_r = turn + lane / LPR * PITCH + 16 * (lane % LPR);
    if constexpr (U8) {
        for (int n = threadIdx.x; n < nr; n += NT) {
            const int nc = n < p.N ? n : 0;
            lcorr[n] = p.colsum[nc] * 128;
            lfac[n] = p.scale[nc];
        }
        if constexpr (!WL) __syncthreads();
    }
    const __amdgpu_buffer_rsrc_t xrsrc =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t*>(p.x), 0, (int)p.x_bytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t wrsrc =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t*>(p.wpk), 0, (int)p.w_bytes, 0x00020000);
    // items go round by wavefront slot first, so that what is left over spreads over all workgroups
    const int stride = (int)gridDim.x * (NT / 64);
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
    // WL: the weights as 32-channel blocks of [step][half][channel][16 bytes]
    uint8_t* const lw = U8 ? reinterpret_cast<uint8_t*>(lfac + nr) : lds;
    const uint8_t* const lw_lane = lw + (lhi * 32 + l32) * kChunk;
    auto load_b = [&](v4i& dst, int n0, int h) __attribute__((always_inline)) {
        if constexpr (WL) {
            dst = *reinterpret_cast<const v4i*>(lw_lane + n0 * KS * 32 + h * 1024);
            return;
        }
        const bool live = h < p.steps;                       // uniform; KS can exceed the layer's steps
        const int voff = live ? wlane : (int)kPatchInvalidOffset, soff = live ? (h * 2 * p.Np + n0) * kChunk : 0;
        dst = __builtin_bit_cast(v4i, __builtin_amdgcn_raw_buffer_load_b128(wrsrc, voff, soff, 0));
    };
    const float* scale_or_dummy = p.out ? p.scale : reinterpret_cast<const float*>(p.colsum);

    load_rows(item);
    if constexpr (WL) {
        for (int q = threadIdx.x; q < nr * KS * 2; q += NT) {
            const int blk = q / (KS * 64), k16 = q % (KS * 64) / 32, n = blk * 32 + q % 32;
            const int off = k16 < 2 * p.steps ? (k16 * p.Np + n) * kChunk : (int)kPatchInvalidOffset;          // (past the last step: 0)
            *reinterpret_cast<v4u*>(lw + q * kChunk) = __builtin_amdgcn_raw_buffer_load_b128(wrsrc, off, 0, 0);
        }
        __syncthreads();
    }
    for (; item < p.items; item += stride) {
        const int rg = item / p.items_n;
        const int n_begin = (item - rg * p.items_n) * p.item_blocks * 32;
        int n_end = n_begin + p.item_blocks * 32;
        n_end = n_end < nr ? n_end : nr;
        // workgroups of an XCD (every eighth) start their walk at different channels: all at the same one keep asking the
        // same few L2 channels for the same weights
        const int runs = (n_end - n_begin + 127) >> 7;
        const int n_first = WL ? n_begin : n_begin + ((int)(blockIdx.x >> 3) % runs) * 128;
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
                // (left to itself the compiler puts some variants' requests right in front of their use: 320 -> 512, 132278 pixels, bytes
                // 64 us, so 49)
                __builtin_amdgcn_sched_barrier(0x0006);      // vector and scalar arithmetic may cross
            }
            if constexpr (U8) {
                const int part = (n0 - n_begin) / 32 % (Cfg::kRun / 32);     // which 32 bytes of a run
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
                    *reinterpret_cast<v4u*>(turn_w + i * 32 * PITCH + 32 * part) = v4u{s02[0], s02[1], s13[0], s13[1]};
                }
                if (part == Cfg::kRun / 32 - 1 || n0 + 32 >= n_end) {        // uniform: a run gathered, or the last channels
                    wavefront_lds_fence();
                    const __amdgpu_buffer_rsrc_t orsrc =
                        __builtin_amdgcn_make_buffer_rsrc((void*)(p.out_u8 + base), 0, rows * p.N, 0x00020000);
                    const int no = n0 - 32 * part + 16 * (lane % LPR);
                    const int lane_off = (lane % LPR < 2 * (part + 1) && no < p.N) ? lane / LPR * p.N + no : (int)kPatchInvalidOffset;
#pragma unroll
                    for (int r = 0; r < RM / RPR; ++r) {
                        const v4u o = *reinterpret_cast<const v4u*>(turn_r + RPR * r * PITCH);
                        __builtin_amdgcn_raw_buffer_store_b128(o, orsrc, lane_off + RPR * r * p.N, 0, 0);
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
    return bytes ? (kRowsThreads / 64) * rm * (128 + 16) + (N + 31) / 32 * 32 * 8 : 0;
}
// ... with the weights in LDS.
template <class Cfg>
int64_t rows_held_lds_bytes(int64_t N, bool bytes) {
    const int64_t nr = (N + 31) / 32 * 32;
    return (bytes ? Cfg::kThreads / 64 * Cfg::kRM * Cfg::kPitch + nr * 8 : 0) + nr * Cfg::kKS * 32;
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

// The same with the weights in LDS, one workgroup per CU.
template <class Cfg, int KIND, bool U8>
sparq_status launch_rows_held_cfg(const RowsParams& p, hipStream_t s) {
    RowsParams q = p;
    q.item_blocks = (p.N + 31) / 32;
    q.items_n = 1;
    q.items = (int)(((int64_t)p.M + Cfg::kRM - 1) / Cfg::kRM);
    const int64_t lds_bytes = rows_held_lds_bytes<Cfg>(p.N, U8);
    if (lds_bytes > kLdsPerCu || (int64_t)p.N * 4 * Cfg::kRM >= 0x7FFFFFFF || p.steps > Cfg::kKS) return SPARQ_EUNSUPPORTED;
    auto kern = conv_rows_kernel<Cfg, KIND, U8>;
    static std::atomic<bool> lds_set_dev[kMaxDevices];       // (concurrent callers at worst repeat the call, with the same value)
    std::atomic<bool>& lds_set = lds_set_dev[current_device_slot()];
    if (!lds_set.load(std::memory_order_relaxed) || current_device_slot() == kMaxDevices - 1) {
        if (hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, kLdsPerCu) != hipSuccess)
            return SPARQ_ELAUNCH;
        lds_set.store(true, std::memory_order_relaxed);
    }
    const int64_t wgs = ((int64_t)q.items + Cfg::kThreads / 64 - 1) / (Cfg::kThreads / 64), cus = device_cu_count();
    kern<<<(unsigned)(wgs < cus ? wgs : cus), Cfg::kThreads, (size_t)lds_bytes, s>>>(q);
    return launch_status();
}

// KS steps: wavefronts per SIMD are what the registers allow (bytes: what the result rows leave LDS for, too); 512 channels without the
// next pixels requested ahead, 512 -> 128 channels, 200704 pixels, bytes: 39.2 us (41.1 with, and two wavefronts per SIMD).
template <int KS, bool U8>
struct RowsHeld {
    typedef RowsCfg<KS, 1, KS <= 12, U8 ? (KS == 2 ? 4 : 3) : KS <= 8 ? 4 : 3, true> Main;
    typedef RowsCfg<KS, 1, true, 2, true, 64> Large;         // bytes: fewer result rows, half as long, and room for more weights
};

// Weights in LDS where they fit and every wavefront slot has pixels of its own.  A wavefront otherwise asks L1 for all weights once per 32
// pixels, 64 bytes a cycle for the whole CU and at the latency of L2 (13 to 23 % of such layers when the requests were left out).  Measured
// cold, us before -> after: bytes, 256 -> 128, 802816 pixels 98 -> 69; 256 -> 64 76 -> 59; 64 -> 256 72 -> 57; 512 -> 128, 200704 pixels
// 48 -> 41; fp32, 288 -> 48, 156800 pixels 25.8 -> 20.9, 192 -> 48 17.5 -> 13.2.  Warm, 2321 drawn layers with pixels for every slot:
// bytes 1.08 x (7 of 1403 below 0.95, the lowest 0.91; 0.94 x with half the pixels).  Four-byte results up to 64 outputs 1.05 x, but with more
// than 256 channels 0.96 x up to 1.3 rounds (lowest 0.86, the second round nearly empty); up to 128 from two rounds on 1.04, up to 96 of more than
// 256 channels from 1.5 on as much faster as slower warm (0.85 to 1.05), cold 27.1 -> 21.8 (288 -> 96; 26328 layers
// of up to 128 outputs on 16 buffers in turn: 33 outputs and more in up to 2.5 rounds 1.04-1.2, on the same ones 0.95-1.03); wider ones are bound by their stores and
// lose as much as they gain (0.78 to 1.1).  More weights than fit beside three wavefronts per SIMD, bytes, up to 128 KB: 1.13 x from three rounds of
// two on, but 0.98 x with up to 256 channels.
// Returns the bytes of a result row that leave together (128: Main, 64: Large); 0: the weights stay in L2.
template <int KS, bool U8>
int rows_held_run(int64_t M, int64_t N) {
    typedef typename RowsHeld<KS, U8>::Main Main;
    const int64_t items = (M + 31) / 32, simds = (int64_t)device_cu_count() * 4, slots = simds * Main::kOcc;
    if (rows_held_lds_bytes<Main>(N, U8) <= kLdsPerCu) {
        constexpr bool SHORT = KS <= 8;
        const int64_t tenths = U8 ? 10 : N <= 64 ? (SHORT ? 11 : 14) : N <= 96 && !SHORT ? 15 : N <= 128 ? 20 : INT64_MAX / (slots + 1);
        return items * 10 >= slots * tenths ? Main::kRun : 0;
    }
    typedef typename RowsHeld<KS, U8>::Large Large;
    return U8 && KS > 8 && rows_held_lds_bytes<Large>(N, U8) <= kLdsPerCu && items >= simds * 6 ? Large::kRun : 0;
}
template <int KS>
int rows_held_run(int64_t M, int64_t N, bool bytes) { return bytes ? rows_held_run<KS, true>(M, N) : rows_held_run<KS, false>(M, N); }

template <int KS, int KIND, bool U8>
sparq_status launch_rows_held(const RowsParams& p, hipStream_t s) {
    typedef typename RowsHeld<KS, U8>::Main Main;
    const int run = rows_held_run<KS, U8>(p.M, p.N);
    if (run == Main::kRun) return launch_rows_held_cfg<Main, KIND, U8>(p, s);
    if constexpr (U8 && KS > 8) {
        typedef typename RowsHeld<KS, U8>::Large Large;
        if (run == Large::kRun) return launch_rows_held_cfg<Large, KIND, U8>(p, s);
    }
    return SPARQ_EUNSUPPORTED;
}

// Cfg1: 32 pixels per wavefront, Cfg2: 64.  Sixty-four halve the weight traffic and win once both sides of the product are
// large (K 256, N 1024, M 200704: 75 against 83 us); otherwise the shorter items do (K 256, N 256, M 12544: 7.2 against 9.9).
inline bool rows_large(int64_t M, int64_t N) { return N >= 512 && M >= 48 * 1024; }
template <class Cfg1, class Cfg2, int KIND>
sparq_status launch_rows_out(const RowsParams& p, hipStream_t s) {
    const sparq_status st = p.out_u8 ? launch_rows_held<Cfg1::kKS, KIND, true>(p, s) : launch_rows_held<Cfg1::kKS, KIND, false>(p, s);
    if (st != SPARQ_EUNSUPPORTED) return st;
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
