// Fused SPARQ convolution for gfx950, 1x1 filters of up to 1024 channels and more output channels: the weights stay in registers.
//
// The form with the activations in registers asks L1 for all weights once per 32 pixels and wavefront, and where pixels are few it splits the
// output channels over wavefronts that each load and trim the same pixels again.  Here a wavefront holds the weights of 64 (or 32) output channels
// for the whole launch, 64 to 128 registers of them, and the pixels pass by: a workgroup of eight wavefronts, one per CU, walks its share of the
// pixels in tiles of 32 or 64, trimmed once for all of its channels into one of two LDS buffers while the tile before is multiplied (256 KB of
// weights per CU and launch instead of per 384 pixels).  A CU's share is counted in fragments of 32 pixels, so that CUs differ by one fragment;
// where all channels need more than eight wavefronts, workgroups of one XCD share the pixels in its L2.
// Up to 256 channels the requantisation's offsets and factors stay in registers, too (as the first matrix instruction's addend the offsets cost
// nothing); beyond, they come from LDS.
// The two wavefronts of a SIMD stage at opposite ends of a tile, so that one multiplies while the other trims or converts.
// Cold, bytes, us before -> after: 256 -> 1024, 50176 pixels 28.5 -> 25.1; 256 -> 512/2, 200704 pixels 57.9 -> 44.8; 512 -> 256 56.2 -> 44.7;
// 512 -> 1024/2, 50176 pixels 48.1 -> 36.0; 512 -> 2048, 12544 pixels 26.1 -> 22.5; 1024 -> 256, 50176 pixels 30.0 -> 26.7; fp32, 768 -> 192, 36992
// pixels 22.8 -> 18.4.
// Bound by vector arithmetic and the stores: per pixel 256 -> 1024 takes 1.4 times as long as a copy of its bytes, and 7 us are the first
// loads, weights and trim.  (Vector issue 53 % of the cycles, the matrix pipeline 29, waits 34 % of a wavefront's
// life; 1024 channels 48, 26 and 38.  Two tiles requested ahead, with the tiles a round of requests
// leaves empty: up to 7 % slower; 16 wavefronts' worth of outputs in two walks instead of two workgroups: within 3 % of this.)
#pragma once
#include "sparq_conv_rows_kernel.h"

namespace sparq {

constexpr int kColsThreads = 512;

// KS 32-index steps and 32 FN output channels of weights in a wavefront's registers; WM wavefronts hold the same ones, each with TI fragments
// of 32 pixels per tile.
template <int KS, int FN, int WM, int TI>
struct ColsCfg {
    static constexpr int kKS = KS, kFN = FN, kWM = WM, kTI = TI, kTF = WM * TI;
    static constexpr bool kTable = KS > 8;                   // bytes: what belongs to the channels stands in LDS, not in registers
    static constexpr int kTableBytes = kTable ? 8 / WM * 32 * FN * 8 : 0;
    static constexpr int kPlane = kTF * 32 * kChunk + 16;    // bytes between a buffer's 16-channel planes
    static constexpr int kBuf = 2 * KS * kPlane;
    static constexpr int kRequests = kTF * 32 * 2 * KS / kColsThreads;       // 16-byte chunks a lane stages per tile
    static constexpr int kPitch = 32 * FN + 16;              // LDS row of result bytes
    static_assert(kRequests * kColsThreads == kTF * 32 * 2 * KS && 8 % WM == 0, "every lane stages the same");
};

struct ColsParams {
    RowsParams r;
    int shares;              // the output channels are split over this many workgroups ...
    int share_groups;        // ... groups of 32 FN channels each
    int wgs;                 // workgroups per share
    int per_wg, one_more;    // fragments of 32 pixels per workgroup; the first one_more take one more
};

template <class Cfg, int KIND, bool U8>
__global__ __launch_bounds__(kColsThreads, 2) void conv_cols_kernel(const ColsParams cp) {
    const RowsParams& p = cp.r;
    constexpr int KS = Cfg::kKS, FN = Cfg::kFN, WM = Cfg::kWM, TI = Cfg::kTI, TF = Cfg::kTF, CH = 2 * KS, NR = Cfg::kRequests, PITCH = Cfg::kPitch;
    constexpr bool LT = Cfg::kTable && U8;
    constexpr int LPR = 2 * FN, RPR = 64 / LPR;              // lanes per result row, rows per store
    extern __shared__ __attribute__((aligned(16))) uint8_t lds[];            // [buffers][U8: result rows per wavefront]
    const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, lhi = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave % WM, wn = wave / WM;
    // (an XCD runs every eighth workgroup: the shares of the same pixels run on the same one)
    const int turn8 = (int)blockIdx.x >> 3, share = turn8 % cp.shares, wg = turn8 / cp.shares * 8 + ((int)blockIdx.x & 7);
    if (wg >= cp.wgs) return;
    const int f0 = wg * cp.per_wg + (wg < cp.one_more ? wg : cp.one_more), f1 = f0 + cp.per_wg + (wg < cp.one_more ? 1 : 0);
    const int nt = (f1 - f0 + TF - 1) / TF;
    const int m_end = f1 * 32 < p.M ? f1 * 32 : p.M;
    const __amdgpu_buffer_rsrc_t xrsrc =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t*>(p.x), 0, (int)p.x_bytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t wrsrc =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t*>(p.wpk), 0, (int)p.w_bytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t krsrc =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<int32_t*>(p.colsum), 0, p.Np * 4, 0x00020000);
    const __amdgpu_buffer_rsrc_t frsrc =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(p.scale), 0, p.scale ? p.N * 4 : 0, 0x00020000);

    // ---- activations: a tile's chunks go round over the lanes, a pixel's side by side ----
    v4u raw[NR];
    auto load_x = [&](int t) __attribute__((always_inline)) {
#pragma unroll
        for (int r = 0; r < NR; ++r) {
            const int q = tid + kColsThreads * r, ch = q % CH, m = (f0 + t * TF) * 32 + q / CH;
            const bool live = m < m_end && ch < 2 * p.steps;
            int pix = m;
            if (p.g.rm_wo) pix = remap_pixel(p.g, live ? m : 0);
            const uint32_t off = live ? (uint32_t)(pix * p.C + ch * kChunk) : kPatchInvalidOffset;
            raw[r] = __builtin_amdgcn_raw_buffer_load_b128(xrsrc, (int)off, 0, 0);
        }
    };
    auto stage = [&](int buf) __attribute__((always_inline)) {
#pragma unroll
        for (int r = 0; r < NR; ++r) {
            const int q = tid + kColsThreads * r;
            v4u v = raw[r];
            if (KIND != kTrimNone && p.trim_in) {
#pragma unroll
                for (int j = 0; j < 4; ++j) v[j] = trim4_kind<KIND>(v[j], p.luts);
            }
#pragma unroll
            for (int j = 0; j < 4; ++j) v[j] ^= 0x80808080u;
            *reinterpret_cast<v4u*>(lds + buf * Cfg::kBuf + q % CH * Cfg::kPlane + q / CH * kChunk) = v;
        }
    };

    // ---- weights and what belongs to the channels ----
    v4i b[FN][KS];
    v16i corr[U8 && !LT ? FN : 1];
    float fac[U8 && !LT ? FN : 1][16];
    int32_t corr1[FN];
    float sc1[FN];
    int n0 = 0;
    auto load_b = [&]() __attribute__((always_inline)) {
        n0 = wn < cp.share_groups ? (share * cp.share_groups + wn) * 32 * FN : p.Np;           // (no such channels: 0)
#pragma unroll
        for (int j = 0; j < FN; ++j) {
            const int n = n0 + 32 * j + l32;
#pragma unroll
            for (int h = 0; h < KS; ++h) {
                const int off = h < p.steps && n < p.Np ? ((2 * h + lhi) * p.Np + n) * kChunk : (int)kPatchInvalidOffset;
                b[j][h] = __builtin_bit_cast(v4i, __builtin_amdgcn_raw_buffer_load_b128(wrsrc, off, 0, 0));
            }
            if constexpr (LT) continue;
            if constexpr (U8) {
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int off = (n0 + 32 * j + 8 * q + 4 * lhi) * 4;
                    const v4i k = __builtin_bit_cast(v4i, __builtin_amdgcn_raw_buffer_load_b128(krsrc, off, 0, 0));
                    const v4f_rows f = __builtin_bit_cast(v4f_rows, __builtin_amdgcn_raw_buffer_load_b128(frsrc, off, 0, 0));
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        corr[j][4 * q + e] = k[e] * 128;
                        fac[j][4 * q + e] = f[e];
                    }
                }
            } else {
                corr1[j] = (int)__builtin_amdgcn_raw_buffer_load_b32(krsrc, n * 4, 0, 0) * 128;
                sc1[j] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(frsrc, n * 4, 0, 0));
            }
        }
    };

    // (waits for all of it at once: inside the walk such a wait would be for the pixels requested since, too)
    auto settle_b = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < FN; ++j) {
#pragma unroll
            for (int h = 0; h < KS; ++h) asm volatile("" ::"v"(b[j][h]));
            if constexpr (LT) continue;
            if constexpr (U8) {
#pragma unroll
                for (int e = 0; e < 16; ++e) asm volatile("" ::"v"(fac[j][e]), "v"(corr[j][e]));
            } else {
                asm volatile("" ::"v"(sc1[j]), "v"(corr1[j]));
            }
        }
    };

    // LT: [corr | factor] of the workgroup's channels
    int32_t* const tcorr = reinterpret_cast<int32_t*>(lds + 2 * Cfg::kBuf + 8 * 32 * PITCH);
    float* const tfac = reinterpret_cast<float*>(tcorr) + 8 / WM * 32 * FN;
    const int tn = wn * 32 * FN + 4 * lhi;
    uint8_t* const turn = lds + 2 * Cfg::kBuf + wave * 32 * PITCH;
    auto fragment = [&](int t, int i) __attribute__((always_inline)) {
        const int f = f0 + t * TF + i;
        const bool live = f < f1 && n0 < p.N;                // uniform
        const int m0 = f * 32, rows = !live ? 0 : p.M - m0 < 32 ? p.M - m0 : 32;
        const size_t base = (size_t)(live ? m0 : 0) * p.N;
        v16i c[FN];
        if (live) {
            const uint8_t* const at = lds + t % 2 * Cfg::kBuf + lhi * Cfg::kPlane + (i * 32 + l32) * kChunk;
#pragma unroll
            for (int j = 0; j < FN; ++j) {
                if constexpr (LT) {
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const v4i k = *reinterpret_cast<const v4i*>(tcorr + tn + 32 * j + 8 * q);
#pragma unroll
                        for (int e = 0; e < 4; ++e) c[j][4 * q + e] = k[e];
                    }
                } else if constexpr (U8) c[j] = corr[j];
                else
#pragma unroll
                    for (int v = 0; v < 16; ++v) c[j][v] = 0;
            }
            constexpr int AR = KS < 8 ? KS : 8;              // fragments read ahead
            v4i a[AR];
#pragma unroll
            for (int h = 0; h < AR; ++h) a[h] = *reinterpret_cast<const v4i*>(at + 2 * h * Cfg::kPlane);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int h = 0; h < KS; ++h) {
#pragma unroll
                for (int j = 0; j < FN; ++j)
                    c[j] = U8 ? __builtin_amdgcn_mfma_i32_32x32x32_i8(b[j][h], a[h % AR], c[j], 0, 0, 0)
                              : __builtin_amdgcn_mfma_i32_32x32x32_i8(a[h % AR], b[j][h], c[j], 0, 0, 0);
                if (h + AR < KS) a[h % AR] = *reinterpret_cast<const v4i*>(at + 2 * (h + AR) * Cfg::kPlane);
            }
        }
        if constexpr (U8) {
            if (live) {
#pragma unroll
                for (int j = 0; j < FN; ++j) {
                    uint32_t w[4];
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        v4f_rows fac_q;
                        if constexpr (LT) fac_q = *reinterpret_cast<const v4f_rows*>(tfac + tn + 32 * j + 8 * q);
                        else
#pragma unroll
                            for (int e = 0; e < 4; ++e) fac_q[e] = fac[j][4 * q + e];
                        uint32_t o = __builtin_amdgcn_cvt_pk_u8_f32(__fmul_rn((float)c[j][4 * q], fac_q[0]), 0, 0);
                        o = __builtin_amdgcn_cvt_pk_u8_f32(__fmul_rn((float)c[j][4 * q + 1], fac_q[1]), 1, o);
                        o = __builtin_amdgcn_cvt_pk_u8_f32(__fmul_rn((float)c[j][4 * q + 2], fac_q[2]), 2, o);
                        w[q] = __builtin_amdgcn_cvt_pk_u8_f32(__fmul_rn((float)c[j][4 * q + 3], fac_q[3]), 3, o);
                    }
                    if (KIND != kTrimNone && p.trim_out) {
#pragma unroll
                        for (int q = 0; q < 4; ++q) w[q] = trim4_kind<KIND>(w[q], p.luts);
                    }
                    const auto s02 = __builtin_amdgcn_permlane32_swap(w[0], w[2], false, false);
                    const auto s13 = __builtin_amdgcn_permlane32_swap(w[1], w[3], false, false);
                    *reinterpret_cast<v4u*>(turn + l32 * PITCH + 32 * j + 16 * lhi) = v4u{s02[0], s02[1], s13[0], s13[1]};
                }
            }
            wavefront_lds_fence();
            const __amdgpu_buffer_rsrc_t orsrc = __builtin_amdgcn_make_buffer_rsrc((void*)(p.out_u8 + base), 0, rows * p.N, 0x00020000);
            const int no = n0 + 16 * (lane % LPR), lane_off = no < p.N ? lane / LPR * p.N + no : (int)kPatchInvalidOffset;
#pragma unroll
            for (int r = 0; r < 32 / RPR; ++r) {
                const v4u o = *reinterpret_cast<const v4u*>(turn + (lane / LPR + RPR * r) * PITCH + 16 * (lane % LPR));
                __builtin_amdgcn_raw_buffer_store_b128(o, orsrc, lane_off + RPR * r * p.N, 0, 0);
            }
            wavefront_lds_fence();
        } else {
            if (!live) return;
            const int pitch = p.N * 4, bytes = rows * pitch;
            const __amdgpu_buffer_rsrc_t arsrc =
                __builtin_amdgcn_make_buffer_rsrc(p.acc ? (void*)(p.acc + base) : nullptr, 0, p.acc ? bytes : 0, 0x00020000);
            const __amdgpu_buffer_rsrc_t orsrc =
                __builtin_amdgcn_make_buffer_rsrc(p.out ? (void*)(p.out + base) : nullptr, 0, p.out ? bytes : 0, 0x00020000);
            auto store = [&](auto acc_, auto out_) __attribute__((always_inline)) {
#pragma unroll
                for (int j = 0; j < FN; ++j) {
                    const int n = n0 + 32 * j + l32;
                    const uint32_t lane_off = n < p.N ? (uint32_t)(4 * lhi * pitch + n * 4) : kPatchInvalidOffset;
#pragma unroll
                    for (int v = 0; v < 16; ++v) {
                        const int32_t r = c[j][v] + corr1[j];
                        const int off = (int)(lane_off + (uint32_t)((8 * (v / 4) + v % 4) * pitch));
                        if constexpr (decltype(acc_)::value) __builtin_amdgcn_raw_buffer_store_b32(r, arsrc, off, 0, kResultStorePolicy);
                        if constexpr (decltype(out_)::value)
                            __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(int, __fmul_rn((float)r, sc1[j])), orsrc, off, 0, kResultStorePolicy);
                    }
                }
            };
            if (p.acc && p.out) store(std::true_type{}, std::true_type{});
            else if (p.out) store(std::false_type{}, std::true_type{});
            else store(std::true_type{}, std::false_type{});
        }
    };

    load_x(0);
    load_b();
    if constexpr (LT)
        for (int i = tid; i < 8 / WM * 32 * FN; i += kColsThreads) {
            const int off = (share * cp.share_groups * 32 * FN + i) * 4;
            tcorr[i] = (int)__builtin_amdgcn_raw_buffer_load_b32(krsrc, off, 0, 0) * 128;
            tfac[i] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(frsrc, off, 0, 0));
        }
    stage(0);
    settle_b();
    load_x(1);
    __syncthreads();
    // The two wavefronts of a SIMD stage at different ends of a tile: in step they would both multiply and then both convert.
    auto walk = [&](auto first_) __attribute__((always_inline)) {
        constexpr bool FIRST = decltype(first_)::value;
        for (int t = 0; t < nt - 1; ++t) {
            if constexpr (FIRST) {
                stage((t + 1) & 1);
                load_x(t + 2);
            }
#pragma unroll
            for (int i = 0; i < TI; ++i) fragment(t, wm + i * WM);
            if constexpr (!FIRST) {
                stage((t + 1) & 1);
                load_x(t + 2);
            }
            __syncthreads();
        }
    };
    if (wave < 4) walk(std::false_type{});
    else walk(std::true_type{});
#pragma unroll
    for (int i = 0; i < TI; ++i) fragment(nt - 1, wm + i * WM);
}

// `p` carries everything except what splits the launch.
template <class Cfg, int KIND, bool U8>
sparq_status launch_cols_cfg(const RowsParams& p, hipStream_t s) {
    ColsParams q{p};
    const int64_t cus = device_cu_count();
    const int64_t groups = ((int64_t)p.N + 32 * Cfg::kFN - 1) / (32 * Cfg::kFN), per_pass = 8 / Cfg::kWM;
    const int64_t fragments = ((int64_t)p.M + 31) / 32;
    if (p.steps > Cfg::kKS || (int64_t)p.N * 4 * 32 >= 0x7FFFFFFF || fragments > (1 << 25)) return SPARQ_EUNSUPPORTED;
    q.shares = (int)((groups + per_pass - 1) / per_pass);
    const int64_t most = cus / (8 * q.shares) * 8, wgs = fragments < most ? fragments : most;
    if (wgs == 0) return SPARQ_EUNSUPPORTED;
    q.share_groups = (int)((groups + q.shares - 1) / q.shares);
    q.wgs = (int)wgs;
    q.per_wg = (int)(fragments / wgs);
    q.one_more = (int)(fragments % wgs);
    constexpr int64_t lds_bytes = 2 * Cfg::kBuf + (U8 ? 8 * 32 * Cfg::kPitch + Cfg::kTableBytes : 0);
    static_assert(lds_bytes <= kLdsPerCu);
    auto kern = conv_cols_kernel<Cfg, KIND, U8>;
    if constexpr (lds_bytes > 64 * 1024) {                   // (what a launch may use without asking)
        static std::atomic<bool> lds_set_dev[kMaxDevices];   // (concurrent callers at worst repeat the call, with the same value)
        std::atomic<bool>& lds_set = lds_set_dev[current_device_slot()];
        if (!lds_set.load(std::memory_order_relaxed) || current_device_slot() == kMaxDevices - 1) {
            if (hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, kLdsPerCu) != hipSuccess)
                return SPARQ_ELAUNCH;
            lds_set.store(true, std::memory_order_relaxed);
        }
    }
    kern<<<(unsigned)((wgs + 7) / 8 * 8 * q.shares), kColsThreads, (size_t)lds_bytes, s>>>(q);
    return launch_status();
}

// One: a wavefront for each 32 FN channels; Bytes, Words: what layers of up to four groups take for bytes and for four-byte results, where the rule
// has two wavefronts for the same channels, which One would leave idle (512 -> 128, 200704 pixels, bytes 45 -> 39 us).
template <class One, class Bytes, class Words, int KIND>
sparq_status launch_cols_out(const RowsParams& p, hipStream_t s) {
    const bool narrow = p.N <= 4 * 32 * One::kFN;
    if (!std::is_same_v<One, Bytes> && narrow && p.out_u8) return launch_cols_cfg<Bytes, KIND, true>(p, s);
    if (!std::is_same_v<One, Words> && narrow && !p.out_u8) return launch_cols_cfg<Words, KIND, false>(p, s);
    return p.out_u8 ? launch_cols_cfg<One, KIND, true>(p, s) : launch_cols_cfg<One, KIND, false>(p, s);
}

template <class One, class Bytes = One, class Words = Bytes>
sparq_status launch_cols_kind(TrimKind kind, const RowsParams& p, hipStream_t s) {
    switch (kind) {
        case kTrimNone: return launch_cols_out<One, Bytes, Words, kTrimNone>(p, s);
        case kTrimFloor: return launch_cols_out<One, Bytes, Words, kTrimFloor>(p, s);
        case kTrimFloorPair: return launch_cols_out<One, Bytes, Words, kTrimFloorPair>(p, s);
        case kTrimFloorPairWide: return launch_cols_out<One, Bytes, Words, kTrimFloorPairWide>(p, s);
        case kTrimRound: return launch_cols_out<One, Bytes, Words, kTrimRound>(p, s);
        case kTrimRound4: return launch_cols_out<One, Bytes, Words, kTrimRound4>(p, s);
        case kTrimRoundPairWide: return launch_cols_out<One, Bytes, Words, kTrimRoundPairWide>(p, s);
        case kTrimRoundPair4: return launch_cols_out<One, Bytes, Words, kTrimRoundPair4>(p, s);
        default: return SPARQ_EUNSUPPORTED;
    }
}

SPARQ_DECLARE_ROWS(launch_cols_k256);
SPARQ_DECLARE_ROWS(launch_cols_k384);
SPARQ_DECLARE_ROWS(launch_cols_k512);
SPARQ_DECLARE_ROWS(launch_cols_k768);
SPARQ_DECLARE_ROWS(launch_cols_k1024);

}  // namespace sparq
