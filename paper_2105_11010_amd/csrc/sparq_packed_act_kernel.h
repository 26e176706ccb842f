// Kernels of the packed activation storage (format: sparq_packed_act.hip; arithmetic: sparq_packed_swar.h).
// One lane handles one record of 32 channels: eight words of activations on one side, N data words + ShiftCtrl words +
// MuxCtrl word on the other.  Both directions move about two bytes per activation and do 40-60 vector instructions
// per four activations (pack) or 25-30 (unpack), so that arithmetic and memory traffic take about the same time.
#pragma once
#include "sparq_common.h"
#include "sparq_fastdiv.h"
#include "sparq_packed_swar.h"

namespace sparq {

constexpr int kPkThreads = 256;
typedef unsigned int v4u __attribute__((ext_vector_type(4)));
typedef v4u v4u_any __attribute__((aligned(1)));             // any byte address: the memory pipeline takes unaligned vectors
typedef uint32_t u32_any __attribute__((aligned(1)));
typedef v4u v4u_w __attribute__((aligned(4)));

struct CodecParams {
    uint8_t* bytes;              // [rows][C] activations
    uint32_t* packed;            // records
    int64_t records, total;      // number of records, rows * C
    int C, nrec;                 // channels, records per row
    FastDiv div_nrec;            // valid when records < 2^31
    PackLuts L;
};

// Where record idx's 32 channels start and how many of them exist.
__device__ __forceinline__ void record_place(const CodecParams& p, int64_t idx, int64_t* off, int* valid) {
    if (p.C % kRecChannels == 0) {                           // uniform: rows are whole records
        *off = idx * kRecChannels;
        *valid = kRecChannels;
        return;
    }
    const int64_t r = p.records < (1ll << 31) ? (int64_t)fastdiv((uint32_t)idx, p.div_nrec) : idx / p.nrec;
    const int c0 = (int)(idx - r * p.nrec) * kRecChannels;
    *off = r * p.C + c0;
    *valid = p.C - c0 < kRecChannels ? p.C - c0 : kRecChannels;
}

__device__ __forceinline__ void load_channels(const CodecParams& p, int64_t off, int valid, uint32_t (&w)[8]) {
    const uint8_t* src = p.bytes + off;
    if (off + kRecChannels <= p.total) {                     // 32 bytes exist, of this row or of the next
        const v4u a = *reinterpret_cast<const v4u_any*>(src), b = *reinterpret_cast<const v4u_any*>(src + 16);
        w[0] = a.x; w[1] = a.y; w[2] = a.z; w[3] = a.w; w[4] = b.x; w[5] = b.y; w[6] = b.z; w[7] = b.w;
        if (valid < kRecChannels) {
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const int n = valid - 4 * i;
                w[i] &= n >= 4 ? 0xFFFFFFFFu : n <= 0 ? 0u : (1u << (8 * n)) - 1u;
            }
        }
    } else {
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            uint32_t v = 0;
#pragma unroll
            for (int j = 0; j < 4; ++j)
                if (4 * i + j < valid) v |= (uint32_t)src[4 * i + j] << (8 * j);
            w[i] = v;
        }
    }
}

__device__ __forceinline__ void store_channels(const CodecParams& p, int64_t off, int valid, const uint32_t (&w)[8]) {
    uint8_t* dst = p.bytes + off;
    if (valid == kRecChannels) {
        *reinterpret_cast<v4u_any*>(dst) = v4u{w[0], w[1], w[2], w[3]};
        *reinterpret_cast<v4u_any*>(dst + 16) = v4u{w[4], w[5], w[6], w[7]};
        return;
    }
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        if (4 * i + 4 <= valid) *reinterpret_cast<u32_any*>(dst + 4 * i) = w[i];
        else {
#pragma unroll
            for (int j = 0; j < 3; ++j)
                if (4 * i + j < valid) dst[4 * i + j] = (uint8_t)(w[i] >> (8 * j));
        }
    }
}

template <int WORDS>
__device__ __forceinline__ void store_words(uint32_t* dst, const uint32_t (&r)[WORDS]) {
#pragma unroll
    for (int i = 0; i + 4 <= WORDS; i += 4) *reinterpret_cast<v4u_w*>(dst + i) = v4u{r[i], r[i + 1], r[i + 2], r[i + 3]};
#pragma unroll
    for (int i = WORDS / 4 * 4; i < WORDS; ++i) dst[i] = r[i];
}
template <int WORDS>
__device__ __forceinline__ void load_words(const uint32_t* src, uint32_t (&r)[WORDS]) {
#pragma unroll
    for (int i = 0; i + 4 <= WORDS; i += 4) {
        const v4u v = *reinterpret_cast<const v4u_w*>(src + i);
        r[i] = v.x; r[i + 1] = v.y; r[i + 2] = v.z; r[i + 3] = v.w;
    }
#pragma unroll
    for (int i = WORDS / 4 * 4; i < WORDS; ++i) r[i] = src[i];
}

// A wavefront's 64 records are WORDS * 256 contiguous bytes, and so are their 2 KB of channels when rows are whole
// records, but a lane's own share is 16 to 36 bytes: read or written straight from the lanes, an instruction touches a
// part of each line.  These two turn the shares through the wavefront's own piece of LDS, so that lane l moves 16-byte
// chunks l, l + 64, ... with non-temporal accesses.
template <int WORDS>
__device__ __forceinline__ void turn_load(const uint32_t* src, int nwords, uint32_t* area, int lane, uint32_t (&r)[WORDS]) {
#pragma unroll
    for (int k = 0; k < (WORDS + 3) / 4; ++k) {
        const int c = lane + 64 * k;
        if (4 * c + 4 <= nwords) *reinterpret_cast<v4u*>(area + 4 * c) = __builtin_nontemporal_load(reinterpret_cast<const v4u_w*>(src + 4 * c));
        else for (int i = 4 * c; i < nwords; ++i) area[i] = src[i];
    }
    wavefront_lds_fence();
#pragma unroll
    for (int i = 0; i < WORDS; ++i) r[i] = area[lane * WORDS + i];
    wavefront_lds_fence();
}
template <int WORDS>
__device__ __forceinline__ void turn_store(uint32_t* dst, int nwords, uint32_t* area, int lane, const uint32_t (&r)[WORDS]) {
#pragma unroll
    for (int i = 0; i < WORDS; ++i) area[lane * WORDS + i] = r[i];
    wavefront_lds_fence();
#pragma unroll
    for (int k = 0; k < (WORDS + 3) / 4; ++k) {
        const int c = lane + 64 * k;
        if (4 * c + 4 <= nwords) __builtin_nontemporal_store(*reinterpret_cast<const v4u*>(area + 4 * c), reinterpret_cast<v4u_w*>(dst + 4 * c));
        else for (int i = 4 * c; i < nwords; ++i) dst[i] = area[i];
    }
    wavefront_lds_fence();
}

// N window bits, SB ShiftCtrl bits, G channels per ShiftCtrl field.
// Bound by its arithmetic with vSPARQ (45 vector instructions per four activations: 134 us on [65536][4608], 4.5 TB/s read
// + written), by memory without (100 us, 5.2 TB/s): records go straight from the lanes (through LDS: 142 and 99 us).
template <int N, int SB, int G, bool PAIR, bool ROUND>
__global__ __launch_bounds__(kPkThreads) void pack_act_kernel(const CodecParams p) {
    constexpr int WORDS = codec_words(N, SB, G, PAIR);
    const int64_t stride = (int64_t)gridDim.x * kPkThreads;
    for (int64_t idx = (int64_t)blockIdx.x * kPkThreads + threadIdx.x; idx < p.records; idx += stride) {
        int64_t off;
        int valid;
        record_place(p, idx, &off, &valid);
        uint32_t w[8], rec[WORDS];
        load_channels(p, off, valid, w);
        pack_record<N, SB, G, PAIR, ROUND>(w, p.L, rec);
        store_words(p.packed + idx * WORDS, rec);
    }
}

// Bound by memory.  TURN: calls on whole records that move more than the last-level cache holds go through LDS (112
// instead of 119 us on [65536][4608] with 32-byte records, 5.4 TB/s; 95 instead of 108 us with 24-byte ones); smaller
// calls are faster straight from the lanes (13.4 against 14.8 us on [65536][512]).
template <int N, int SB, int G, bool PAIR, bool TURN>
__global__ __launch_bounds__(kPkThreads) void unpack_act_kernel(const CodecParams p) {
    constexpr int WORDS = codec_words(N, SB, G, PAIR);
    if constexpr (TURN) {
        __shared__ __attribute__((aligned(16))) uint32_t lds[kPkThreads / 64][64 * (WORDS > 8 ? WORDS : 8)];
        const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
        for (int64_t base = ((int64_t)blockIdx.x * (kPkThreads / 64) + wave) * 64; base < p.records; base += (int64_t)gridDim.x * kPkThreads) {
            const int live = p.records - base < 64 ? (int)(p.records - base) : 64;
            uint32_t rec[WORDS], w[8];
            turn_load(p.packed + base * WORDS, live * WORDS, lds[wave], lane, rec);
            unpack_record<N, SB, G, PAIR>(rec, p.L, w);
            turn_store(reinterpret_cast<uint32_t*>(p.bytes) + base * 8, live * 8, lds[wave], lane, w);
        }
    } else {
        const int64_t stride = (int64_t)gridDim.x * kPkThreads;
        for (int64_t idx = (int64_t)blockIdx.x * kPkThreads + threadIdx.x; idx < p.records; idx += stride) {
            int64_t off;
            int valid;
            record_place(p, idx, &off, &valid);
            uint32_t rec[WORDS], w[8];
            load_words(p.packed + idx * WORDS, rec);
            unpack_record<N, SB, G, PAIR>(rec, p.L, w);
            store_channels(p, off, valid, w);
        }
    }
}

typedef void (*CodecKernel)(const CodecParams);

// The kernels of one window width; null: no such format.  variant: rounding (pack), through LDS (unpack).
template <int N, int SB, bool PACK>
CodecKernel codec_kernel_sb(int group, bool pair, bool variant) {
    if constexpr (PACK) {
#define SPARQ_PACK_G(GG) if (group == GG) return variant ? pack_act_kernel<N, SB, GG, false, true> : pack_act_kernel<N, SB, GG, false, false>;
        if (pair) return group != 1 ? nullptr : variant ? pack_act_kernel<N, SB, 1, true, true> : pack_act_kernel<N, SB, 1, true, false>;
        SPARQ_PACK_G(1) SPARQ_PACK_G(2) SPARQ_PACK_G(4) SPARQ_PACK_G(8) SPARQ_PACK_G(16) SPARQ_PACK_G(32)
#undef SPARQ_PACK_G
    } else {
        if (pair) return group != 1 ? nullptr : variant ? unpack_act_kernel<N, SB, 1, true, true> : unpack_act_kernel<N, SB, 1, true, false>;
#define SPARQ_UNPACK_G(GG) if (group == GG) return variant ? unpack_act_kernel<N, SB, GG, false, true> : unpack_act_kernel<N, SB, GG, false, false>;
        SPARQ_UNPACK_G(1) SPARQ_UNPACK_G(2) SPARQ_UNPACK_G(4) SPARQ_UNPACK_G(8) SPARQ_UNPACK_G(16) SPARQ_UNPACK_G(32)
#undef SPARQ_UNPACK_G
    }
    return nullptr;
}
template <int N, bool PACK>
CodecKernel codec_kernel_n(int sb, int group, bool pair, bool variant) {
    switch (sb) {
        case 1: return codec_kernel_sb<N, 1, PACK>(group, pair, variant);
        case 2: return codec_kernel_sb<N, 2, PACK>(group, pair, variant);
        case 3: return codec_kernel_sb<N, 3, PACK>(group, pair, variant);
        default: return nullptr;
    }
}

// One translation unit per window width.
CodecKernel codec_kernel_4bit(bool pack, int sb, int group, bool pair, bool variant);
CodecKernel codec_kernel_3bit(bool pack, int sb, int group, bool pair, bool variant);
CodecKernel codec_kernel_2bit(bool pack, int sb, int group, bool pair, bool variant);

}  // namespace sparq
