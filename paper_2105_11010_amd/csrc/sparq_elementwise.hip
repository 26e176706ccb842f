// Streaming kernels of libsparq: the standalone trim (Sections 3.1-3.2), the
// per-output-channel dequantisation (Section 5), the one-time weight packing
// and the trimmed, channel-padded copy used for channel counts that are not a
// multiple of four and where trimming while staging would take longer.  Nearly all are
// bound by memory: each lane moves 128-bit words, and the grid is sized by how much
// there is to do per word (ew_grid, stream_grid).
#include <type_traits>

#include "sparq_common.h"
#include "sparq_fastdiv.h"

namespace sparq {

constexpr int kEwThreads = 256;
typedef unsigned int v4u __attribute__((ext_vector_type(4)));
typedef v4u v4u_any __attribute__((aligned(1)));             // any byte address
typedef int v4s __attribute__((ext_vector_type(4)));
typedef float v4f __attribute__((ext_vector_type(4)));

static int ew_grid(int64_t work_items, int per_block) {
    int64_t blocks = (work_items + per_block - 1) / per_block;
    const int64_t cap = 256 * 16;            // 256 compute units, 16 workgroups each
    if (blocks > cap) blocks = cap;
    if (blocks < 1) blocks = 1;
    return (int)blocks;
}

// Kernels that only stream: one word per lane and as many workgroups as that takes, so that the accesses of the moment lie close
// together (65536 x 4608 trimmed, 604 MB moved, 105 us with 4096 workgroups striding through the tensor, 122 with four words ahead per
// lane, 96 this way).  What has much to do per word or to set up per lane is better off with fewer workgroups (ew_grid), and so are
// trims within the last-level cache (75000 x 320 7.4 against 8.0 us, two-bit windows 100000 x 320 11.6 against 12.2).
// (2^19 workgroups move 2 GiB; larger tensors go round again.)
constexpr int kMaxStreamGrid = 1 << 19;
static int stream_grid(int64_t words) {
    const int64_t blocks = (words + kEwThreads - 1) / kEwThreads;
    return (int)(blocks < 1 ? 1 : blocks > kMaxStreamGrid ? kMaxStreamGrid : blocks);
}

// ---- standalone trim ---------------------------------------------------------
// Even C: pairs (2j, 2j+1) of a row are also pairs of the flattened array, so
// the tensor is processed as one stream of 16-byte words.
// NT: non-temporal loads and stores, for tensors larger than the last-level cache that are streamed once (+8 % there;
// cache-resident or in-place tensors are faster with ordinary accesses).
// tail: bytes past the last whole word, done pair by pair by the first lanes (a launch of their own made small calls 5.0 -> 9.0 us).
template <int KIND, bool NT>
__global__ __launch_bounds__(kEwThreads) void trim_vec_kernel(const uint4* x, uint4* y,
                                                              int64_t n_vec, int tail, TrimLuts L) {
    const int t = 2 * (int)threadIdx.x;
    if (blockIdx.x == 0 && t < tail) {
        const uint8_t* src = reinterpret_cast<const uint8_t*>(x + n_vec) + t;
        uint8_t* dst = reinterpret_cast<uint8_t*>(y + n_vec) + t;
        const bool has_b = t + 1 < tail;
        const uint32_t v = trim4_kind<KIND>(src[0] | (has_b ? (uint32_t)src[1] << 8 : 0u), L);
        dst[0] = (uint8_t)v;
        if (has_b) dst[1] = (uint8_t)(v >> 8);
    }
    const int64_t stride = (int64_t)gridDim.x * kEwThreads;
    for (int64_t i = (int64_t)blockIdx.x * kEwThreads + threadIdx.x; i < n_vec; i += stride) {
        const v4u* src = reinterpret_cast<const v4u*>(x) + i;
        v4u v = NT ? __builtin_nontemporal_load(src) : *src;
        v.x = trim4_kind<KIND>(v.x, L);
        v.y = trim4_kind<KIND>(v.y, L);
        v.z = trim4_kind<KIND>(v.z, L);
        v.w = trim4_kind<KIND>(v.w, L);
        if (NT) __builtin_nontemporal_store(v, reinterpret_cast<v4u*>(y) + i);
        else reinterpret_cast<v4u*>(y)[i] = v;
    }
}

// Any C, any alignment: one lane per pair of channels of one row.
template <int KIND>
__global__ __launch_bounds__(kEwThreads) void trim_pair_kernel(const uint8_t* x, uint8_t* y, int64_t rows, int C, TrimLuts L) {
    const int pairs = (C + 1) / 2;
    const int64_t total = rows * pairs;
    const int64_t stride = (int64_t)gridDim.x * kEwThreads;
    for (int64_t i = (int64_t)blockIdx.x * kEwThreads + threadIdx.x; i < total; i += stride) {
        const int64_t r = i / pairs;
        const int c = (int)(i - r * pairs) * 2;
        const int64_t off = r * C + c;
        const bool has_b = c + 1 < C;
        const uint32_t a = x[off];
        const uint32_t b = has_b ? x[off + 1] : 0u;
        const uint32_t t = trim4_kind<KIND>(a | (b << 8), L);
        y[off] = (uint8_t)t;
        if (has_b) y[off + 1] = (uint8_t)(t >> 8);
    }
}

// Odd C >= 16 with pairing, 16-byte aligned, x and y apart: still one stream of aligned 16-byte words, one per lane; a
// word learns from its neighbours (lanes, at a wavefront's ends memory) whether the bytes next to it are zero.  Bound by
// memory and its arithmetic about equally (35 vector instructions per four activations).  156800 x 289: 49.8 -> 20.4 us
// (4.4 TB/s; one lane per pair, byte accesses and a 64-bit division before).
// col_step: channel by which a wavefront's position in its row moves per round.
template <int KIND, bool NT>
__global__ __launch_bounds__(kEwThreads) void trim_odd_rows_kernel(const uint8_t* __restrict__ x, uint8_t* __restrict__ y,
                                                                   int64_t bytes, uint32_t C, FastDiv divC, uint32_t col_step,
                                                                   TrimLuts L) {
    const int lane = threadIdx.x & 63;
    const int64_t stride = (int64_t)gridDim.x * kEwThreads;
    int64_t w0 = (int64_t)blockIdx.x * kEwThreads + (threadIdx.x & ~63);         // the wavefront's first word
    uint32_t wave_col = (uint32_t)w0 * 16;                   // (the first round's words: below 2^25)
    wave_col -= fastdiv(wave_col, divC) * C;
    for (; w0 * 16 < bytes; w0 += stride) {
        const int64_t at = (w0 + lane) * 16;
        const int valid = bytes - at >= 16 ? 16 : bytes > at ? (int)(bytes - at) : 0;
        uint32_t w[4] = {0, 0, 0, 0}, nz[4], pm[4];
        if (valid == 16) {
            const v4u* src = reinterpret_cast<const v4u*>(x + at);
            const v4u v = NT ? __builtin_nontemporal_load(src) : *src;
#pragma unroll
            for (int k = 0; k < 4; ++k) w[k] = v[k];
        } else {
#pragma unroll
            for (int k = 0; k < 16; ++k)
                if (k < valid) w[k >> 2] |= (uint32_t)x[at + k] << (8 * (k & 3));
        }
        const int64_t edge_at = lane == 0 ? at - 1 : at + 16;
        uint32_t edge = 0;
        if ((lane == 0 || lane == 63) && edge_at >= 0 && edge_at < bytes) edge = x[edge_at] ? 0xFFFFFFFFu : 0u;
#pragma unroll
        for (int k = 0; k < 4; ++k) nz[k] = expand_bit7(nonzero_flag(w[k]));
        uint32_t before = __shfl_up(nz[3], 1, 64), after = __shfl_down(nz[0], 1, 64);
        before = lane == 0 ? edge : before;
        after = lane == 63 ? edge : after;
        const uint32_t off = wave_col + 16u * (uint32_t)lane;
        odd_row_partners(off - fastdiv(off, divC) * C, C, nz, before, after, pm);
#pragma unroll
        for (int k = 0; k < 4; ++k) w[k] = trim4_kind_beside<KIND>(w[k], pm[k], L);
        if (valid == 16) {
            const v4u v = {w[0], w[1], w[2], w[3]};
            if (NT) __builtin_nontemporal_store(v, reinterpret_cast<v4u*>(y + at));
            else *reinterpret_cast<v4u*>(y + at) = v;
        } else {
#pragma unroll
            for (int k = 0; k < 16; ++k)
                if (k < valid) y[at + k] = (uint8_t)(w[k >> 2] >> (8 * (k & 3)));
        }
        wave_col += col_step;
        wave_col -= wave_col >= C ? C : 0u;
    }
}

template <int KIND>
static void launch_trim_kind(const uint8_t* x, uint8_t* y, int64_t rows, int C, const TrimLuts& L, hipStream_t s) {
    const int64_t bytes = rows * C;
    const bool aligned16 = aligned(x, 16) && aligned(y, 16);
    // one flat stream: pairs do not depend on where rows begin (even C), or there are none
    if (aligned16 && bytes >= 16 && (C % 2 == 0 || !trim_kind_pairs(KIND))) {
        const int64_t n_vec = bytes / 16;
        if (x != y && 2 * bytes >= kStreamedBytes)
            trim_vec_kernel<KIND, true><<<stream_grid(n_vec), kEwThreads, 0, s>>>(
                reinterpret_cast<const uint4*>(x), reinterpret_cast<uint4*>(y), n_vec, (int)(bytes % 16), L);
        else
            trim_vec_kernel<KIND, false><<<ew_grid(n_vec, kEwThreads * 4), kEwThreads, 0, s>>>(
                reinterpret_cast<const uint4*>(x), reinterpret_cast<uint4*>(y), n_vec, (int)(bytes % 16), L);
        return;
    }
    if constexpr (trim_kind_pairs(KIND)) {
        if (aligned16 && x != y && C >= 16 && C < (1 << 30)) {
            const int64_t words = (bytes + 15) / 16;
            const int grid = ew_grid(words, kEwThreads);
            const auto kernel = 2 * bytes >= kStreamedBytes ? trim_odd_rows_kernel<KIND, true> : trim_odd_rows_kernel<KIND, false>;
            kernel<<<grid, kEwThreads, 0, s>>>(x, y, bytes, (uint32_t)C, make_fastdiv((uint32_t)C),
                                               (uint32_t)((int64_t)grid * kEwThreads * 16 % C), L);
            return;
        }
    }
    trim_pair_kernel<KIND><<<ew_grid(rows * ((C + 1) / 2), kEwThreads), kEwThreads, 0, s>>>(x, y, rows, C, L);
}

// ---- trimmed copy with channels padded to a multiple of 16 -------------------
template <int KIND>
__global__ __launch_bounds__(kEwThreads) void trim_pad_kernel(const uint8_t* __restrict__ x, uint32_t* __restrict__ xp,
                                                              int64_t pixels, int C, int Cp, TrimLuts L) {
    const int words = Cp / 4;
    const int64_t total = pixels * words;
    const int64_t stride = (int64_t)gridDim.x * kEwThreads;
    for (int64_t i = (int64_t)blockIdx.x * kEwThreads + threadIdx.x; i < total; i += stride) {
        const int64_t pix = i / words;
        const int c = (int)(i - pix * words) * 4;
        const uint8_t* src = x + pix * C + c;
        uint32_t v = 0;
#pragma unroll
        for (int j = 0; j < 4; ++j)
            if (c + j < C) v |= (uint32_t)src[j] << (8 * j);   // channels past C act as zeros (implicit zero partner)
        xp[i] = trim4_kind<KIND>(v, L);
    }
}

// The same with 16 channels per lane (C > 16): the row's last chunk is read as the 16 bytes that end with the row and
// shifted down, so every read stays inside the row, is one (unaligned) vector and brings zeros in past C.
// 156800 x 65 -> 80: 13.8 -> 6.8 us (four byte reads per word and a 64-bit division before).
template <int KIND>
__global__ __launch_bounds__(kEwThreads) void trim_pad16_kernel(const uint8_t* __restrict__ x, v4u* __restrict__ xp, uint32_t total,
                                                                int C, int chunks, FastDiv div_chunks, TrimLuts L) {
    const uint32_t stride = gridDim.x * kEwThreads;
    for (uint32_t i = blockIdx.x * kEwThreads + threadIdx.x; i < total; i += stride) {
        const uint32_t pix = fastdiv(i, div_chunks);
        const int c = (int)(i - pix * (uint32_t)chunks) * 16;
        const int from = c + 16 <= C ? c : C - 16, sh = c - from;
        const v4u v = *reinterpret_cast<const v4u_any*>(x + (int64_t)pix * C + from);
        uint64_t lo = ((uint64_t)v[1] << 32) | v[0], hi = ((uint64_t)v[3] << 32) | v[2];
        if (sh) {                                            // 1..15 bytes
            const int bits = 8 * (sh & 7);
            if (sh >= 8) { lo = hi; hi = 0; }
            if (bits) { lo = (lo >> bits) | (hi << (64 - bits)); hi >>= bits; }
        }
        v4u o = {(uint32_t)lo, (uint32_t)(lo >> 32), (uint32_t)hi, (uint32_t)(hi >> 32)};
#pragma unroll
        for (int k = 0; k < 4; ++k) o[k] = trim4_kind<KIND>(o[k], L);
        xp[i] = o;
    }
}

// Three channels to four (a network's first layer): a lane turns four pixels, three words, into four words.
// 12.8 M pixels: 40.8 -> 16.3 us (5.5 TB/s).
template <int KIND>
__global__ __launch_bounds__(kEwThreads) void trim_pad_3to4_kernel(const uint32_t* __restrict__ x, v4u* __restrict__ xp, uint32_t quads,
                                                                   TrimLuts L) {
    const uint32_t stride = gridDim.x * kEwThreads;
    for (uint32_t i = blockIdx.x * kEwThreads + threadIdx.x; i < quads; i += stride) {
        const uint32_t* src = x + 3 * (size_t)i;
        const uint32_t a = src[0], b = src[1], c = src[2];
        v4u o = {a & 0xFFFFFFu, perm(b, a, 0x0C050403u), perm(c, b, 0x0C040302u), c >> 8};
#pragma unroll
        for (int k = 0; k < 4; ++k) o[k] = trim4_kind<KIND>(o[k], L);
        xp[i] = o;
    }
}

template <int KIND>
static void launch_trim_pad_kind(const uint8_t* x, uint8_t* xp, int64_t pixels, int C, int Cp, const TrimLuts& L,
                                 hipStream_t s) {
    if (C == 3 && Cp == 4 && pixels % 4 == 0 && pixels < (1ll << 31) && aligned(x, 4) && aligned(xp, 16)) {
        const uint32_t quads = (uint32_t)(pixels / 4);
        trim_pad_3to4_kernel<KIND><<<ew_grid(quads, kEwThreads * 2), kEwThreads, 0, s>>>(
            reinterpret_cast<const uint32_t*>(x), reinterpret_cast<v4u*>(xp), quads, L);
        return;
    }
    // (the grid's stride is at most 2^20, so the index stays below 2^32)
    if (C > 16 && Cp % 16 == 0 && pixels * (Cp / 16) < (1ll << 31) && aligned(xp, 16)) {
        const uint32_t total = (uint32_t)(pixels * (Cp / 16));
        trim_pad16_kernel<KIND><<<ew_grid(total, kEwThreads * 2), kEwThreads, 0, s>>>(
            x, reinterpret_cast<v4u*>(xp), total, C, Cp / 16, make_fastdiv((uint32_t)(Cp / 16)), L);
        return;
    }
    const int64_t total = pixels * (Cp / 4);
    trim_pad_kernel<KIND><<<ew_grid(total, kEwThreads * 2), kEwThreads, 0, s>>>(x, reinterpret_cast<uint32_t*>(xp),
                                                                               pixels, C, Cp, L);
}

#define SPARQ_DISPATCH_KIND(kind, FN, ...)                                                  \
    switch (kind) {                                                                         \
        case kTrimNone: FN<kTrimNone>(__VA_ARGS__); break;                                  \
        case kTrimFloor: FN<kTrimFloor>(__VA_ARGS__); break;                                \
        case kTrimFloorPair: FN<kTrimFloorPair>(__VA_ARGS__); break;                        \
        case kTrimFloorPairWide: FN<kTrimFloorPairWide>(__VA_ARGS__); break;                \
        case kTrimRound: FN<kTrimRound>(__VA_ARGS__); break;                                \
        case kTrimRound4: FN<kTrimRound4>(__VA_ARGS__); break;                              \
        case kTrimRoundPair4: FN<kTrimRoundPair4>(__VA_ARGS__); break;                      \
        default: FN<kTrimRoundPairWide>(__VA_ARGS__); break;                                \
    }

sparq_status launch_trim_pad(const uint8_t* x, uint8_t* xp, int64_t pixels, int C, int Cp, const sparq_mode* mode,
                             hipStream_t stream) {
    const TrimLuts L = make_luts(mode->window_bits, mode->shift_mask);
    SPARQ_DISPATCH_KIND(trim_kind(mode), launch_trim_pad_kind, x, xp, pixels, C, Cp, L, stream);
    return launch_status();
}

// ---- dequantisation, and requantisation to the next layer's unsigned 8-bit activations ----
// out = (float)acc * scale[n];  y = clamp(round_to_nearest_even(acc * factor[n]), 0, 255), the product and the rounding in fp32
// (requant_u8 and the packing conversion instruction, which rounds and saturates the same way).
// The accumulators are one stream of words of four, whatever N is.  N a multiple of four: a word's factors are one aligned word.
// Bound by memory; the streamed form's workgroups do one word per lane (200704 x 512 dequantised 150 -> 130 us), smaller calls stride.
template <bool U8, bool NT>
__device__ __forceinline__ void per_channel_word(v4s a, v4f f, void* out, int64_t i) {
    if constexpr (U8) {
        uint32_t w = 0;
#pragma unroll
        for (int k = 0; k < 4; ++k) w = __builtin_amdgcn_cvt_pk_u8_f32(__fmul_rn((float)a[k], f[k]), k, w);
        static_cast<uint32_t*>(out)[i] = w;
    } else {
        v4f o;
#pragma unroll
        for (int k = 0; k < 4; ++k) o[k] = __fmul_rn((float)a[k], f[k]);
        if (NT) __builtin_nontemporal_store(o, static_cast<v4f*>(out) + i);
        else static_cast<v4f*>(out)[i] = o;
    }
}
template <bool U8, bool NT>
__global__ __launch_bounds__(kEwThreads) void per_channel_vec_kernel(const v4s* __restrict__ acc, const float* __restrict__ factor,
                                                                     void* __restrict__ out, int64_t n_vec, uint32_t N, FastDiv divN) {
    const int64_t stride = (int64_t)gridDim.x * kEwThreads;
    for (int64_t i = (int64_t)blockIdx.x * kEwThreads + threadIdx.x; i < n_vec; i += stride) {
        const v4s a = NT ? __builtin_nontemporal_load(acc + i) : acc[i];
        uint32_t col = (uint32_t)i * 4;
        if (n_vec <= (1 << 29)) col -= fastdiv(col, divN) * N;               // uniform
        else col = (uint32_t)(i * 4 % N);
        per_channel_word<U8, NT>(a, *reinterpret_cast<const v4f*>(factor + col), out, i);
    }
}
// Any N the table holds: the factors come from LDS, where the first three are repeated after the last, so that a word that ends a
// row and begins the next reads four in a row as well.  A workgroup does UNROLL neighbouring groups of words: two, or with more than 1024
// channels eight, for its table's sake.  Before (results one at a time, a 64-bit division each) -> now, us: 36992 x 161 dequantised
// 10.1 -> 9.2, requantised 9.0 -> 7.2; 200000 x 161 60 -> 46, 47 -> 30; 200704 x 511 189 -> 132, 146 -> 89.
constexpr int kMaxTable = 2 * 1024;
template <bool U8, bool NT, int UNROLL>
__global__ __launch_bounds__(kEwThreads) void per_channel_table_kernel(const v4s* __restrict__ acc, const float* __restrict__ factor,
                                                                       void* __restrict__ out, int64_t n_vec, int tail, uint32_t N,
                                                                       FastDiv divN) {
    extern __shared__ float table[];
    int64_t i = (int64_t)blockIdx.x * UNROLL * kEwThreads + threadIdx.x;
    v4s a[UNROLL];
    auto request = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < UNROLL; ++u)
            if (i + u * kEwThreads < n_vec) a[u] = NT ? __builtin_nontemporal_load(acc + i + u * kEwThreads) : acc[i + u * kEwThreads];
    };
    request();
    for (uint32_t n = threadIdx.x; n < N + 3; n += kEwThreads) table[n] = factor[n < N ? n : (n - N) % N];
    __syncthreads();
    for (;;) {
#pragma unroll
        for (int u = 0; u < UNROLL; ++u) {
            const int64_t at = i + u * kEwThreads;
            if (at >= n_vec) break;
            uint32_t col = (uint32_t)at * 4;
            if (n_vec <= (1 << 29)) col -= fastdiv(col, divN) * N;           // uniform
            else col = (uint32_t)(at * 4 % N);
            v4f f;
#pragma unroll
            for (int k = 0; k < 4; ++k) f[k] = table[col + k];
            per_channel_word<U8, NT>(a[u], f, out, at);
        }
        i += (int64_t)gridDim.x * UNROLL * kEwThreads;
        if (i >= n_vec) break;
        request();
    }
    if (blockIdx.x == 0 && (int)threadIdx.x < tail) {        // results past the last whole word
        const int64_t at = n_vec * 4 + threadIdx.x;
        const float f = factor[at % N];
        const int32_t v = reinterpret_cast<const int32_t*>(acc)[at];
        if constexpr (U8) static_cast<uint8_t*>(out)[at] = (uint8_t)requant_u8(v, f);
        else static_cast<float*>(out)[at] = __fmul_rn((float)v, f);
    }
}

// Pointers off their words' alignment, or calls the table is not for.
template <bool U8>
__global__ __launch_bounds__(kEwThreads) void per_channel_scalar_kernel(const int32_t* __restrict__ acc, const float* __restrict__ factor,
                                                                        void* __restrict__ out, int64_t total, int N) {
    const int64_t stride = (int64_t)gridDim.x * kEwThreads;
    for (int64_t i = (int64_t)blockIdx.x * kEwThreads + threadIdx.x; i < total; i += stride) {
        if constexpr (U8) static_cast<uint8_t*>(out)[i] = (uint8_t)requant_u8(acc[i], factor[i % N]);
        else static_cast<float*>(out)[i] = __fmul_rn((float)acc[i], factor[i % N]);
    }
}

template <bool U8>
static sparq_status launch_per_channel(const int32_t* acc, const float* factor, void* out, int64_t total, int N, hipStream_t s) {
    const bool words = aligned(acc, 16) && aligned(out, U8 ? 4 : 16), nt = !U8 && 8 * total >= kStreamedBytes;
    const int64_t n_vec = total / 4;
    const v4s* acc4 = reinterpret_cast<const v4s*>(acc);
    if (words && N % 4 == 0 && aligned(factor, 16)) {
        const FastDiv div = make_fastdiv((uint32_t)N);
        if (nt) per_channel_vec_kernel<U8, true><<<stream_grid(n_vec), kEwThreads, 0, s>>>(acc4, factor, out, n_vec, (uint32_t)N, div);
        else per_channel_vec_kernel<U8, false><<<ew_grid(n_vec, kEwThreads * 4), kEwThreads, 0, s>>>(acc4, factor, out, n_vec, (uint32_t)N, div);
        return launch_status();
    }
    // A workgroup fills its table before its first result, so calls with fewer rows than three quarters of their channels, or of less than
    // two workgroups' words, are ahead without (us, without -> with, replayed as a graph, requantised: 1 x 255 1.90 -> 2.19, 31 x 511 2.31 ->
    // 2.49, 62 x 1023 2.46 -> 2.71, 391 x 1023 2.59 -> 2.75; even at 250 x 511, 782 x 767, 899 x 1001; 1955 x 1023 3.74 -> 3.30), and those
    // of more than 1024 factors are for large calls (200 x 2001 3.5 us without, 5.4 with it, 20000 x 2001 76 and 60).
    const bool table = N <= 1024 ? total >= 2048 && 4 * (total / N) >= 3ll * N : N <= kMaxTable && total >= (4 << 20);
    if (words && table) {
        const int tail = (int)(total % 4);
        const FastDiv div = make_fastdiv((uint32_t)N);
        const size_t lds = (size_t)(N + 3) * sizeof(float);
        const auto launch = [&](auto nt_, auto unroll_) {
            constexpr int U = decltype(unroll_)::value;
            per_channel_table_kernel<U8, decltype(nt_)::value, U><<<stream_grid((n_vec + U - 1) / U), kEwThreads, lds, s>>>(
                acc4, factor, out, n_vec, tail, (uint32_t)N, div);
        };
        if (N <= 1024) nt ? launch(std::true_type{}, std::integral_constant<int, 2>{}) : launch(std::false_type{}, std::integral_constant<int, 2>{});
        else nt ? launch(std::true_type{}, std::integral_constant<int, 8>{}) : launch(std::false_type{}, std::integral_constant<int, 8>{});
        return launch_status();
    }
    per_channel_scalar_kernel<U8><<<ew_grid(total, kEwThreads * 4), kEwThreads, 0, s>>>(acc, factor, out, total, N);
    return launch_status();
}

// ---- weight packing ----------------------------------------------------------
// packed[w_off + ((kb*4 + kc)*Np + n)*16 + j] = w[n][tap][c + j]  with  k = kb*64 + kc*16 = tap*Cp + c
__global__ __launch_bounds__(kEwThreads) void pack_weights_kernel(const int8_t* __restrict__ w, uint4* __restrict__ dst,
                                                                  int N, int Np, int C, int Cq, int taps, int Kp) {
    const int64_t total = (int64_t)(Kp / kChunk) * Np;
    const int64_t stride = (int64_t)gridDim.x * kEwThreads;
    for (int64_t i = (int64_t)blockIdx.x * kEwThreads + threadIdx.x; i < total; i += stride) {
        const int n = (int)(i % Np);
        const int k = (int)(i / Np) * kChunk;
        const int tap = k / Cq;
        const int c = k - tap * Cq;
        uint32_t v[4] = {0, 0, 0, 0};
        if (n < N && tap < taps) {
            const int8_t* src = w + ((int64_t)n * taps + tap) * C + c;
#pragma unroll
            for (int j = 0; j < kChunk; ++j)
                if (c + j < C) v[j >> 2] |= (uint32_t)(uint8_t)src[j] << (8 * (j & 3));
        }
        dst[i] = make_uint4(v[0], v[1], v[2], v[3]);
    }
}

// Weights of a pixel-folded layer (ConvGeom::fold): output channel n' = p * N + n of the folded
// problem holds, at tap (kh, kwf) and folded channel 4 * q + c, the weight w[n][kh][kw][c] of the
// original tap kw that super-pixel slot q lines up with for output class p (zero where there is none).
__global__ __launch_bounds__(kEwThreads) void pack_weights_fold_kernel(const int8_t* __restrict__ w, uint4* __restrict__ dst,
                                                                       int N, int Np, int C, int KH, int KW, int Kp,
                                                                       int P, int KWf, int kw_min, int sw, int pw) {
    const int64_t total = (int64_t)(Kp / kChunk) * Np;
    const int64_t stride = (int64_t)gridDim.x * kEwThreads;
    for (int64_t i = (int64_t)blockIdx.x * kEwThreads + threadIdx.x; i < total; i += stride) {
        const int nf = (int)(i % Np);
        const int tap = (int)(i / Np);              // one 16-byte chunk = one folded tap (kh, kwf)
        const int kh = tap / KWf, kwf = tap - kh * KWf;
        uint32_t v[4] = {0, 0, 0, 0};
        if (nf < P * N && kh < KH) {
            const int p = nf / N, n = nf - p * N;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int kw = 4 * (kwf + kw_min) + q - (sw * p - pw);
                if (kw < 0 || kw >= KW) continue;
                const int8_t* src = w + (((int64_t)n * KH + kh) * KW + kw) * C;
                for (int c = 0; c < C; ++c) v[q] |= (uint32_t)(uint8_t)src[c] << (8 * c);
            }
        }
        dst[i] = make_uint4(v[0], v[1], v[2], v[3]);
    }
}

// colsum[n] = sum_k w[n % N][k]; one wavefront per (possibly replicated) output channel
__global__ __launch_bounds__(64) void weight_colsum_kernel(const int8_t* __restrict__ w, int32_t* __restrict__ colsum, int N,
                                                           int Nrep, int K) {
    const int n = (int)blockIdx.x < Nrep ? (int)blockIdx.x % N : N;
    int32_t s = 0;
    if (n < N)
        for (int k = threadIdx.x; k < K; k += 64) s += w[(int64_t)n * K + k];
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) s += __shfl_down(s, off, 64);
    if (threadIdx.x == 0) colsum[blockIdx.x] = s;
}

}  // namespace sparq

using namespace sparq;

extern "C" sparq_status sparq_trim(const uint8_t* x, uint8_t* y, int64_t rows, int32_t C, const sparq_mode* mode,
                                   void* stream) {
    if (rows < 0 || C <= 0 || !mode_valid(mode)) return SPARQ_EINVAL;
    if (rows == 0) return SPARQ_OK;          // empty input: nothing to read or write
    if (!x || !y) return SPARQ_EINVAL;
    if (rows > (INT64_MAX / 4) / C) return SPARQ_EINVAL;
    const int64_t bytes = rows * C;
    if (x != y) {
        const uintptr_t xa = (uintptr_t)x, ya = (uintptr_t)y;
        if (xa < ya + (uint64_t)bytes && ya < xa + (uint64_t)bytes) return SPARQ_EINVAL;   // partial overlap
    }
    hipStream_t s = static_cast<hipStream_t>(stream);
    const TrimKind kind = trim_kind(mode);
    if (kind == kTrimNone) {
        if (x != y && hipMemcpyAsync(y, x, (size_t)bytes, hipMemcpyDeviceToDevice, s) != hipSuccess) return SPARQ_ELAUNCH;
        return SPARQ_OK;
    }
    const TrimLuts L = make_luts(mode->window_bits, mode->shift_mask);
    SPARQ_DISPATCH_KIND(kind, launch_trim_kind, x, y, rows, C, L, s);
    return launch_status();
}

extern "C" sparq_status sparq_dequant(const int32_t* acc, const float* scale, float* out, int64_t M, int32_t N,
                                      void* stream) {
    if (M < 0 || N <= 0) return SPARQ_EINVAL;
    if (M == 0) return SPARQ_OK;
    if (!acc || !scale || !out) return SPARQ_EINVAL;
    if (M > (INT64_MAX / 8) / N) return SPARQ_EINVAL;
    return launch_per_channel<false>(acc, scale, out, M * N, N, static_cast<hipStream_t>(stream));
}

extern "C" sparq_status sparq_requant(const int32_t* acc, const float* factor, uint8_t* y, int64_t M, int32_t N,
                                      void* stream) {
    if (M < 0 || N <= 0) return SPARQ_EINVAL;
    if (M == 0) return SPARQ_OK;
    if (!acc || !factor || !y) return SPARQ_EINVAL;
    if (M > (INT64_MAX / 8) / N) return SPARQ_EINVAL;
    return launch_per_channel<true>(acc, factor, y, M * N, N, static_cast<hipStream_t>(stream));
}

extern "C" size_t sparq_packed_bytes(const sparq_conv_desc* desc) {
    ConvGeom g;
    return conv_geom(desc, &g) ? g.packed_bytes : 0;
}

extern "C" sparq_status sparq_pack_weights(const int8_t* w, const sparq_conv_desc* desc, void* packed,
                                           size_t packed_bytes, void* stream) {
    ConvGeom g;
    if (!w || !packed || !conv_geom(desc, &g) || !aligned(packed, 256)) return SPARQ_EINVAL;
    if (packed_bytes < g.packed_bytes) return SPARQ_EWORKSPACE;
    hipStream_t s = static_cast<hipStream_t>(stream);
    uint8_t* base = static_cast<uint8_t*>(packed);
    weight_colsum_kernel<<<g.Np, 64, 0, s>>>(w, reinterpret_cast<int32_t*>(base), g.N, g.fold_p * g.N, g.K);
    const int64_t chunks = (int64_t)(g.Kp / kChunk) * g.Np;
    if (g.fold)
        pack_weights_fold_kernel<<<ew_grid(chunks, kEwThreads), kEwThreads, 0, s>>>(
            w, reinterpret_cast<uint4*>(base + g.w_off), g.N, g.Np, g.C, g.KH, g.KW, g.Kp, g.fold_p, g.fold_kw,
            g.fold_kw_min, g.sw, g.pw);
    else
        pack_weights_kernel<<<ew_grid(chunks, kEwThreads), kEwThreads, 0, s>>>(
            w, reinterpret_cast<uint4*>(base + g.w_off), g.N, g.Np, g.C, g.Cq, g.KH * g.KW, g.Kp);
    return launch_status();
}

extern "C" const char* sparq_strerror(sparq_status status) {
    switch (status) {
        case SPARQ_OK: return "ok";
        case SPARQ_EINVAL: return "invalid argument";
        case SPARQ_EUNSUPPORTED: return "unsupported configuration";
        case SPARQ_EWORKSPACE: return "buffer too small";
        case SPARQ_ELAUNCH: return "HIP launch failed";
        default: return "unknown status";
    }
}
