// The packed-storage codec on four activations at a time (SIMD within a register), shared by the pack and unpack
// kernels; the record format is described in sparq_packed_act.hip.
//
// Packing: the shift of every byte follows from the residual mask low = 2^s - 1 the trim looks up (one byte permute
// more).  A pair with a zero stores the other value's 2n-bit window as two halves; it is brought into the ordinary
// form -- the value in both channels' places, the even one at shift t + n, the odd one at shift t -- so that one
// sequence of shifts (two bytes at a time, v_pk_lshrrev_b16) and one table of ShiftCtrl codes serves every pair.  The
// four data / ShiftCtrl / MuxCtrl fields of a word are squeezed together before they go into the record's bit strings.
// Unpacking runs the other way on eight channels: fields are spread to one byte each, even channels in one word, odd
// channels in another, so that a pair's two data sit in the same byte of the two words.
// The file compiles for the host as well (the intrinsics are emulated).
#pragma once
#include "sparq_swar.h"

namespace sparq {

struct PackLuts {
    TrimLuts trim;
    uint32_t code_lo, code_hi;       // ShiftCtrl code by shift 0..7, eight bytes
    uint32_t shift_lo, shift_hi;     // decoder: shift by ShiftCtrl code
};

inline PackLuts make_pack_luts(int n, uint32_t S) {
    PackLuts L{};
    uint64_t code = 0, shift = 0;
    int next = 0;
    for (int t = 0; t < 8; ++t) {
        code |= (uint64_t)__builtin_popcount(S & ((1u << t) - 1u)) << (8 * t);     // rank of t among the allowed shifts
        if ((S >> t) & 1u) shift |= (uint64_t)t << (8 * next++);
    }
    L.code_lo = (uint32_t)code; L.code_hi = (uint32_t)(code >> 32);
    L.shift_lo = (uint32_t)shift; L.shift_hi = (uint32_t)(shift >> 32);
    L.trim = make_luts(n, S);
    return L;
}

// Two 16-bit lanes shifted by the low four bits of the matching lane of s.
#if defined(__HIP_DEVICE_COMPILE__)
SPARQ_HD uint32_t shr16x2(uint32_t v, uint32_t s) { uint32_t r; asm("v_pk_lshrrev_b16 %0, %1, %2" : "=v"(r) : "v"(s), "v"(v)); return r; }
SPARQ_HD uint32_t shl16x2(uint32_t v, uint32_t s) { uint32_t r; asm("v_pk_lshlrev_b16 %0, %1, %2" : "=v"(r) : "v"(s), "v"(v)); return r; }
SPARQ_HD uint32_t min16x2(uint32_t a, uint32_t b) { uint32_t r; asm("v_pk_min_u16 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b)); return r; }
SPARQ_HD uint32_t add_up_bytes(uint32_t v, uint32_t sum) { return __builtin_amdgcn_sad_u8(v, 0u, sum); }
#else
SPARQ_HD uint32_t shr16x2(uint32_t v, uint32_t s) { return ((v & 0xFFFFu) >> (s & 15u)) | (((v >> 16) >> ((s >> 16) & 15u)) << 16); }
SPARQ_HD uint32_t shl16x2(uint32_t v, uint32_t s) { return (((v & 0xFFFFu) << (s & 15u)) & 0xFFFFu) | (((v >> 16) << ((s >> 16) & 15u)) << 16); }
SPARQ_HD uint32_t min16x2(uint32_t a, uint32_t b) {
    const uint32_t al = a & 0xFFFFu, bl = b & 0xFFFFu, ah = a >> 16, bh = b >> 16;
    return (al < bl ? al : bl) | ((ah < bh ? ah : bh) << 16);
}
SPARQ_HD uint32_t add_up_bytes(uint32_t v, uint32_t sum) { return sum + (v & 255u) + ((v >> 8) & 255u) + ((v >> 16) & 255u) + (v >> 24); }
#endif

constexpr uint32_t kEvenBytes = 0x00FF00FFu;

// s from per-byte masks 2^s - 1.  4-bit windows: s <= 4, and the permute's selector 15 (constant 255) serves as a ninth
// table entry; narrower windows: s <= 6, population count of two three-bit halves.
template <int N>
SPARQ_HD uint32_t mask_to_shift(uint32_t low) {
    if constexpr (N == 4) {
        return perm(0xF8000000u, 0xF900FAFBu, low) ^ 0xFBFBFBFBu;      // entries 0, 1, 3, 7: 0xFB ^ s; 15: 255 = 0xFB ^ 4
    } else {
        const uint32_t hi = (low >> 3) & 0x07070707u;
        return perm(0x03020201u, 0x02010100u, low & 0x07070707u) + perm(0x03020201u, 0x02010100u, hi);
    }
}

// Four fields of B bits in the four bytes' places of two words (even channels: 16-bit lanes of e, odd: of o) as one
// string of 4B bits in channel order.
template <int B>
SPARQ_HD uint32_t squeeze_fields(uint32_t e, uint32_t o) {
    const uint32_t v = e | (o << B);
    return (v & ((1u << (2 * B)) - 1u)) | (v >> (16 - 2 * B));
}
// OR a bit string of BITS bits into the words of an area at a position known at compile time.
template <int BITS, int WORDS>
SPARQ_HD void append_bits(uint32_t (&area)[WORDS], int pos, uint32_t value) {
    const int w = pos >> 5, off = pos & 31;
    area[w] |= value << off;
    if (off + BITS > 32 && w + 1 < WORDS) area[w + 1] |= value >> (32 - off);
}

struct PackedWord { uint32_t e, o, code, mux; };     // data (even / odd channels, 16-bit lanes), codes (bytes), MuxCtrl (byte masks)

// Four channels with a ShiftCtrl field each (group = 1).  N: window bits.
template <int N, int SB, bool PAIR, bool ROUND>
SPARQ_HD PackedWord pack_word(uint32_t x, const PackLuts& L) {
    constexpr bool kRankIsShift = N == 4 && SB == 3;     // five placements of a 4-bit window: every shift is allowed
    constexpr uint32_t kMask = ((1u << N) - 1u) * 0x00010001u;
    const uint32_t selA = (x >> 5) & 0x07070707u, selB = (x >> 2) & 0x07070707u;
    const uint32_t low = low_mask(selA, selB, L.trim.a_hi, L.trim.a_lo, L.trim.b_hi, L.trim.b_lo);
    uint32_t s = mask_to_shift<N>(low);
    uint32_t both = 0xFFFFFFFFu;                         // 16-bit lanes whose two values are non-zero
    PackedWord r{0, 0, 0, 0};
    if constexpr (PAIR) {
        const uint32_t f = nonzero_flag(x);
        const uint32_t nz = expand_bit7(f);
        both = nz & expand_bit7_swapped(f);
        // MuxCtrl: datum 1 goes to the odd channel if that is non-zero, datum 0 if it is and the even one is zero
        r.mux = perm(f << 8, f, 0x09090808u) & ~(nz & kEvenBytes);
        if constexpr (N == 4) {
            s = bfi(both, s, 0x00040004u);
        } else {
            const uint32_t lw = low_mask(selA, selB, L.trim.wa_hi, L.trim.wa_lo, L.trim.wb_hi, L.trim.wb_lo);
            const uint32_t tw = mask_to_shift<N>((lw | (lw >> 8)) & kEvenBytes);    // (a zero's mask is 0)
            s = bfi(both, s, (tw | (tw << 8)) + N * 0x00010001u);
        }
    }
    // what is shifted: the activation plus its rounding offset; residual bits fall off
    uint32_t v = x;
    if constexpr (ROUND && N == 4) {
        const uint32_t half = low & ~(low >> 1);
        const uint32_t sat = expand_bit7(lerp(x, perm(L.trim.ncap_hi, L.trim.ncap_lo, selA), 0u));
        v = x + (half & ~sat & both);
    } else if constexpr (ROUND) {
        v = trim4<true, PAIR, PAIR>(x, L.trim);
    }
    const uint32_t e = v & kEvenBytes, o = (v >> 8) & kEvenBytes;
    if constexpr (PAIR) {
        r.e = shr16x2(e | (o & ~both), s);
        r.o = shr16x2(o | (e & ~both), s >> 8) & kMask;
    } else {
        r.e = shr16x2(e, s);
        r.o = shr16x2(o, s >> 8);
    }
    r.code = kRankIsShift ? s : perm(L.code_hi, L.code_lo, s);
    return r;
}

// Shared shifts (group > 1): s and half are the group's shift and rounding offset in every byte of the group.
template <int N, bool ROUND>
SPARQ_HD PackedWord pack_word_shared(uint32_t x, uint32_t s, uint32_t half) {
    constexpr uint32_t kMask = ((1u << N) - 1u) * 0x00010001u;
    uint32_t e = x & kEvenBytes, o = (x >> 8) & kEvenBytes;
    if (ROUND) {
        const uint32_t h = half & kEvenBytes;              // a group holds whole pairs: even and odd bytes agree
        e = min16x2(shr16x2(e + h, s), kMask);
        o = min16x2(shr16x2(o + h, s), kMask);
    } else {                                               // the group's largest value fits its window: no saturation
        e = shr16x2(e, s);
        o = shr16x2(o, s);
    }
    return PackedWord{e, o, 0, 0};
}

// The data of two words as one bit string of 8N bits.
template <int N>
SPARQ_HD uint32_t squeeze_data(const PackedWord& a, const PackedWord& b) {
    if constexpr (N == 4) return perm(b.e | (b.o << 4), a.e | (a.o << 4), 0x06040200u);
    else return squeeze_fields<N>(a.e, a.o) | (squeeze_fields<N>(b.e, b.o) << (4 * N));
}

// Eight fields of B bits (a string of 8B bits) as one byte each: even fields in *e, odd fields in *o.
template <int B>
SPARQ_HD void spread_fields(uint32_t v, uint32_t* e, uint32_t* o) {
    constexpr uint32_t kField = ((1u << B) - 1u) * 0x01010101u;
    uint32_t u = v;
    if constexpr (B == 3) {
        u = (v & 0x00000FFFu) | ((v & 0x00FFF000u) << 4);
        u = (u & 0x003F003Fu) | ((u & 0x0FC00FC0u) << 2);
    } else if constexpr (B == 2) {
        u = (v & 0x000000FFu) | ((v & 0x0000FF00u) << 8);
        u = (u & 0x000F000Fu) | ((u & 0x00F000F0u) << 4);
    } else if constexpr (B == 1) {
        u = (v & 0x0000000Fu) | ((v & 0x000000F0u) << 12);
        u = (u & 0x00030003u) | ((u & 0x000C000Cu) << 6);
    }
    *e = u & kField;
    *o = (u >> B) & kField;
}
// BITS bits of an area at a position known at compile time (bits above them unspecified)
template <int BITS, int WORDS>
SPARQ_HD uint32_t read_bits(const uint32_t (&area)[WORDS], int pos) {
    const int w = pos >> 5, off = pos & 31;
    uint32_t v = area[w] >> off;
    if (off + BITS > 32 && w + 1 < WORDS) v |= area[w + 1] << (32 - off);
    return v;
}

SPARQ_HD uint32_t shift_bytes_left(uint32_t q, uint32_t s) {
    return shl16x2(q & kEvenBytes, s) | (shl16x2((q >> 8) & kEvenBytes, s >> 8) << 8);
}
SPARQ_HD uint32_t add_bytes(uint32_t a, uint32_t b) {      // per byte, modulo 256
    return ((a & 0x7F7F7F7Fu) + (b & 0x7F7F7F7Fu)) ^ ((a ^ b) & 0x80808080u);
}

// Eight channels from their data (even / odd), shifts (even / odd) and MuxCtrl string: Eq. 4, each datum adds to the
// channel its MuxCtrl names.
template <bool PAIR>
SPARQ_HD void unpack_eight(uint32_t de, uint32_t dd, uint32_t se, uint32_t so, uint32_t mux_rep, uint32_t* w0, uint32_t* w1) {
    uint32_t ev = shift_bytes_left(de, se), od = shift_bytes_left(dd, so);
    if constexpr (PAIR) {
        // mux_rep: the eight MuxCtrl bits in every byte; byte j looks at bits 2j and 2j + 1
        const uint32_t me = expand_bit7(nonzero_flag(mux_rep & 0x40100401u)), mo = expand_bit7(nonzero_flag(mux_rep & 0x80200802u));
        const uint32_t a = ev, b = od;
        ev = add_bytes(a & ~me, b & ~mo);
        od = add_bytes(a & me, b & mo);
    }
    *w0 = perm(od, ev, 0x05010400u);
    *w1 = perm(od, ev, 0x07030602u);
}

constexpr int kRecChannels = 32;
constexpr int codec_shift_words(int sb, int group) { return (kRecChannels / group * sb + 31) / 32; }
constexpr int codec_words(int n, int sb, int group, bool pair) { return n + codec_shift_words(sb, group) + (pair ? 1 : 0); }

// One record from 32 channels.  G channels share a ShiftCtrl field.
template <int N, int SB, int G, bool PAIR, bool ROUND>
SPARQ_HD void pack_record(const uint32_t (&w)[8], const PackLuts& L, uint32_t (&rec)[codec_words(N, SB, G, PAIR)]) {
    constexpr int SW = codec_shift_words(SB, G);
            uint32_t data[N] = {}, shifts[SW] = {}, mux = 0;
    PackedWord f[8];
    if constexpr (G == 1) {
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            f[i] = pack_word<N, SB, PAIR, ROUND>(w[i], L);
            append_bits<4 * SB>(shifts, i * 4 * SB, squeeze_fields<SB>(f[i].code & kEvenBytes, (f[i].code >> 8) & kEvenBytes));
        }
        if constexpr (PAIR) {
#pragma unroll
            for (int i = 0; i < 8; i += 2)
                mux |= add_up_bytes(f[i + 1].mux & 0x80402010u, add_up_bytes(f[i].mux & 0x08040201u, 0u)) << (4 * i);
        }
    } else {
        // the leading one of a group's largest value is the leading one of the OR of its values
        constexpr int GW = G >= 8 ? G / 4 : 1;                   // words per group (or one word with one or two groups)
#pragma unroll
        for (int i0 = 0; i0 < 8; i0 += GW) {
            uint32_t o = w[i0];
#pragma unroll
            for (int i = 1; i < GW; ++i) o |= w[i0 + i];
            o |= perm(o, o, 0x02030001u);
            if constexpr (G >= 4) o |= perm(o, o, 0x01000302u);
            const uint32_t low = low_mask((o >> 5) & 0x07070707u, (o >> 2) & 0x07070707u, L.trim.a_hi, L.trim.a_lo,
                                          L.trim.b_hi, L.trim.b_lo);
            const uint32_t s = mask_to_shift<N>(low), code = perm(L.code_hi, L.code_lo, s);
            const uint32_t half = low & ~(low >> 1);
            if constexpr (G == 2) append_bits<2 * SB>(shifts, i0 * 2 * SB, (code & 255u) | (((code >> 16) & 255u) << SB));
            else append_bits<SB>(shifts, i0 / GW * SB, code & 255u);
#pragma unroll
            for (int i = 0; i < GW; ++i) f[i0 + i] = pack_word_shared<N, ROUND>(w[i0 + i], s, half);
        }
    }
#pragma unroll
    for (int i = 0; i < 8; i += 2) append_bits<8 * N>(data, i * 4 * N, squeeze_data<N>(f[i], f[i + 1]));
#pragma unroll
    for (int i = 0; i < N; ++i) rec[i] = data[i];
#pragma unroll
    for (int i = 0; i < SW; ++i) rec[N + i] = shifts[i];
    if constexpr (PAIR) rec[N + SW] = mux;
}

// The 32 channels a record encodes.
template <int N, int SB, int G, bool PAIR>
SPARQ_HD void unpack_record(const uint32_t (&rec)[codec_words(N, SB, G, PAIR)], const PackLuts& L, uint32_t (&w)[8]) {
    constexpr int SW = codec_shift_words(SB, G), WORDS = codec_words(N, SB, G, PAIR);
            uint32_t data[N], shifts[SW];
    #pragma unroll
            for (int i = 0; i < N; ++i) data[i] = rec[i];
    #pragma unroll
            for (int i = 0; i < SW; ++i) shifts[i] = rec[N + i];
            #pragma unroll
            for (int q = 0; q < 4; ++q) {                        // eight channels at a time
                uint32_t de, dd, ce, co;
                spread_fields<N>(read_bits<8 * N>(data, q * 8 * N), &de, &dd);
                if constexpr (G == 1) {
                    spread_fields<SB>(read_bits<8 * SB>(shifts, q * 8 * SB), &ce, &co);
                } else {
                    constexpr uint32_t kCode = (1u << SB) - 1u;
                    if constexpr (G == 2) {                      // four fields: one per pair
                        const uint32_t f = read_bits<4 * SB>(shifts, q * 4 * SB);
                        ce = (f & kCode) | (((f >> SB) & kCode) << 8) | (((f >> (2 * SB)) & kCode) << 16) | (((f >> (3 * SB)) & kCode) << 24);
                    } else if constexpr (G == 4) {
                        const uint32_t f = read_bits<2 * SB>(shifts, q * 2 * SB);
                        ce = (f & kCode) * 0x0101u | ((f >> SB) & kCode) * 0x01010000u;
                    } else {
                        ce = (read_bits<SB>(shifts, q * 8 / G * SB) & kCode) * 0x01010101u;
                    }
                    co = ce;
                }
                unpack_eight<PAIR>(de, dd, perm(L.shift_hi, L.shift_lo, ce), perm(L.shift_hi, L.shift_lo, co),
                                   PAIR ? perm(rec[WORDS - 1], rec[WORDS - 1], 0x01010101u * q) : 0u, &w[2 * q], &w[2 * q + 1]);
            }
}

}  // namespace sparq
