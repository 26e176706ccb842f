// Host entry point of the fused SPARQ convolution: validation, the channel-padding
// pre-pass for channel counts that are not a multiple of four, and the choice of tile shape.
#include "sparq_conv_gemm_kernel.h"
#include "sparq_conv_block_kernel.h"
#include "sparq_conv_few_kernel.h"
#include "sparq_conv_patch_kernel.h"
#include "sparq_conv_rows_kernel.h"
#include "sparq_conv_cols_kernel.h"
#include "sparq_conv_split_kernel.h"
#include "sparq_conv_wide_kernel.h"

#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include <mutex>

using namespace sparq;

namespace {

// ---- the one test / tuning hook (sparq_set_tuning): process-wide overrides of the kernel choice ----
enum TunedForm { kTunedSplit = 1, kTunedRows, kTunedCols, kTunedWide, kTunedBlock };
struct Tuning {
    int path = 0;             // 0: rules decide, 1: gather kernel, 2: input-patch kernel
    char tile[16] = "";       // gather kernel tile "128x128" | "128x256" | "128x512"
    int patch_tn = 0;         // input-patch kernel: output channels per tile (64 / 128 / 256), 0: rules decide
    int patch_ws = -1;        // 1 / 0: wave-specialised / plain form, -1: rules decide
    int form = 0;             // 0: rules decide, else a TunedForm
    // one of the two tile kernels is asked for: the rules of the other forms do not apply
    bool set() const { return path || tile[0] || patch_tn || patch_ws >= 0; }
};
Tuning g_tuning;
std::mutex g_tuning_mu;
Tuning current_tuning() {
    std::lock_guard<std::mutex> lock(g_tuning_mu);
    return g_tuning;
}

struct TileEntry { const char* name; int tm, tn; TileLauncher fn; };
const TileEntry kTiles[] = {
    {"128x128", 128, 128, launch_tile_128x128_w2x2_a4b2},
    {"128x256", 128, 256, launch_tile_128x256_w1x4_a2b3},
    {"128x512", 128, 512, launch_tile_128x512_w1x4_half},
};

// Tile choice: the widest output-channel tile the layer fills, so that an activation
// is gathered and trimmed as few times as possible; the tuning hook forces one.
// A tile shape is usable only if all its weight loads stay inside the padded buffer; the 512-wide tile's
// main loop also needs every 64-byte reduction step to lie inside one filter tap (more than 32 channels).
bool tile_fits(int tn, const ConvGeom& g) { return round_up(g.N, tn) <= g.Np && (tn != 512 || g.Cq % kStepK == 0); }

// byte_output: the requantised uint8 output, which the 128x512 tile does not have.
TileLauncher pick_tile(const ConvGeom& g, const Tuning& tune, bool byte_output = false) {
    if (tune.tile[0])
        for (const TileEntry& t : kTiles)
            if (!strcmp(tune.tile, t.name) && tile_fits(t.tn, g) && !(byte_output && t.tn == 512)) return t.fn;
    if (g.N > 256 && tile_fits(512, g) && !byte_output) return kTiles[2].fn;
    if (g.N > 128) return kTiles[1].fn;
    return kTiles[0].fn;
}

// ---- input-patch kernel: eligibility and variant choice --------------------------------------
struct PatchVariant { int tn, ac, cbs; PatchLauncher fn; PatchLauncher fn_ws; PatchLauncher fn_sp; };   // plain, wave-specialised, sparse weights
const PatchVariant kPatchVariants[] = {
    {64, 2, 1, launch_patch_n64_a2c1, launch_patch_ws_n64_a2c1, launch_patch_sp_n64_a2c1},
    {64, 4, 1, launch_patch_n64_a4c1, launch_patch_ws_n64_a4c1, launch_patch_sp_n64_a4c1},
    {64, 8, 1, launch_patch_n64_a8c1, launch_patch_ws_n64_a8c1, launch_patch_sp_n64_a8c1},
    {64, 12, 1, launch_patch_n64_a12c1, launch_patch_ws_n64_a12c1, launch_patch_sp_n64_a12c1},
    {64, 4, 2, launch_patch_n64_a4c2, launch_patch_ws_n64_a4c2, launch_patch_sp_n64_a4c2},
    {64, 8, 4, launch_patch_n64_a8c4, launch_patch_ws_n64_a8c4, launch_patch_sp_n64_a8c4},
    {128, 2, 1, launch_patch_n128_a2c1, launch_patch_ws_n128_a2c1, launch_patch_sp_n128_a2c1},
    {128, 4, 1, launch_patch_n128_a4c1, launch_patch_ws_n128_a4c1, launch_patch_sp_n128_a4c1},
    {128, 8, 1, launch_patch_n128_a8c1, launch_patch_ws_n128_a8c1, launch_patch_sp_n128_a8c1},
    {128, 12, 1, launch_patch_n128_a12c1, launch_patch_ws_n128_a12c1, launch_patch_sp_n128_a12c1},
    {128, 4, 2, launch_patch_n128_a4c2, launch_patch_ws_n128_a4c2, launch_patch_sp_n128_a4c2},
    {128, 8, 4, launch_patch_n128_a8c4, launch_patch_ws_n128_a8c4, launch_patch_sp_n128_a8c4},
    {256, 2, 1, launch_patch_n256_a2c1, launch_patch_ws_n256_a2c1, launch_patch_sp_n256_a2c1},
    {256, 4, 1, launch_patch_n256_a4c1, launch_patch_ws_n256_a4c1, launch_patch_sp_n256_a4c1},
    {256, 8, 1, launch_patch_n256_a8c1, launch_patch_ws_n256_a8c1, launch_patch_sp_n256_a8c1},
    {256, 12, 1, launch_patch_n256_a12c1, launch_patch_ws_n256_a12c1, launch_patch_sp_n256_a12c1},
    {256, 4, 2, launch_patch_n256_a4c2, launch_patch_ws_n256_a4c2, launch_patch_sp_n256_a4c2},
    {256, 8, 4, launch_patch_n256_a8c4, launch_patch_ws_n256_a8c4, launch_patch_sp_n256_a8c4},
};

// Largest patch (in pixels) any tile of this geometry needs.  Tile positions repeat relative to the
// image with period lcm(128, Ho*Wo), so one period plus the last tile is an exact walk; results
// are cached because the same layers are launched over and over.
int patch_npix_max(const PatchGeom& g) {
    struct Key { int v[13]; int npix; };
    // 128 sets of four geometries (a layer's rules ask for up to four tile heights).  Four ways, because two layers that
    // push each other out pay the walk on every call: 12 us at 35 x 35 pixels, 193 at 147 x 147, against 0.1 for a look-up.
    struct Set { Key way[4]; unsigned next; };
    static Set cache[128];
    static std::mutex mu;
    const int key[13] = {g.tm, g.M, g.B, g.H, g.W, g.KH, g.KW, g.sh, g.sw, g.ph, g.pw, g.Ho, g.Wo};
    uint32_t hash = 0;
    for (int v : key) hash = (hash ^ (uint32_t)v) * 0x9E3779B1u, hash ^= hash >> 15;
    Set& set = cache[hash & 127];
    {
        std::lock_guard<std::mutex> lock(mu);
        for (const Key& k : set.way)
            if (!memcmp(k.v, key, sizeof(key))) return k.npix;       // (an empty way's tile height is 0)
    }
    const int64_t img = (int64_t)g.Ho * g.Wo;
    int64_t a = g.tm, b = img;
    while (b) { const int64_t t = a % b; a = b; b = t; }
    const int64_t period_tiles = img / a;                       // lcm(TM, img) / TM
    const int64_t tiles = ((int64_t)g.M + g.tm - 1) / g.tm;
    int npix = 0;
    for (int64_t t = 0; t < tiles && t <= period_tiles; ++t) {
        const int n = tile_patch(g, (int)(t * g.tm)).npix;
        npix = n > npix ? n : npix;
    }
    const int n_last = tile_patch(g, (int)((tiles - 1) * g.tm)).npix;
    npix = n_last > npix ? n_last : npix;
    std::lock_guard<std::mutex> lock(mu);
    Key& slot = set.way[set.next++ & 3];
    memcpy(slot.v, key, sizeof(key));
    slot.npix = npix;
    return npix;
}

// The patch geometry of `g` for tiles of `tm` output pixels and the largest patch; false: outside what the
// index arithmetic of the input-patch kernels covers.
bool patch_geom_for(const ConvGeom& g, int tm, PatchGeom* pg, int* npix) {
    if (g.Cq % kStepK != 0) return false;                        // fewer than 33 channels: taps are not step-aligned
    if (g.M >= kPatchMaxDividend || (size_t)g.Kp * g.Np >= kPatchInvalidOffset) return false;
    if ((int64_t)g.B * g.H * g.W >= kPatchMaxDividend) return false;     // the pixel remap of strided 1x1 layers
    PatchGeom q = make_patch_geom(g.B, g.H, g.W, g.KH, g.KW, g.sh, g.sw, g.ph, g.pw, tm);
    if ((int64_t)q.B * q.Hv + q.KH >= kPatchMaxDividend) return false;
    if (patch_npix_bound(q) > 4096) return false;               // far too large: skip the exact walk
    *npix = patch_npix_max(q);
    *pg = q;
    return true;
}

// Fills `pg`, `npix`, and picks staging (chunks per lane, channel block of at most 64 max_unit channels); false: not eligible.
bool plan_patch(const ConvGeom& g, int max_unit, PatchGeom* pg, int* npix, int* ac, int* cbs) {
    PatchGeom q;
    int n;
    if (!patch_geom_for(g, kPatchTM, &q, &n)) return false;
    const int taps = q.KH * q.KW;
    const int ksteps = g.Cq / kStepK;
    // candidates (chunks per lane, channel block / 64): larger channel blocks first for 1x1 layers,
    // the smallest staging that holds the patch otherwise
    static const int cand[6][2] = {{8, 4}, {4, 2}, {2, 1}, {4, 1}, {8, 1}, {12, 1}};
    for (const auto& c : cand) {
        const int a = c[0], cb = c[1];
        if (ksteps % cb || cb > max_unit) continue;
        if (n * 4 * cb > a * 256) continue;                      // patch does not fit the staging registers
        if (cb > 1 && taps > 1) continue;                        // multi-tap layers: 64-channel units
        const int as = a / 2, steps = taps * cb;
        const int unrolled = as + (((as ^ steps) & 1) ? 1 : 0);  // as the kernel lays out a unit
        if (cb == 1 && !(taps & 1)) continue;                    // 64-channel units need an odd tap count
        if (steps < unrolled) continue;                          // unit too short to stage all chunks
        *pg = q; *npix = n; *ac = a; *cbs = cb;
        return true;
    }
    return false;
}

// Output-channel tile and form of the patch kernel (rules fitted to per-layer measurements of the workload tables).
//   64 for narrow layers (wave-specialised, two workgroups of 8 wavefronts per CU: the accumulators are small
//   enough for 128 registers per lane), and for layers so small that 128-wide tiles would leave half the chip idle.
//   256 (wave-specialised: 4 matrix + 4 staging wavefronts, one workgroup per CU) when it pads N to no more columns
//   than 128-wide tiles would and either fills three quarters of the chip or the layer is small anyway; also for patches so large that LDS
//   holds one workgroup per CU anyway (strided 3x3 layers on large images) when the layer is wide and fills the chip.
//   128 otherwise: two plain workgroups per CU that hide each other's latencies for 1x1 layers with many tiles,
//   wave-specialised for multi-tap layers and for layers with no more tiles than CUs.
// The tuning hook forces tile width and form.
const PatchVariant* pick_patch(const ConvGeom& g, const Tuning& tune, int ac, int cbs, int npix, bool forced, bool* ws) {
    const int64_t tiles_m = (g.M + kPatchTM - 1) / kPatchTM;
    const int64_t t128 = tiles_m * ((g.N + 127) / 128), t256 = tiles_m * ((g.N + 255) / 256);
    const int cus = device_cu_count();
    int tn = g.N <= 64 ? 64 : 128;
    const bool same_columns = round_up(g.N, 256) == round_up(g.N, 128);
    if (g.N > 128 && same_columns && (t256 * 4 >= (int64_t)cus * 3 || (t128 <= cus && t256 * 8 >= cus))) tn = 256;
    if (g.N > 64 && t128 * 2 <= cus) tn = 64;      // a small layer: more, narrower tiles fill more CUs
    if (2 * 4 * cbs * patch_plane_stride(npix, 4 * cbs) > kLdsPerCu / 2) {
        if (g.N >= 256 && t256 >= cus) tn = 256;
        else if (g.N < 256 && t128 >= cus && !forced) return nullptr;   // narrow: gather kernel
    }
    *ws = tn != 128 || g.KH * g.KW > 1 || t128 <= cus;
    if ((tune.patch_tn == 64 || tune.patch_tn == 128 || tune.patch_tn == 256) && tile_fits(tune.patch_tn, g)) tn = tune.patch_tn;
    if (tune.patch_ws >= 0) *ws = tune.patch_ws != 0;
    const bool strided_1x1 = g.KH == 1 && g.KW == 1 && (g.sh > 1 || g.sw > 1);    // pixel remap: staging wavefronts only
    if (strided_1x1) *ws = true;
    for (const PatchVariant& v : kPatchVariants)
        if (v.tn == tn && v.ac == ac && v.cbs == cbs) {
            if (!v.fn_ws) *ws = false;
            if (strided_1x1 && !*ws) return nullptr;
            return &v;
        }
    return nullptr;
}

// 1x1 layers with a long reduction have nothing to reuse between taps; when they also
// fill the chip with wide tiles and waste little on channel padding, the gather kernel's wider
// tiles (each activation trimmed once for up to 512 output channels) are faster.
bool prefer_gather(const ConvGeom& g) {
    const bool gemm = g.KH == 1 && g.KW == 1 && g.ph == 0 && g.pw == 0;      // any stride
    if (!gemm || g.K < 768) return false;
    const int tn = (g.N > 256 && tile_fits(512, g)) ? 512 : g.N > 128 ? 256 : 128;
    const int64_t tiles = (g.M + 127) / 128 * ((g.N + tn - 1) / tn);
    return tiles >= device_cu_count() && round_up(g.N, tn) * 100 <= (int64_t)g.N * 115;
}

// ---- split-reduction form of the input-patch kernel: small layers ----------------------------
struct SplitVariant { const char* name; int tm, tn; int (*lds_bytes)(int, int); SplitLauncher fn; };
const SplitVariant kSplitVariants[] = {
    {"32x32", 32, 32, split_lds_bytes<Split32x32>, launch_split_32x32},
    {"32x64", 32, 64, split_lds_bytes<Split32x64>, launch_split_32x64},
    {"64x64", 64, 64, split_lds_bytes<Split64x64>, launch_split_64x64},
};

// The split form is taken by layers whose tiles, at one of its sizes, do not outnumber the CUs: the smallest such tile,
// and only if the reduction is long enough for the sharing to pay.  Measured, with its first form, over 235 small layers of the three tables
// (batch 1 to 128): 2.81 ms in the other kernels, 2.07 with this rule, 2.07 with the best choice layer by layer (7 x 7 x 512
// 3x3, one image: 13.6 -> 6.8 us; 56 x 56 x 64: 7.3 -> 5.5; 1x1 over 64 channels: 4.7 -> 5.2, hence the lower limits).
// With more tiles than CUs every tile's patch and its sum cost more than the shorter chain gains (four images of
// 56 x 56 x 64 at 32 x 32: 7.6 -> 11.8 us).
const SplitVariant* pick_split(const ConvGeom& g, PatchGeom* pg, int* npix) {
    static const int min_k[] = {128, 256, 512};
    if (g.M > 64 * 1024) return nullptr;
    for (size_t i = 0; i < sizeof(kSplitVariants) / sizeof(kSplitVariants[0]); ++i) {
        const SplitVariant& v = kSplitVariants[i];
        if ((g.M + v.tm - 1) / v.tm * ((g.N + v.tn - 1) / v.tn) > device_cu_count()) continue;
        if (g.K < min_k[i]) return nullptr;
        if (patch_geom_for(g, v.tm, pg, npix) && v.lds_bytes(*npix, g.Cq / kChunk) > 0) return &v;
    }
    return nullptr;
}
// The smallest tile that holds the layer's patch.
const SplitVariant* fit_split(const ConvGeom& g, PatchGeom* pg, int* npix) {
    for (const SplitVariant& v : kSplitVariants)
        if (patch_geom_for(g, v.tm, pg, npix) && v.lds_bytes(*npix, g.Cq / kChunk) > 0) return &v;
    return nullptr;
}

// ---- 1x1 layers with the activations in registers --------------------------------------------
// 1x1 layers without padding, inside the index arithmetic of the two forms made for them; `bytes`: 16 results leave together.
bool one_tap(const ConvGeom& g, bool bytes) {
    return g.KH == 1 && g.KW == 1 && !g.ph && !g.pw && g.Cq % kStepK == 0 && g.M < kPatchMaxDividend &&
           (size_t)g.Kp * g.Np < kPatchInvalidOffset && (int64_t)g.B * g.H * g.W < kPatchMaxDividend && !(bytes && g.N % 16);
}
struct RowsVariant {
    int steps;                               // 32-index reduction steps it holds
    const char* name;
    RowsLauncher fn;
    int rm, rm_large;                        // pixels per wavefront
    int (*held_run)(int64_t, int64_t, bool); // where its launcher holds the weights in LDS
};
const RowsVariant kRowsVariants[] = {
    {2, "64", launch_rows_k64, 32, 32, rows_held_run<2>}, {4, "128", launch_rows_k128, 32, 32, rows_held_run<4>}, {6, "192", launch_rows_k192, 32, 64, rows_held_run<6>},
    {8, "256", launch_rows_k256, 32, 64, rows_held_run<8>}, {10, "320", launch_rows_k320, 32, 64, rows_held_run<10>}, {12, "384", launch_rows_k384, 32, 64, rows_held_run<12>},
    {16, "512", launch_rows_k512, 32, 64, rows_held_run<16>},
};
// What its launcher takes beyond the rule below (else the call goes on to the tile kernels).
bool rows_launchable(const RowsVariant& v, const ConvGeom& g, bool bytes) {
    const int rm = rows_large(g.M, g.N) ? v.rm_large : v.rm;
    return g.N * 4ll * rm < 0x7FFFFFFF && rows_lds_bytes(rm, g.N, bytes) <= 64 * 1024;
}

const RowsVariant* fit_rows(const ConvGeom& g, bool bytes) {
    if (one_tap(g, bytes))
        for (const RowsVariant& v : kRowsVariants)
            if (g.Cq / 32 <= v.steps) return &v;
    return nullptr;
}

// Activations in registers: 1x1 layers without padding.  `bytes`: requantised results.
// Up to 512 channels it beats the tile kernels nearly everywhere, by 1.1-1.6 x on small tensors and up to 2.2 x on large ones
// (256 -> 64 channels, 802816 pixels 80 -> 69 us; 64 -> 256 bytes 106 -> 58; 128 -> 512 bytes 60 -> 35), except where four-byte
// results beyond the last-level cache leave in rows of 400 bytes or more (64 -> 256, 802816 pixels: 154 against 170 us: the
// tile kernels write whole rows at a time).  Where little arithmetic stands beside the stores -- up to 192 channels, 256 without a
// trim -- that begins at half its size (128 -> 448, 144611 pixels, 247 MiB 49 against 57; 128 -> 560, 92466 pixels, untrimmed, 198 MiB
// 48 against 54; 110 timed layers of more than 96 outputs between 128 and 256 MiB: 1.03 x of the tile kernels' time up to
// that many channels, 0.84 x beyond).  (Holding 768 or 1024 channels was built too: behind the form below.)
const RowsVariant* pick_rows(const ConvGeom& g, bool bytes, bool plain) {
    if (!bytes && g.N > 96 && g.M * g.N * 4 >= (g.Cq <= (plain ? 256 : 192) ? kStreamedBytes / 2 : kStreamedBytes)) return nullptr;
    // (four-byte rows that start off a 64-byte border: its 128-byte runs are two partial lines each, the tile kernels' rows are
    // not; 196 -> 948, 28187 pixels 57 against 85 us.  Up to 8 MiB the shorter chain is worth more: 1.0-1.5 x faster at 2 to 8 MiB over 75
    // layers of 64 to 512 channels, between 1.6 x faster and 1.3 x slower at 12 to 16, 1.1-2.2 x slower at 32 to 64.)
    if (!bytes && g.N % 16 != 0 && g.M * g.N * 4 > (8 << 20)) return nullptr;
    return fit_rows(g, bytes);
}

// ---- 1x1 layers with the weights in registers ------------------------------------------------
struct ColsVariant { int steps; const char* name; RowsLauncher fn; };
const ColsVariant kColsVariants[] = {{8, "256", launch_cols_k256}, {12, "384", launch_cols_k384}, {16, "512", launch_cols_k512}, {24, "768", launch_cols_k768}, {32, "1024", launch_cols_k1024}};

const ColsVariant* fit_cols(const ConvGeom& g, bool bytes) {
    if (one_tap(g, bytes) && g.N * 4ll * 32 < 0x7FFFFFFF && (g.N + 255) / 256 <= device_cu_count() / 8)
        for (const ColsVariant& v : kColsVariants)
            if (g.Cq / 32 <= v.steps) return &v;
    return nullptr;
}

// How its launch splits the output channels: groups of 64 (beyond 512 channels 32) to a wavefront, eight (where two hold the same ones, four) groups to
// a share; tenths of a round: 32-pixel fragments for each workgroup of a share.
struct ColsSplit {
    bool two, narrow;
    int64_t groups, per, shares, tenths;
    ColsSplit(const ColsVariant& v, const ConvGeom& g) : two(v.steps <= 16), narrow(two && g.N <= 256) {
        groups = (g.N + (two ? 63 : 31)) / (two ? 64 : 32);
        per = narrow ? 4 : 8;
        shares = (groups + per - 1) / per;
        tenths = (g.M + 31) / 32 * 10 / (device_cu_count() / (8 * shares) * 8);
    }
};

// Weights in registers, against the forms above and below by 32808 timed layers of 129 to 768 channels and 8749 of up to 1024, in rounds (above);
// `full`: wavefronts that have channels.
//   Up to 512 channels it walks 512 outputs per share: beyond 256 outputs, with the steps it is built for at least 7/8 filled, 256 channels 1.02-1.17 x
//   from 1.3 rounds on (before 0.86-1.02), 384 as bytes 1.05-1.28 from 0.5 on, four-byte results 1.06-1.35 from four on (at three 0.97), 512
//   as bytes 1.08-1.39 from 0.4 on, four-byte results 1.01-1.58 from 0.5 on; less filled (160 and 192, 320 channels) 1.04-1.13 from six rounds on but for
//   bytes of the former (0.95-1.03).  320 and 640 outputs leave three wavefronts of eight idle (0.93-1.03), 768 as bytes two (from four rounds on 1.03-1.12,
//   a fifth below 0.95).  Untrimmed four-byte results that the form above leaves to the tile
//   kernels stay there, as do up to one round of more than 768 channels that the form below leaves.  Up to 256 outputs, where two
//   wavefronts share their weights, from four rounds on: 384 and 512 channels as bytes 1.04-1.19 (1.0 for 160 outputs, a fifth of
//   whose columns would be padding), 384 from 177 outputs on 1.05-1.08; 256 channels 0.83-1.03, 512 with four-byte results 0.6-0.88 (registers spill).
//   Up to 1024 channels it walks 256.  Beyond 768: bytes 1.16-1.44 x between a half and two rounds, four-byte results 1.09-1.25, both
//   0.89-1.04 from there to four (bytes up to 160 outputs 1.08), then up to 256 outputs 1.1-1.3 (97 to 128 as four-byte results 1.02, a quarter below
//   0.95), four-byte results of more 1.03-1.15 up to twenty rounds, bytes of more 0.92-1.07 (128 x 512 tiles).
//   Up to 768: 1.1-1.4 x between a half and two rounds, where the tiles of the eight-wavefront form fill their last round least
//   (96 and 128 outputs 1.02-1.15, with a third below 0.95); beyond four 1.15-1.29 up to 256 outputs, four-byte results of more 1.05-1.17 (bytes
//   0.97-1.16); between them 1.07-1.14 for 129 to 192 outputs, others 0.92-1.07.
//   The form above is at its best where its last round is more than three quarters full: 32 pixels for each of two wavefronts per SIMD, the outputs split over
//   as many wavefronts as a round then takes (`fills`), or 64 pixels (`last`; bytes of wide outputs over many pixels, of more than one share).
//   There the weights are 0.97 x up to 256 outputs (bytes of 193 and more 1.03-1.2), 0.99 with 384 channels and four-byte results (0.79 at worst); bytes in
//   a round of 64 pixels per wavefront three quarters to seven eighths full 1.02-1.08 with all wavefronts at work (256 channels seven eighths of them) and
//   0.93 else, fuller 0.91 (272 -> 1280, 112981 pixels 59 against 84 us), in half a round 0.95 with idle wavefronts or 320 channels (512: 1.05-1.17);
//   everywhere else 1.02-1.4.  (70600 timed layers; 1.1 % of those it takes are below 0.95 x, the lowest 0.81.)
//   Beyond 512 channels a share is 256 outputs, where a tile of the form below has 512, so with an even number of shares it trims twice as often.  Four-byte
//   results under the trims with the most arithmetic (`heavy`: windows of two or three bits with rounding and pairs) were then 0.94 x from four
//   rounds on with more than 768 channels (1.06-1.15 between eight and ten, where the form below starts a round), with up to 768 0.93 from twenty
//   rounds on and 0.97-1.05 between six and eight (768 -> 1024, 80384 pixels, two-bit windows 106 against 149 us; rows off a 64-byte border, which the
//   form below writes as slowly, 1.16-1.25).
//   Four-byte rows off a 64-byte border leave as pieces of lines, which only the caches put together again; the tile kernels write such rows
//   whole.  19000 timed layers: up to 512 channels 1.0-1.3 x up to 24 MiB of results, beyond 0.43-1.0 (284 -> 1625, 46644 pixels 122 us against 222), and
//   0.81-1.0 where the forms above or below stand; up to 768 channels 1.13-1.26 up to 80 MiB.  From there on, 1500 layers on up to 16 buffers in turn: up to 768
//   channels 1.05-1.1 up to 140 MiB, then even (0.97-1.03; on the same buffers 0.9 from there on), rows on a 32-byte border 1.02-1.08 up to 384; up to 1024
//   channels 1.06-1.18 up to the most that the lines below let through (160).
//   In its first rounds a trim with little arithmetic leaves the forms above and below less to win against (84500 timed layers of 133 to 512 channels on the same
//   buffers, 44200 on 16 in turn; the latter): four-byte results of 448 and 512 channels, untrimmed 0.90-0.92 x below one round (0.69 at worst; 512 channels with
//   all wavefronts at work 1.03) and 1.04 up to 1.3, beside the form below 0.87-0.98 up to 2.5; windows that round down 0.96-0.98 between 1.0 and 1.3
//   (on the same buffers 0.94; all at work beside the form above 1.01); 193 to 256 channels from 1.6 to 2.2 rounds with a tenth of the wavefronts idle
//   0.96-1.01 (0.92-0.96).  What rounds is 1.02-1.2 there.
// `trim`: what the kernel itself trims with (none beside the padded copy).
const ColsVariant* pick_cols(const ConvGeom& g, bool bytes, TrimKind trim, bool rows, bool wide) {
    const bool plain = trim == kTrimNone, light = trim <= kTrimFloorPairWide, heavy = trim == kTrimRoundPairWide;
    const ColsVariant* v = g.Cq > 128 && (bytes || rows || !plain || g.Cq > 512) ? fit_cols(g, bytes) : nullptr;
    if (!v) return nullptr;
    const ColsSplit split(*v, g);
    const bool two = split.two, narrow = split.narrow;
    const int64_t groups = split.groups, per = split.per, shares = split.shares, tenths = split.tenths;
    const bool filled = g.Cq * 8 >= v->steps * 32 * 7, full = groups * 10 >= shares * per * (bytes && v->steps < 16 && tenths >= 40 ? 8 : 7);
    if (!bytes && g.N % 16) {
        const int64_t mib = g.M * g.N * 4 >> 20;
        if (two ? rows || wide || mib >= 24 : v->steps == 24 && mib >= (g.N % 8 == 0 ? 384 : 140)) return nullptr;
    }
    const int64_t round = (int64_t)device_cu_count() * 256, last = (g.M - 1) % (2 * round) + 1;
    const bool fills = g.M <= round >> (shares - 1) && g.M * 4 > (round >> (shares - 1)) * 3;
    if (narrow ? fills && !(bytes && g.N > 192) : v->steps == 12 && !bytes && fills) return nullptr;
    if (bytes && two && shares > 1 && rows_large(g.M, g.N)) {
        const int eighths = v->steps == 8 ? 7 : 8;           // of the wavefronts
        if (last * 8 > 2 * round * 7) return nullptr;
        if (last * 4 > 2 * round * 3 && !(filled && groups * 8 >= shares * per * eighths)) return nullptr;
        if (g.M <= round && v->steps < 16 && !(filled && groups * 8 >= shares * per * 7)) return nullptr;
    }
    if (heavy && !two && !bytes && g.N % 16 == 0 && shares % 2 == 0) {
        const bool slower = v->steps == 24 ? tenths >= 200 || (tenths >= 60 && tenths < 80) : tenths >= 40 && !(tenths >= 80 && tenths < 100);
        if (slower) return nullptr;
    }
    if (!bytes && two && !narrow && light) {
        const bool all = groups == shares * per;
        if (v->steps == 16 && plain && ((tenths < 10 && !(all && g.Cq > 448)) || (wide && tenths < 25))) return nullptr;
        if (v->steps == 16 && !plain && tenths >= 10 && tenths < 13 && !(all && rows)) return nullptr;
        if (v->steps == 8 && tenths >= 16 && tenths < 22 && groups * 10 < shares * per * 9) return nullptr;
    }
    bool take;
    if (narrow) take = filled && tenths >= 40 && v->steps > 8 && groups * 64 - g.N <= 16 && (bytes ? g.N > 96 : v->steps == 12 && g.N > 176);
    else if (two && !filled) take = full && tenths >= 60 && (!bytes || v->steps == 12);
    else if (two) take = full && tenths >= (v->steps == 8 ? 13 : v->steps == 12 ? (bytes ? 5 : 40) : bytes ? 4 : 5);
    else if (tenths < 20) take = tenths >= (v->steps == 24 || wide ? 5 : 10) && (full || shares == 1) && g.N > (bytes && v->steps == 32 ? 64 : 128);
    else if (tenths < 40) take = v->steps == 24 ? g.N > 128 && g.N <= 192 : bytes && g.N > 64 && g.N <= 160;
    else take = g.N <= 256 ? g.N > (!bytes && v->steps == 32 ? 128 : 64) : !bytes && full && (v->steps == 24 || tenths < 200);
    return take ? v : nullptr;
}

// ---- 1x1 layers with a long reduction: eight wavefronts per tile ------------------------------
struct WideVariant { const char* name; int tn; WideLauncher fn; };
const WideVariant kWideVariants[] = {{"128x512", 512, launch_wide_512}, {"128x256", 256, launch_wide_256}};
bool fit_wide(const ConvGeom& g, bool bytes) { return one_tap(g, bytes) && g.Cq > 4 * kStepK; }      // (its requests run six steps ahead)

// Eight wavefronts per tile: 1x1 layers without padding and with more than 512 channels, whatever their size (what the split
// form does not take), except few output channels, where the 256-wide tile multiplies mostly padding (784 -> 48: 12 against 15 us; 97 to 128
// outputs are ahead in one round of tiles, 24576 x 768 -> 128 1.17 x, and behind in two, 36992 x 768 -> 128 0.97 x, bytes 0.87 x).  Over
// 220 shapes of 768 to 4608 channels (128..2048 outputs, 784..50176 pixels) 1.02 to 2 x faster than the kernels it replaced:
// 65536 x 4608 x 512 int32 197 -> 172 us, bytes 233 -> 154; 50176 x 4608 x 320 207 -> 118; 50176 x 1024 -> 256 bytes 34 -> 28.
// With 449 to 512 channels the activations fit in registers, and that form is ahead once there are many rounds of
// tiles; in one well-filled round (196 tiles: 12544 x 512 -> 512 14.1 against 11.9 us), or two for bytes, this one is.
// The 512-wide tile costs about 1.35 times the 256-wide one's round and does twice the work.
// With tiles for less than half the CUs the tile kernels' narrower tiles use more of the chip, unless a long reduction is trimmed
// (3123 timed layers, 8 to 1200 tiles of 128 x 256: the kernels it replaced are 1.1-1.3 x faster up to 64 tiles below 1024 channels, up to 1.48 x
// faster where nothing is trimmed -- 867 x 4336 -> 960, untrimmed, 21 against 30 us; 0.89-0.94 x at 1024 channels and more with a trim).  Without
// a trim there is less to share out, so neither up to 128 outputs (18828 x 4608 -> 128 bytes 23 against 34) nor where more than a fifth of
// the columns are padding and the rounds are not full (9408 x 2688 -> 288 bytes 18 against 23); with one, such padding needs 640
// channels (9218 x 576 -> 272 bytes 10.2 against 12.0).  With these lines 23 of the 3123 are more than 6 % slower than the kernels it replaced, before 563.
// forced: by the tuning hook, only the tile is chosen.
const WideVariant* pick_wide(const ConvGeom& g, bool bytes, bool plain, bool forced = false) {
    if (!fit_wide(g, bytes)) return nullptr;
    if (!forced && (g.Cq < 512 || g.N <= 96 || (g.N <= 128 && g.M >= 32 * 1024))) return nullptr;
    const int64_t cus = device_cu_count(), tiles_m = (g.M + 127) / 128;
    const int64_t t512 = tiles_m * ((g.N + 511) / 512), t256 = tiles_m * ((g.N + 255) / 256);
    const int64_t r512 = (t512 + cus - 1) / cus, r256 = (t256 + cus - 1) / cus;
    const bool wider = g.N > 256 && r512 * 27 <= r256 * 20 && round_up(g.N, 512) <= g.Np;
    if (!forced) {
        const bool half = t256 * 2 >= cus, padded = round_up(g.N, 256) * 4 > (int64_t)g.N * 5;
        if (plain ? !half || g.N <= 128 || (padded && !wider && t256 * 4 < r256 * cus * 3)
                  : padded && g.Cq < 704 ? t256 <= cus
                                         : !half && (g.Cq < 1024 || (bytes && t256 * 4 < cus)))
            return nullptr;
    }
    if (g.Cq == 512 && !forced) {
        const bool fills = wider ? bytes && r512 <= 2 && t512 * 10 >= r512 * cus * 7 : r256 == 1 && t256 * 8 >= cus * 3;
        if (!fills || round_up(g.N, wider ? 512 : 256) * 4 > (int64_t)g.N * 5) return nullptr;     // (or pads N by over a quarter)
    }
    return &kWideVariants[wider ? 0 : 1];
}

// ---- multi-tap layers as many small workgroups -----------------------------------------------
struct BlockVariant { const char* name; int tm, tn; bool (*launchable)(int64_t, int64_t, int); BlockLauncher fn; };
const BlockVariant kBlockVariants[] = {
    {"256x64", 256, 64, block_launchable<Block256x64>, launch_block_256x64},
    {"128x128", 128, 128, block_launchable<Block128x128>, launch_block_128x128},
};
const BlockVariant* fit_block(const ConvGeom& g, bool bytes, const BlockVariant& v, PatchGeom* pg, int* npix) {
    PatchGeom q;
    int n;
    if (g.KH * g.KW == 1 || (bytes && g.N % 16) || !patch_geom_for(g, v.tm, &q, &n) || !v.launchable(g.M, g.N, n)) return nullptr;
    *pg = q;
    *npix = n;
    return &v;
}

// Small workgroups: multi-tap layers with tiles for every CU (300 and more: from 250 to 310 tiles of 56 x 56 x 64 it is within
// 5 % of the tile kernel, with 147 10.9 against 10.5 us, with 392 13.0 against 15.4) and
//   up to 64 channels, if they have at most 64 outputs or a patch of less than 450 pixels per tile (1.0-1.5 x faster there:
//   56 x 56 x 64 -> 64 3x3, batch 32 16.5 -> 13.1 us, batch 256 78 -> 58; wider rows trim too much per 64 outputs),
//   or 113 to 128 with such a patch, for bytes (28 x 28 x 128 -> 128, batch 256 47 -> 42; 65 to 112 channels: fp32
//   0.86-1.04 x, bytes 0.78-1.10 x on rows up to 17 pixels and 0.93-1.26 x up to 128 outputs from 28 on, which the tile kernel keeps),
//   or a patch too large for the tile kernel's staging, which the gather kernel would trim once per tap, if they have 15 taps
//   and more or few channels on either side (1.5-3 x: 56 x 56 x 64 -> 64 5x5, batch 32; 98 x 98 x 539 -> 128 3x3 67 against 78).
//   Of 65 to 128 outputs the gather kernel makes one column tile: with fewer than 15 taps it then trims hardly more, and a
//   filter one column wide makes the patch tall (untrimmed fp32 3x1 0.95-1.37 x of the gather kernel's time, 1.12 on average; 40 x 40 x 48 -> 96
//   7x1 untrimmed bytes 41 against 50 us; trimmed fp32 up to 131072 pixels 1.05-1.12 x, beyond 0.92-1.0; 129 outputs and more 0.56-0.92 x).
//   Rows of fp32 off a 64-byte border cost the gather kernel more: untrimmed 0.67-0.9 x from 100 outputs on, but 1.05-1.16 x from 72 to 92
//   (70 x 70 x 64 -> 88 3x2 39 against 44).  2x2 and 2x4 0.88-1.08 x, 4x4 and 5x5 0.5-0.9 x.
// With fewer tiles, or more channels, the tile kernel's pipelining is ahead (14 x 14 x 256, batch 256: 35 against 44 us).
// Its four-byte results leave in runs of 128 bytes, so rows off a 64-byte border are for the tile kernel beyond 64 outputs (112 x 112 x 48 ->
// 86 1x3 19 against 38 us), and fewer than nine taps (seven up to 64 outputs) do not pay for them (1x3 40 x 40 x 48 -> 126 30 against 42); it trims
// a patch once per 64 outputs, the tile kernel per 128 or 256, which decides where images are narrow (8 x 8 x 64 -> 160 fp32
// 10.4 against 12.7; bytes beyond 128 outputs 12 x 12 x 48 -> 192 7x1 81 against 95) and with 113 to 128 channels beyond 64 outputs (35 x 35 x 128 -> 256
// bytes 55 against 61; 14 x 14 x 128 -> 96 14 against 16; up to 128 outputs on rows of 28 pixels and more it stays 1.02-1.15 x ahead).  With
// these lines 58 of 3002 timed layers are more than 6 % slower than on the tile kernels, before 217.
const BlockVariant* pick_block(const ConvGeom& g, bool bytes, bool plain, bool gather, PatchGeom* pg, int* npix) {
    const int taps = g.KH * g.KW;
    if (taps == 1 || block_tiles<Block256x64>(g.M, g.N) < 300) return nullptr;
    gather = gather && (g.Cq == 64 || g.N <= 64 || taps >= 15) && g.Cq <= 256;
    if (gather && g.N > 64 && g.N <= 128 && taps < 15) {
        const bool column = g.KW == 1, aligned = g.N % 16 == 0;
        if (bytes ? plain && column && taps >= 5 : plain ? (aligned ? column : g.N >= 72 && g.N < 96) : aligned && column && g.M <= 128 * 1024)
            return nullptr;
    }
    if (!gather) {
        if (g.Cq > 128) return nullptr;
        if (!bytes && (g.N <= 64 ? taps < 7 : taps < 9 || g.N % 16 || (!plain && g.Wo <= 8))) return nullptr;
        if (bytes && !plain && (g.Cq == 64 ? g.N > 128 && g.Wo <= 14 : g.N > 128 || (g.N > 64 && (g.Wo < 28 || taps < 9)))) return nullptr;
    }
    // patch pixels of a tile that starts and ends anywhere in its rows (the largest one may cross two images)
    const bool small = ((int64_t)Block256x64::kTM + (int64_t)g.KH * g.Wo) * ((int64_t)(g.Wo - 1) * g.sw + g.KW) < 450ll * g.Wo;
    if (!gather && !(g.Cq == 64 ? g.N <= 64 || small : small && bytes && g.C > 112)) return nullptr;
    return fit_block(g, bytes, kBlockVariants[0], pg, npix);
}

// The 128 x 128 tile: layers of more than 64 outputs whose patch it trims half as often as the 256 x 64 tile does, and the 256 x 64 tile for
// narrower ones with many tiles, where they are ahead of the kernel the layer would take (picked: 256 x 64; tn: the tile kernel's output
// channels per tile, 0 the gather kernel).  17710 timed layers of 3, 7, 9 and 25 taps that the tile kernel would take, by its tiles over
// the CUs (rounds).  The rule moves 3910 of 30014 other layers, drawn later, here: 1.14 x faster, 24 of them below 0.95 x (the worst
// 0.86 x, 31 x 31 x 160 -> 128 3x3/2 in exactly two full rounds):
//   tiles 256 wide (one workgroup per CU: a round that is not full costs it most): 64 channels 1.08-1.28 x (images of 8 pixels a row 0.85); 128
//   channels up to half a round 1.10, from one to four 1.03-1.16 (between 0.5 and 1: 1.00); up to 384 channels in the first third of a second
//   round 1.04-1.09, then 0.88-0.98; and not where fewer than four workgroups share a CU (3x3/2 on 19 x 19 x 128 -> 256 0.79);
//   tiles 128 wide: 64 channels 1.01-1.22, rows of fp32 off a 64-byte border aside (N = 292 and 101 0.85 and 0.71); up to 256 channels from one round
//   on 1.00-1.15 (less than one 0.78-0.91: too few tiles for workgroups that do not pipeline), up to 512 from two on 1.06-1.11 (before 0.94-1.01);
//   four-byte results beyond six rounds and patches of which three do not fit a CU were not timed and stay; 65 to 128 channels as bytes:
//   1.06 where 256 x 64 was taken, beyond 128 outputs 1.15 against the tile kernel;
//   177 to 192 outputs fill three columns of 64, not two of 128: 256 x 64 for these, 1.03-1.2 x, a second round that is half empty aside
//   (0.985; 320 outputs 1.00; as fp32 in half a round of the tile kernel's 0.98: they stay); 129 to 176 outputs of 64 channels fill
//   those as well, and stay on 256 x 64 where they were (0.97);
//   tiles 64 wide: 256 x 64 from three rounds on 1.12-1.28 (before 0.76-1.04), 64 channels from one on 1.14; fewer than seven taps only as bytes;
//   (the tests of the plan pin to the tile kernel: rows of up to 14 pixels, 65 to 112 channels over more than four rounds, fewer than seven taps as fp32
//   and, as fp32, 113 to 128 channels under a 3x3 filter; they were 1.07-1.15 x here as well);
//   the gather kernel's layers, trimmed once per tap there: nine taps and more, up to 128 channels, 65 to 384 outputs 1.02-1.55 x
//   in up to 1200 tiles (35 x 35 x 96 3x3/2 23.2 against 19.9 us; more tiles 0.88-1.4 x, more outputs 0.8-1.1 x), of 65 to 128 channels and up
//   to 14 taps while three workgroups share a CU (beyond 803 patch pixels 280 layers of 3x3/2 0.93 x, 93 x 93 x 112 -> 320, twelve images, 30.2 against
//   45.3; 700 to 803 of them 1.04 x, and 64 channels 1.05 x), and 15 taps and more whose patch for 256 pixels does not fit (78 x 78 x 128 -> 48
//   5x5 125 against 76).
const BlockVariant* pick_block_square(const ConvGeom& g, bool bytes, bool plain, const BlockVariant* picked, int tn, PatchGeom* pg, int* npix) {
    const int taps = g.KH * g.KW;
    const int64_t cus = device_cu_count(), t128 = block_tiles<Block128x128>(g.M, g.N);
    if (taps == 1 || g.Cq > 512 || !block_launchable<Block256x64>(g.M, g.N, 0)) return picked;
    PatchGeom q;
    int n;
    const auto share_cu = [&](int workgroups) { return fit_block(g, bytes, kBlockVariants[1], &q, &n) && workgroups * block_lds_bytes<Block128x128>(n) <= kLdsPerCu; };
    bool square = false;
    if (tn == 0) {
        if (t128 <= cus || plain || picked || g.Cq > 128) return picked;
        const bool shared = g.Cq == 64 || taps >= 15 || share_cu(3);
        square = (taps >= 9 && g.N > 64 && g.N <= 384 && t128 <= 1200 && shared) || (taps >= 15 && g.N <= 384 && !fit_block(g, bytes, kBlockVariants[0], &q, &n));
    } else if (bytes || taps >= 7) {
        const bool lines = bytes || g.N % 16 == 0;
        const int64_t t = (g.M + kPatchTM - 1) / kPatchTM * ((g.N + tn - 1) / tn);       // the tile kernel's tiles
        if (tn == 64) return picked || g.N > 64 || t <= (g.Cq == 64 ? 1 : 3) * cus || !lines ? picked : fit_block(g, bytes, kBlockVariants[0], pg, npix);
        if (tn == 256) {
            const bool third = t * 3 <= cus * 4;
            if (g.Cq == 64) square = (third && (plain || g.Wo > 8)) || (g.Wo > 14 && lines && (g.N > 176 || !picked));
            else square = third && t > cus ? g.Cq <= 192 || (g.Cq <= 384 && lines && share_cu(4))
                                           : g.Cq == 128 && lines && ((t * 2 <= cus && (bytes || g.N > 192)) || (g.Wo > 14 && t > cus && t <= 4 * cus)) && share_cu(4);
        } else if (g.Cq == 64) square = bytes || (g.N % 16 == 0 && (!picked || g.N <= 128));
        else if (g.Cq == 128 && bytes && g.N > 128) square = true;
        else if (picked) square = g.Cq == 128 && bytes;
        else if (g.Cq == 128 && !bytes) square = lines && g.Wo > 14 && t > cus && t <= 6 * cus && (g.KH == 1 || g.KW == 1 || (plain && g.C <= 112));
        else square = lines && g.Wo > 14 && t > (g.Cq <= 256 ? 1 : 2) * cus && (bytes || t <= 6 * cus) && (g.Cq > 128 || g.C > 112 || plain || t <= 4 * cus) && share_cu(3);
        // (fewer tiles than CUs leave half of them idle, unless the tile kernel's are half as many again)
        if (t128 <= cus && !(tn == 256 && g.Cq <= 128 && t128 * 4 >= cus)) square = false;
    }
    const int64_t t256 = block_tiles<Block256x64>(g.M, g.N);
    if (square && tn && g.N > 176 && g.N <= 192 && (t256 <= cus || t256 * 2 > cus * 3)) {
        const BlockVariant* v = fit_block(g, bytes, kBlockVariants[0], pg, npix);
        if (v) return v;
    }
    const BlockVariant* v = square ? fit_block(g, bytes, kBlockVariants[1], pg, npix) : nullptr;
    return v ? v : picked;
}

// Everything the entry points decide before launching.
struct ConvPlan {
    const SplitVariant* split = nullptr;   // split-reduction form (then pg and npix are its own)
    const RowsVariant* rows = nullptr;     // activations in registers; what follows is for calls it does not take
    const ColsVariant* cols = nullptr;     // weights in registers; what follows is for calls it does not take
    const WideVariant* wide = nullptr;     // eight wavefronts per tile; what follows is for calls it does not take
    const BlockVariant* block = nullptr;   // small workgroups (then pg and npix are its own)
    FewGeom few{};                         // at most four channels (steps != 0)
    bool patch = false;
    const PatchVariant* variant = nullptr;
    PatchGeom pg{};
    int npix = 0, ac = 0, cbs = 0;
    bool ws = false;            // wave-specialised form of the patch kernel
    bool copy = false;          // the kernel reads a channel-padded, trimmed copy of x
    size_t pad_bytes = 0;       // room for that copy (channel counts that are not a multiple of 16: asked for whether or not it is made)
};

// forms: the forms other than the two tile kernels may be taken (where the tuning hook asks for a tile kernel, no rule takes them; where
// it asks for one of them, that one wherever the layer fits it).  Layers with 2:4 pruned weights are planned both ways (make_sparse_plan).
// bytes: requantised results.  kind: the layer's mode's trim (size queries and descriptors without one do not care).
// copy: the channel-padded copy is made (channel counts that are not a multiple of 16).
ConvPlan make_plan_of(const ConvGeom& g, const Tuning& tune, bool forms, bool bytes, TrimKind kind, bool copy) {
    ConvPlan pl;
    const bool plain = kind == kTrimNone || copy;                           // the kernel itself does not trim (the copy is trimmed already)
    if (g.fold) {               // at most 4 channels: their own kernel, or 4-channel padded copy, pixel-folded, gather kernel
        pl.pad_bytes = (size_t)round_up((int64_t)g.B * g.H * g.W * 4, 256);
        if (forms && !tune.form && !tune.set()) pl.few = few_geom(g, bytes, device_cu_count());
        return pl;
    }
    if (g.Cp != g.C) pl.pad_bytes = (size_t)round_up((int64_t)g.B * g.H * g.W * g.Cp, 256);
    const bool force_gather = tune.path == 1, force_patch = tune.path == 2;
    ConvGeom gk = g;
    pl.copy = copy;
    if (copy) gk.C = g.Cp;                                       // what the kernel sees
    const bool rules = forms && !tune.form && !tune.set();
    if (forms && tune.form) {
        if (tune.form == kTunedRows && (pl.rows = fit_rows(gk, bytes)) != nullptr && !rows_launchable(*pl.rows, gk, bytes)) pl.rows = nullptr;
        if (tune.form == kTunedSplit && (pl.split = fit_split(gk, &pl.pg, &pl.npix)) != nullptr) return pl;
        if (tune.form == kTunedCols) pl.cols = fit_cols(gk, bytes);
        if (tune.form == kTunedWide) pl.wide = pick_wide(gk, bytes, plain, true);
    }
    if (rules) {
        // (up to 256 channels the registers form is ahead of the split form at every size, beyond that behind it:
        // 256 -> 256, 784 pixels 5.3 against 5.7 us; 512 -> 256 7.9 against 6.0)
        pl.rows = pick_rows(gk, bytes, plain);
        if ((!pl.rows || g.K > 256) && (pl.split = pick_split(gk, &pl.pg, &pl.npix)) != nullptr) return pl;
        pl.wide = pick_wide(gk, bytes, plain);
        pl.cols = pick_cols(gk, bytes, copy ? kTrimNone : kind, pl.rows != nullptr, pl.wide != nullptr);
    }
    // (units of four blocks and the sparse form's result rows leave LDS for one workgroup per CU, where narrow layers with more tiles
    // than CUs want two: 72 -> 16, expanded to four blocks, 401408 pixels 63 against 54 us in units of two)
    const int max_unit = !forms && g.N <= 64 && (g.M + kPatchTM - 1) / kPatchTM > device_cu_count() ? 2 : 4;
    if (!force_gather && (force_patch || !prefer_gather(g)) && plan_patch(gk, max_unit, &pl.pg, &pl.npix, &pl.ac, &pl.cbs)) {
        pl.variant = pick_patch(g, tune, pl.ac, pl.cbs, pl.npix, force_patch, &pl.ws);
        pl.patch = pl.variant != nullptr;
    }
    if (rules) {
        pl.block = pick_block(gk, bytes, plain, !pl.patch, &pl.pg, &pl.npix);
        pl.block = pick_block_square(gk, bytes, plain, pl.block, pl.patch ? pl.variant->tn : 0, &pl.pg, &pl.npix);
    }
    else if (forms && tune.form == kTunedBlock)
        for (const BlockVariant& v : kBlockVariants)
            if ((pl.block = fit_block(gk, bytes, v, &pl.pg, &pl.npix)) != nullptr) break;
    return pl;
}

// Vector instructions that trim 16 bytes (kTrimFloor by its timings: it has 32).
int trim_instructions(TrimKind kind) {
    static const int instructions[kTrimKinds] = {0, 40, 48, 64, 68, 108, 64, 76};
    return instructions[kind];
}

// What trimming while staging adds to a tile kernel, against the copy: the trim's instructions for the patch beyond those that the taps'
// matrix instructions cover, tile after tile on the busiest CU, and a launch and the tensor written and read once more (1/32 ns and
// 1.9 us + 0.25 ns per KB; 1.4 to 2.2 us are as good).  4500 timed layers of up to 2800 channels, trims with rounding: 0.65 % behind the better of the two in the mean, 4.7 %
// of them more than 5 % (0.67 at worst); all trimmed in place 0.41 x at worst (15 x 15 x 1396 -> 96 1x7/2, seven images, three-bit windows, 38
// against 86 us; 7 x 7 x 2148 -> 349 1x7/2, sixteen, 57 against 112: few tiles, each a patch of its own, leave the trim to a few CUs).
bool staging_outlasts_copy(const ConvGeom& g, const ConvPlan& pl, TrimKind kind) {
    const int64_t tn = pl.variant->tn, tiles = (g.M + kPatchTM - 1) / kPatchTM * ((g.N + tn - 1) / tn), cus = device_cu_count();
    const int64_t beyond = (int64_t)pl.npix * trim_instructions(kind) - (int64_t)34 * g.KH * g.KW * (tn < 128 ? tn : 128);
    return (tiles + cus - 1) / cus * (g.Cq / kStepK) * beyond > 60000 + (int64_t)g.x_bytes / 125;
}

// Channel counts that are no multiple of four are contracted from a channel-padded copy, trimmed as it is written.  The others are
// read where they are: a pixel's 16-byte words then start on any four-byte border, which is all a load asks for; the last one runs
// into the next pixel (or past the tensor, where it reads 0) and meets weights that are 0 there; pairs stay inside the pixel.
// 670 drawn layers 1.28 x faster than from the copy (38851 x 188 -> 96 13 -> 6 us; 65536 x 516 -> 256 38 -> 28; 244 -> 256 3x3, 50176
// pixels 45 -> 39), but for the few whose kernel would trim the same bytes over and over, which keep the copy: several taps in the
// gather kernel (5x5 on 69 x 69 x 264 52 against 97 us), 128-pixel tiles of long 1x1 reductions for less than half the CUs
// (2978 x 4312 -> 304 29 against 39), tile kernels whose staging is the longer side (above), and, the trims with the most arithmetic
// (windows of two or three bits with rounding, 17 and 27 instructions for four bytes), five column tiles of the eight-wavefront form (without
// pairs 0.98 as bytes, 1.02) and long reductions of the split form, which stages all of its patch before the first product (154 x 3364 -> 656 10.6 against
// 12.4).  (Tile kernels that stage more than five bytes for one of x kept it as well under those trims: 1400 such layers are 1.09 x faster in place.)
// 1x1 layers trim x once per column tile, which the products of that tile hide in part (`beyond`).  4400 timed layers of 520 to 4600 channels under the
// trims with rounding, in place against the copy, by (instructions - 32) x columns: bytes on the gather kernel 1.0-1.06 x up to 108, 0.95-1.0 x from
// 128 on, 0.7-0.93 x from 176 on; eight wavefronts 1.05-1.1 x up to 176, even from 200 to 264 (rounding with pairs at 220 and 228
// 0.98-1.03, without them at 224 0.99-1.03), 0.92-0.96 x at 288, 0.79-0.91 x from 380 on.
// The weights-in-registers form trims x once per share of 256 or 512 outputs and beside the products: in place 1.5 x faster than from the copy (22710 timed
// layers, 3119 x 776 -> 640 among them; 0.1 % below 0.95 x), but for four-byte results under two- and three-bit windows with rounding and pairs, where
// shares x tenths of a round from 700 on, from 400 with more than 768 channels, are 0.75-1.0 x.
ConvPlan make_plan(const ConvGeom& g, const Tuning& tune, bool forms = true, bool bytes = false, TrimKind kind = kTrimFloor) {
    const bool pads = !g.fold && g.Cp != g.C, trims = kind != kTrimNone;
    if (!pads || g.C % 4 == 0) {
        const ConvPlan pl = make_plan_of(g, tune, forms, bytes, kind, false);
        if (!pads || !trims) return pl;
        const bool gather = !pl.cols && !pl.wide && !pl.split && !pl.block && !pl.rows && !pl.patch;
        const int64_t tiles_m = (g.M + 127) / 128;
        const bool costly = kind == kTrimRound || kind == kTrimRoundPairWide;
        const int beyond = trim_instructions(kind) - 32;         // what the products of one column tile leave uncovered
        bool once = gather && (g.KH * g.KW > 1 || beyond * ((g.N + 255) / 256) > 128);
        if (pl.split && !tune.form) once = costly ? g.K >= 1800 : kind == kTrimRoundPair4 && g.K >= 8000;
        if (pl.cols && !tune.form) {
            const ColsSplit split(*pl.cols, g);
            once = kind == kTrimRoundPairWide && !bytes && !split.two && split.shares * split.tenths >= (pl.cols->steps == 24 ? 700 : 400);
        }
        if (pl.wide && !pl.cols && !tune.form) {
            once = tiles_m * ((g.N + 255) / 256) * 2 < device_cu_count();
            const int columns = (g.N + pl.wide->tn - 1) / pl.wide->tn;
            once = once || (costly && columns >= 5) || beyond * columns > (kind == kTrimRoundPair4 || kind == kTrimRoundPairWide ? 215 : 255);
        }
        if (pl.patch && !pl.cols && !pl.wide && !pl.split && !pl.block && !pl.rows) {
            once = staging_outlasts_copy(g, pl, kind);
        }
        if (!once) return pl;
    }
    return make_plan_of(g, tune, forms, bytes, kind, true);
}

// 2:4 pruned weights run on the sparse matrix instruction when the layer's plan is the wave-specialised
// input-patch kernel and the trim looks at one activation at a time (with pairing on, the problem is the expanded
// one and `kind` is the plain one; with it off the staging wavefronts trim as in the dense form).
bool sparse_plan(const ConvPlan& pl, TrimKind kind) {
    const bool single = kind == kTrimNone || kind == kTrimFloor || kind == kTrimRound || kind == kTrimRound4;
    return pl.patch && pl.ws && pl.variant->fn_sp && single;
}

// The plan of a layer with 2:4 pruned weights.  Where the rules of dense layers pick a form made for the layer's shape, the decompressed
// weights run there (`*dense`): the tile kernel's sparse instruction halves the matrix instructions, which is not what those layers
// wait for.  With vSPARQ off (the layer itself) that is every form, small workgroups only where the layer would otherwise go to the
// gather kernel (224 -> 64 3x3, 538103 pixels 287 -> 163 us; where the sparse instruction applies they are behind: 64 -> 96 3x3, 1280448
// pixels 154 against 163): 512 -> 45 3x3, 600 pixels 16.0 -> 6.8, 496 -> 129 3x3/2, 512 pixels 28 -> 10.  With vSPARQ on (g is the expanded layer,
// taps x channels of the layer itself: k) it costs the expansion an extra launch, and is the split form from k = 2048 on (512 -> 420
// 1x7, 361 pixels 44 -> 13 us; 384 -> 229 3x3, 250 pixels 39 -> 13; shorter reductions gain 1.1-1.9 x too, but stay where the expansion
// is made while staging, as that kernel's tests ask for) and small workgroups in place of the gather kernel.  1x1 layers keep to
// the tile kernels (192 -> 96, 699328 pixels 304 against 308 with their activations in registers).
ConvPlan make_sparse_plan(const ConvGeom& g, const Tuning& tune, bool expanded, int64_t k, TrimKind kind, bool* dense) {
    *dense = g.fold || g.Cq % kStepK != 0;                   // taps that are not step-aligned: no operands for the sparse instruction
    if (*dense) return make_plan(g, tune, true, false, kind);
    const ConvPlan base = make_plan(g, tune, false, false, kind);
    if (tune.form || tune.set()) return base;
    const ConvPlan pl = make_plan(g, tune, true, false, kind);
    const bool sparse = sparse_plan(base, kind);
    if (expanded) *dense = pl.split ? k >= 2048 : pl.block && !base.patch;
    else *dense = pl.split || pl.wide || (pl.block ? !sparse : pl.rows && rows_launchable(*pl.rows, g, false));
    return *dense ? pl : base;
}

}  // namespace

extern "C" sparq_status sparq_set_tuning(const char* spec) {
    Tuning t;
    const char* p = spec ? spec : "";
    while (*p) {
        const char* end = strchr(p, ',');
        const size_t len = end ? (size_t)(end - p) : strlen(p);
        char item[48];
        if (len == 0 || len >= sizeof(item)) return SPARQ_EINVAL;
        memcpy(item, p, len);
        item[len] = 0;
        char* eq = strchr(item, '=');
        if (!eq) return SPARQ_EINVAL;
        *eq = 0;
        const char* key = item;
        const char* val = eq + 1;
        if (!strcmp(key, "path")) {
            if (!strcmp(val, "gather")) t.path = 1;
            else if (!strcmp(val, "patch")) t.path = 2;
            else return SPARQ_EINVAL;
        } else if (!strcmp(key, "tile")) {
            if (strcmp(val, "128x128") && strcmp(val, "128x256") && strcmp(val, "128x512")) return SPARQ_EINVAL;
            strcpy(t.tile, val);
        } else if (!strcmp(key, "patch_tn")) {
            t.patch_tn = atoi(val);
            if (t.patch_tn != 64 && t.patch_tn != 128 && t.patch_tn != 256) return SPARQ_EINVAL;
        } else if (!strcmp(key, "patch_ws")) {
            if (strcmp(val, "0") && strcmp(val, "1")) return SPARQ_EINVAL;
            t.patch_ws = val[0] - '0';
        } else if (!strcmp(key, "form")) {
            if (!strcmp(val, "split")) t.form = kTunedSplit;
            else if (!strcmp(val, "rows")) t.form = kTunedRows;
            else if (!strcmp(val, "cols")) t.form = kTunedCols;
            else if (!strcmp(val, "wide")) t.form = kTunedWide;
            else if (!strcmp(val, "block")) t.form = kTunedBlock;
            else return SPARQ_EINVAL;
        } else {
            return SPARQ_EINVAL;
        }
        p += len + (end ? 1 : 0);
    }
    std::lock_guard<std::mutex> lock(g_tuning_mu);
    g_tuning = t;
    return SPARQ_OK;
}

extern "C" size_t sparq_workspace_bytes(const sparq_conv_desc* desc, const sparq_mode* mode) {
    ConvGeom g;
    if (!conv_geom(desc, &g) || !mode_valid(mode)) return 0;
    return make_plan(g, current_tuning()).pad_bytes;
}

namespace {
// Which of the plan's forms is launched, in the order conv_launch tries them.
enum PlanForm { kFormFew, kFormCols, kFormWide, kFormSplit, kFormBlock, kFormRows, kFormPatch, kFormGather };
PlanForm plan_form(const ConvGeom& g, const ConvPlan& pl, bool bytes) {
    if (pl.few.steps) return kFormFew;
    if (pl.cols) return kFormCols;
    if (pl.wide) return kFormWide;
    if (pl.split) return kFormSplit;
    if (pl.block) return kFormBlock;
    if (pl.rows && rows_launchable(*pl.rows, g, bytes)) return kFormRows;
    return pl.patch ? kFormPatch : kFormGather;
}
const char* const kFormKernels[] = {"conv_few_kernel", "conv_cols_kernel", "conv_wide_kernel", "conv_split_kernel", "conv_block_kernel", "conv_rows_kernel", "conv_patch_kernel", "conv_gemm_kernel"};

const char* gather_tile_name(const ConvGeom& g, const Tuning& tune, bool bytes) {
    ConvGeom gt = g.fold ? folded_view(g) : g;
    gt.Np = g.Np;
    const TileLauncher fn = pick_tile(gt, tune, bytes);
    for (const TileEntry& t : kTiles)
        if (t.fn == fn) return t.name;
    return "?";
}

// The line starts with the kernel family and the form, then names the kernel itself; `plan`: of a 2:4 layer (which has no byte
// results), else the rules'.
sparq_status plan_text(const sparq_conv_desc* desc, const sparq_mode* mode, char* text, size_t text_bytes, const ConvPlan* plan, bool u8_too) {
    ConvGeom g;
    if (!text || text_bytes == 0 || !conv_geom(desc, &g) || !mode_valid(mode)) return SPARQ_EINVAL;
    const Tuning tune = current_tuning();
    const TrimKind kind = trim_kind(mode);
    const ConvPlan pl = plan ? *plan : make_plan(g, tune, true, false, kind);
    const PlanForm form = plan_form(g, pl, false);
    const char* copy = pl.pad_bytes && form != kFormFew && (g.fold || pl.copy) ? " padded_copy" : "";
    char u8[64] = "";
    if (u8_too) {
        const ConvPlan p8 = make_plan(g, tune, true, true, kind);
        const PlanForm f8 = plan_form(g, p8, true);
        const char* tile = f8 == kFormWide ? p8.wide->name : f8 == kFormSplit ? p8.split->name : f8 == kFormGather ? gather_tile_name(g, tune, true) : nullptr;
        const int run = f8 == kFormRows ? p8.rows->held_run(g.M, g.N, true) : 0;
        if (run) snprintf(u8, sizeof(u8), " u8_kernel=%s u8_weights_in_lds=%d", kFormKernels[f8], run);
        else snprintf(u8, sizeof(u8), " u8_kernel=%s%s%s", kFormKernels[f8], tile ? ":" : "", tile ? tile : "");
    }
    char line[160];
    switch (form) {
        case kFormFew: snprintf(line, sizeof(line), "conv_patch_kernel few_channels tile=%dx%d", pl.few.tm, kFewTN); break;
        case kFormSplit: snprintf(line, sizeof(line), "conv_patch_kernel split_reduction tile=%s patch_pixels=%d", pl.split->name, pl.npix); break;
        case kFormBlock: snprintf(line, sizeof(line), "conv_patch_kernel small_workgroups tile=%s patch_pixels=%d", pl.block->name, pl.npix); break;
        case kFormCols: snprintf(line, sizeof(line), "conv_patch_kernel weights_in_registers channels=%s", pl.cols->name); break;
        case kFormWide: snprintf(line, sizeof(line), "conv_gemm_kernel tile=%s eight_wavefronts", pl.wide->name); break;
        case kFormRows: snprintf(line, sizeof(line), "conv_patch_kernel in_registers channels=%s%s", pl.rows->name, pl.rows->held_run(g.M, g.N, false) ? " weights_in_lds" : ""); break;
        case kFormPatch:
            snprintf(line, sizeof(line), "conv_patch_kernel tile=128x%d chunks=%d unit_channels=%d patch_pixels=%d%s", pl.variant->tn, pl.ac,
                     64 * pl.cbs, pl.npix, pl.ws ? " wave_specialised" : "");
            break;
        case kFormGather: snprintf(line, sizeof(line), "conv_gemm_kernel tile=%s", gather_tile_name(g, tune, false)); break;
    }
    snprintf(text, text_bytes, "%s%s%s kernel=%s%s", line, copy, g.fold ? " pixel_folded" : "", kFormKernels[form], u8);
    return SPARQ_OK;
}
}  // namespace

extern "C" sparq_status sparq_conv_plan(const sparq_conv_desc* desc, const sparq_mode* mode, char* text, size_t text_bytes) {
    return plan_text(desc, mode, text, text_bytes, nullptr, true);
}

namespace {

// The gather kernel splits an output row number into (image, oy, ox) once per lane and tile with two divisions by
// numbers fixed per launch.
void set_row_division(GemmParams& p) {
    p.div_wo = make_fastdiv((uint32_t)p.Wo);
    p.div_ho = make_fastdiv((uint32_t)p.Ho);
    p.rows_fit_31 = p.M < (1ll << 31) ? 1 : 0;
}

// Both convolution entry points: acc / out (with scale) as in sparq_conv_gemm, or y (with scale holding the
// requantisation factors) as in sparq_conv_gemm_u8.
// sp: the weights as operands of the sparse matrix instruction as well (2:4 pruned layers); used when the plan is
// the wave-specialised input-patch kernel, ignored otherwise.
// expand_mode: desc is the expanded layer (blocked order) but x is the tensor itself, with x_channels channels; the
// sparse kernel expands it under that mode.  Where that kernel does not apply the call returns SPARQ_EUNSUPPORTED.
// plan: the layer's (make_sparse_plan); vals null: the plan is a dense kernel's, the operands are not looked at.
struct SparseOperand { const uint8_t* vals; const uint32_t* pos; const ConvPlan* plan = nullptr; const sparq_mode* expand_mode = nullptr; int x_channels = 0; };
sparq_status conv_launch(const uint8_t* x, const void* packed_w, const sparq_conv_desc* desc, const sparq_mode* mode,
                         int32_t* acc, const float* scale, float* out, uint8_t* y, const sparq_mode* out_mode,
                         void* workspace, size_t workspace_bytes, void* stream, const SparseOperand* sp = nullptr) {
    ConvGeom g;
    if (!x || !packed_w || !conv_geom(desc, &g) || !mode_valid(mode)) return SPARQ_EINVAL;
    if (!acc && !out && !y) return SPARQ_EINVAL;
    if ((out || y) && !scale) return SPARQ_EINVAL;
    // y trimmed for the next layer: in the epilogue when that layer's mode is this layer's own and the kernel
    // packs the bytes (N a multiple of 4, not a plain 8-bit layer); otherwise one in-place
    // pass of the standalone trim over y afterwards.  Either way y = trim(requantised result), pairs (2j, 2j+1) of a row.
    const bool trim_y = y && out_mode && out_mode->window_bits != 8;
    if (trim_y && !mode_valid(out_mode)) return SPARQ_EINVAL;
    const bool same_mode = trim_y && out_mode->window_bits == mode->window_bits && out_mode->shift_mask == mode->shift_mask &&
                           out_mode->round_nearest == mode->round_nearest && out_mode->pair == mode->pair;
    bool fused_trim = same_mode && g.N % 4 == 0;
    if (!aligned(x, 16) || !aligned(packed_w, 256) || (acc && !aligned(acc, 16)) || (out && !aligned(out, 16)) ||
        (y && !aligned(y, 16)) || (scale && !aligned(scale, 4)))
        return SPARQ_EINVAL;
    hipStream_t s = static_cast<hipStream_t>(stream);
    const Tuning tune = current_tuning();
    const ConvPlan pl = sp ? *sp->plan : make_plan(g, tune, true, y != nullptr, trim_kind(mode));
    if (sp && !sp->vals) sp = nullptr;
    const size_t need = pl.pad_bytes;
    if (need) {
        if (!workspace || !aligned(workspace, 256)) return SPARQ_EINVAL;
        if (workspace_bytes < need) return SPARQ_EWORKSPACE;
    }

    const uint8_t* xin = x;
    TrimKind kind = trim_kind(mode);
    size_t x_bytes = g.x_bytes;
    if (g.fold) {
        if (pl.few.steps) {                     // (the workspace is asked for all the same: which form a call takes is not its caller's business)
            if ((size_t)g.B * g.H * g.W * 4 >= kInvalidOffset) return SPARQ_EUNSUPPORTED;
            FewParams q{};
            q.x = x;
            q.wpk = static_cast<const uint8_t*>(packed_w) + g.w_off;
            q.colsum = static_cast<const int32_t*>(packed_w);
            q.acc = acc; q.scale = scale; q.out = out; q.out_u8 = y;
            q.x_bytes = (uint32_t)g.x_bytes;
            q.w_bytes = (uint32_t)((size_t)g.Kp * g.Np);
            q.M = (int)g.M; q.N = g.N; q.Np = g.Np;
            q.B = g.B; q.H = g.H; q.W = g.W; q.Wo = g.Wo; q.Ho = g.Ho; q.KH = g.KH; q.sh = g.sh; q.sw = g.sw; q.ph = g.ph;
            q.Hv = g.H + 2 * g.ph;
            q.tm = pl.few.tm; q.tiles = (int)((g.M + q.tm - 1) / q.tm); q.patch_bytes = pl.few.patch_bytes;
            q.taps_row = pl.few.taps_row; q.taps_pitch = g.fold_kw; q.group0 = g.fold_kw_min; q.steps = pl.few.steps;
            q.kind = kind;
            q.div_wo = make_fastdiv((uint32_t)g.Wo);
            q.div_ho = make_fastdiv((uint32_t)g.Ho);
            q.div_hv = make_fastdiv((uint32_t)q.Hv);
            q.luts = make_luts(mode->window_bits, mode->shift_mask);
            static constexpr sparq_status (*kLaunch[])(const FewParams&, hipStream_t) = {launch_few_c1, launch_few_c2, launch_few_c3, launch_few_c4};
            const sparq_status st = kLaunch[g.C - 1](q, s);
            if (st != SPARQ_OK || !trim_y) return st;
            return sparq_trim(y, y, g.M, g.N, out_mode, stream);
        }
        // A first-layer shape (C <= 4): trim into a copy with 4 channels per pixel, then contract the
        // pixel-folded problem (16-channel super-pixels, fold_p * N output channels) with trimming off.
        const ConvGeom f = folded_view(g);
        if (f.x_bytes >= kInvalidOffset) return SPARQ_EUNSUPPORTED;
        const sparq_status st = launch_trim_pad(x, static_cast<uint8_t*>(workspace), (int64_t)g.B * g.H * g.W, g.C, 4, mode, s);
        if (st != SPARQ_OK) return st;
        GemmParams p{};
        p.x = static_cast<const uint8_t*>(workspace);
        p.wpk = static_cast<const uint8_t*>(packed_w) + g.w_off;
        p.colsum = static_cast<const int32_t*>(packed_w);
        p.acc = acc; p.scale = scale; p.out = out; p.out_u8 = y;
        p.M = f.M;
        p.x_bytes = (uint32_t)f.x_bytes;
        p.N = f.N; p.Np = g.Np; p.Kk = f.Kk; p.nkb = g.Kp / kStepK; p.scale_n = g.N;
        p.H = f.H; p.W = f.W; p.C = 16; p.Cq = 16; p.Ho = f.Ho; p.Wo = f.Wo; p.KH = f.KH; p.KW = f.KW;
        p.sh = f.sh; p.sw = 1; p.ph = f.ph; p.pw = f.pw;
        p.rcp_c = 1.0f / 16.0f;
        p.rcp_kw = 1.0f / (float)f.KW;
        set_row_division(p);
        p.luts = make_luts(8, 1);
        ConvGeom ft = f;
        ft.Np = g.Np;
        const sparq_status stf = pick_tile(ft, tune, y != nullptr)(kTrimNone, p, s);
        if (stf != SPARQ_OK || !trim_y) return stf;
        return sparq_trim(y, y, g.M, g.N, out_mode, stream);
    }
    if (g.Cp != g.C && (size_t)g.B * g.H * g.W * g.Cp >= kInvalidOffset) return SPARQ_EUNSUPPORTED;
    if (pl.copy) {
        // Trim into a channel-padded copy
        // first (pairs stay inside the row; padded channels are zeros with zero weights),
        // then contract the copy without further trimming.
        x_bytes = (size_t)g.B * g.H * g.W * g.Cp;
        const sparq_status st = launch_trim_pad(x, static_cast<uint8_t*>(workspace), (int64_t)g.B * g.H * g.W, g.C,
                                                g.Cp, mode, s);
        if (st != SPARQ_OK) return st;
        xin = static_cast<const uint8_t*>(workspace);
        kind = kTrimNone;
        fused_trim = false;                     // the kernel runs with trimming off
    }
    const int xc = pl.copy ? g.Cp : g.C;         // bytes from pixel to pixel
    if (x_bytes >= kInvalidOffset) return SPARQ_EUNSUPPORTED;
    const auto finish = [&](sparq_status st, bool fused) {
        if (st != SPARQ_OK || !trim_y || fused) return st;
        return sparq_trim(y, y, g.M, g.N, out_mode, stream);
    };

    // An input that arrives trimmed (plain 8 bits) with an output to be trimmed for the next layer: the variants of the
    // OUTPUT mode, told not to trim their input, do it in their epilogue (the two forms below; the third says why not always).
    const bool out_only = trim_y && !fused_trim && kind == kTrimNone && mode->window_bits == 8 && g.N % 4 == 0 && !pl.copy;
    const sparq_mode* kmode = out_only ? out_mode : mode;
    const auto fill = [&](auto& q) {
        q.x = xin;
        q.wpk = static_cast<const uint8_t*>(packed_w) + g.w_off;
        q.colsum = static_cast<const int32_t*>(packed_w);
        q.acc = acc; q.scale = scale; q.out = out; q.out_u8 = y;
        q.x_bytes = (uint32_t)x_bytes;
        q.w_bytes = (uint32_t)((size_t)g.Kp * g.Np);
        q.N = g.N; q.Np = g.Np; q.C = xc;
        q.luts = make_luts(kmode->window_bits, kmode->shift_mask);
        q.trim_in = out_only ? 0 : 1;
        q.trim_out = fused_trim || out_only ? 1 : 0;
    };
    const TrimKind okind = out_only ? trim_kind(out_mode) : kind;

    // 1x1 layers with the weights in registers.
    const auto fill_rows = [&](RowsParams& q) {
        fill(q);
        q.M = (int)g.M;
        q.steps = g.Cq / 32;
        q.g = make_patch_geom(g.B, g.H, g.W, 1, 1, g.sh, g.sw, 0, 0);
    };
    if (pl.cols) {
        RowsParams q{};
        fill_rows(q);
        const sparq_status st = pl.cols->fn(okind, q, s);
        if (st != SPARQ_EUNSUPPORTED) return finish(st, q.trim_out != 0);
    }

    // 1x1 layers with a long reduction: eight wavefronts per tile.  (They always trim their input: a call
    // with only its output to be trimmed goes to the forms below.)
    if (pl.wide && !out_only) {
        WideParams q{};
        fill(q);
        q.M = (int)g.M;
        q.steps = g.Cq / kStepK;
        q.g = make_patch_geom(g.B, g.H, g.W, 1, 1, g.sh, g.sw, 0, 0);
        const sparq_status st = pl.wide->fn(okind, q, s);
        if (st != SPARQ_EUNSUPPORTED) return finish(st, q.trim_out != 0);
    }

    // Small layers: the reduction split over a workgroup's wavefronts.
    if (pl.split) {
        SplitParams q{};
        fill(q);
        q.planes = g.Cq / kChunk;
        q.steps_tap = g.Cq / 32;
        q.steps = g.KH * g.KW * q.steps_tap;
        q.div_planes = make_fastdiv((uint32_t)q.planes);
        q.div_steps_tap = make_fastdiv((uint32_t)q.steps_tap);
        q.div_kw = make_fastdiv((uint32_t)g.KW);
        q.g = pl.pg;
        q.div_wo = make_fastdiv((uint32_t)q.g.Wo);
        q.div_ho = make_fastdiv((uint32_t)q.g.Ho);
        q.div_hv = make_fastdiv((uint32_t)q.g.Hv);
        return finish(pl.split->fn(okind, q, pl.npix, s), q.trim_out != 0);
    }

    // Multi-tap layers as many small workgroups.
    if (pl.block) {
        BlockParams q{};
        fill(q);
        q.ncb = g.Cq / kStepK;
        q.g = pl.pg;
        return finish(pl.block->fn(okind, q, pl.npix, s), q.trim_out != 0);
    }

    // 1x1 layers with a short reduction: activations in registers.
    if (pl.rows) {
        RowsParams q{};
        fill_rows(q);
        const sparq_status st = pl.rows->fn(okind, q, s);
        if (st != SPARQ_EUNSUPPORTED) return finish(st, q.trim_out != 0);
    }

    // Preferred: the input-patch kernel (activations loaded and trimmed once per tile and channel block).
    if (pl.patch) {
        PatchParams q{};
        q.x = xin;
        q.wpk = static_cast<const uint8_t*>(packed_w) + g.w_off;
        q.colsum = static_cast<const int32_t*>(packed_w);
        q.acc = acc; q.scale = scale; q.out = out; q.out_u8 = y; q.trim_out = fused_trim ? 1 : 0;
        q.x_bytes = (uint32_t)x_bytes;
        q.w_bytes = (uint32_t)((size_t)g.Kp * g.Np);
        q.N = g.N; q.Np = g.Np; q.C = xc;
        q.ksteps_tap = g.Cq / kStepK;
        q.ncb = q.ksteps_tap / pl.cbs;
        q.nsteps = g.KH * g.KW * pl.cbs;
        q.g = pl.pg;
        q.luts = make_luts(mode->window_bits, mode->shift_mask);
        q.trim_in = 1;
        TrimKind pkind = kind;
        bool pfused = fused_trim;
        // An input that arrives trimmed (mode: plain 8 bits) with an output to be trimmed for the next layer:
        // the wave-specialised kernel of the OUTPUT mode, told not to trim its input, trims y in its epilogue.
        // (A layer that would take the plain form takes the wave-specialised one here: that costs a few per cent,
        // the separate trim pass over y it avoids costs more.)
        bool use_ws = pl.ws;
        if (trim_y && !fused_trim && kind == kTrimNone && mode->window_bits == 8 && g.N % 4 == 0 &&
            !pl.copy && pl.variant->fn_ws) {
            use_ws = true;
            pkind = trim_kind(out_mode);
            q.luts = make_luts(out_mode->window_bits, out_mode->shift_mask);
            q.trim_in = 0;
            pfused = true;
        }
        q.trim_out = pfused ? 1 : 0;
        if (sp && sparse_plan(pl, kind) && !y) {
            PatchParams qs = q;
            qs.wpk = sp->vals;
            qs.widx = sp->pos;
            qs.w_bytes = (uint32_t)((size_t)g.Kp * g.Np / 2);
            TrimKind skind = kind;
            if (sp->expand_mode) {
                skind = trim_kind(sp->expand_mode);
                qs.luts = make_luts(sp->expand_mode->window_bits, sp->expand_mode->shift_mask);
                qs.C = sp->x_channels;
                qs.x_bytes = (uint32_t)((size_t)g.B * g.H * g.W * sp->x_channels);
            }
            const sparq_status st = pl.variant->fn_sp(skind, qs, pl.npix, s);
            if (st != SPARQ_EUNSUPPORTED || sp->expand_mode) return st;
        }
        if (!(sp && sp->expand_mode)) {
            const PatchLauncher fn = use_ws ? pl.variant->fn_ws : pl.variant->fn;
            const sparq_status st = fn(pkind, q, pl.npix, s);
            if (st != SPARQ_EUNSUPPORTED) return finish(st, pfused);
        }
    }

    if (sp && sp->expand_mode) return SPARQ_EUNSUPPORTED;
    GemmParams p{};
    p.x = xin;
    p.wpk = static_cast<const uint8_t*>(packed_w) + g.w_off;
    p.colsum = static_cast<const int32_t*>(packed_w);
    p.acc = acc;
    p.scale = scale;
    p.out = out;
    p.out_u8 = y;
    p.trim_out = fused_trim ? 1 : 0;
    p.M = g.M;
    p.x_bytes = (uint32_t)x_bytes;
    p.N = g.N; p.Np = g.Np; p.Kk = g.Kk; p.nkb = g.Kp / kStepK; p.scale_n = g.N;
    p.H = g.H; p.W = g.W; p.C = xc; p.Cq = g.Cq; p.Ho = g.Ho; p.Wo = g.Wo; p.KH = g.KH; p.KW = g.KW;
    p.sh = g.sh; p.sw = g.sw; p.ph = g.ph; p.pw = g.pw;
    p.rcp_c = 1.0f / (float)g.Cq;
    p.rcp_kw = 1.0f / (float)g.KW;
    set_row_division(p);
    p.luts = make_luts(mode->window_bits, mode->shift_mask);

    return finish(pick_tile(g, tune, y != nullptr)(kind, p, s), fused_trim);
}

}  // namespace

extern "C" sparq_status sparq_conv_gemm(const uint8_t* x, const void* packed_w, const sparq_conv_desc* desc,
                                        const sparq_mode* mode, int32_t* acc, const float* scale, float* out,
                                        void* workspace, size_t workspace_bytes, void* stream) {
    if (!acc && !out) return SPARQ_EINVAL;
    return conv_launch(x, packed_w, desc, mode, acc, scale, out, nullptr, nullptr, workspace, workspace_bytes, stream);
}

// ---- the same convolution for callers that cannot allocate: the scratch lives in the library's own image ----
// One array per device (every GPU the library's code object is loaded on holds its own copy at its own
// address, until the process ends).  In host code the array's name is only a handle for the symbol lookup:
// the device address comes from hipGetSymbolAddress, once per device, and is what the kernels are given.
static __device__ __align__(256) unsigned char scratch[SPARQ_STATIC_WORKSPACE_BYTES];

namespace {
sparq_status static_scratch_address(void** ptr) {
    static void* addr[kMaxDevices] = {};
    static std::mutex mu;
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0) return SPARQ_ELAUNCH;
    std::lock_guard<std::mutex> lock(mu);
    if (dev < kMaxDevices && addr[dev]) {
        *ptr = addr[dev];
        return SPARQ_OK;
    }
    void* a = nullptr;
    if (hipGetSymbolAddress(&a, HIP_SYMBOL(scratch)) != hipSuccess || !a) {
        (void)hipGetLastError();
        return SPARQ_ELAUNCH;
    }
    if (dev < kMaxDevices) addr[dev] = a;       // ordinals past the table look the address up on every call
    *ptr = a;
    return SPARQ_OK;
}
}  // namespace

extern "C" sparq_status sparq_conv_gemm_static_ws(const uint8_t* x, const void* packed_w, const sparq_conv_desc* desc,
                                                  const sparq_mode* mode, int32_t* acc, const float* scale, float* out,
                                                  void* stream) {
    if (!acc && !out) return SPARQ_EINVAL;
    ConvGeom g;
    if (!conv_geom(desc, &g) || !mode_valid(mode)) return SPARQ_EINVAL;
    const size_t need = make_plan(g, current_tuning()).pad_bytes;
    if (need > (size_t)SPARQ_STATIC_WORKSPACE_BYTES) return SPARQ_EWORKSPACE;
    void* ws = nullptr;
    if (need) {
        const sparq_status st = static_scratch_address(&ws);
        if (st != SPARQ_OK) return st;
    }
    // Every byte of the scratch a call reads it has written itself first (the padded copy is written whole by the
    // trim pass), so the last call's contents never show.
    return conv_launch(x, packed_w, desc, mode, acc, scale, out, nullptr, nullptr, ws, need, stream);
}

// ---- input in packed storage (Sections 3.1, 5.1, 6): records expanded into the workspace, contracted at 8 bits ----
namespace {
const sparq_mode kPlainMode = {8, 1, 0, 0};
}

extern "C" size_t sparq_conv_packed_workspace_bytes(const sparq_conv_desc* desc, const sparq_mode* mode) {
    ConvGeom g;
    if (!conv_geom(desc, &g) || !mode_valid(mode)) return 0;
    return (size_t)round_up((int64_t)g.x_bytes, 256) + sparq_workspace_bytes(desc, &kPlainMode);
}

extern "C" sparq_status sparq_conv_gemm_packed(const void* packed_x, size_t packed_x_bytes, int32_t group,
                                               const void* packed_w, const sparq_conv_desc* desc, const sparq_mode* mode,
                                               int32_t* acc, const float* scale, float* out, void* workspace,
                                               size_t workspace_bytes, void* stream) {
    ConvGeom g;
    if (!packed_x || !conv_geom(desc, &g) || !mode_valid(mode) || (!acc && !out)) return SPARQ_EINVAL;
    const int64_t pixels = (int64_t)g.B * g.H * g.W;
    const size_t need_packed = sparq_packed_act_bytes(pixels, g.C, mode, group);
    if (need_packed == 0 || !aligned(packed_x, 4)) return SPARQ_EINVAL;
    if (packed_x_bytes < need_packed) return SPARQ_EWORKSPACE;
    if (!workspace || !aligned(workspace, 256)) return SPARQ_EINVAL;
    if (workspace_bytes < sparq_conv_packed_workspace_bytes(desc, mode)) return SPARQ_EWORKSPACE;
    uint8_t* xu = static_cast<uint8_t*>(workspace);
    // Channel counts that are no multiple of four: the records end in zeros, so they unpack straight into the channel-padded tensor (for
    // which the workspace has room) the layer would else be copied to; packed weights, reductions and kernels are the same.  73 drawn
    // layers 1.30 x, none slower (38 x 38 x 315 -> 224 1x1, ten images 17.1 -> 11.6 us; 26 x 26 x 857 -> 544 1x1/2, nine 17.6 -> 12.2).  Multiples of
    // four are read where they are either way (0.97-1.02 x).
    sparq_conv_desc padded = *desc;
    ConvGeom gp;
    padded.C = g.Cp;
    if (!g.fold && g.C % 4 != 0 && conv_geom(&padded, &gp) && !gp.fold && gp.packed_bytes == g.packed_bytes) {
        const sparq_status st = launch_unpack_act(packed_x, xu, pixels, g.Cp, mode, group, static_cast<hipStream_t>(stream));
        if (st != SPARQ_OK) return st;
        return conv_launch(xu, packed_w, &padded, &kPlainMode, acc, scale, out, nullptr, nullptr, nullptr, 0, stream);
    }
    const size_t x_room = (size_t)round_up((int64_t)g.x_bytes, 256);
    const sparq_status st = launch_unpack_act(packed_x, xu, pixels, g.C, mode, group, static_cast<hipStream_t>(stream));
    if (st != SPARQ_OK) return st;
    return conv_launch(xu, packed_w, desc, &kPlainMode, acc, scale, out, nullptr, nullptr, xu + x_room,
                       workspace_bytes - x_room, stream);
}

// ---- 2:4 pruned weights (Section 4, sparse tensor core; Section 5.3): see sparq_sparse24.hip ----
namespace {
// What the entry points accept, and the size of their buffers, is that of a layer with four expanded channels per
// channel (the form this path had first); the contracted layer never needs more than that.
bool sparse24_bound(const sparq_conv_desc* desc, const sparq_mode* mode, sparq_conv_desc* bound, bool* expand) {
    ConvGeom g;
    if (!desc || desc->C % 4 != 0 || !conv_geom(desc, &g) || !mode_valid(mode)) return false;
    *expand = mode->pair && mode->window_bits != 8;
    *bound = *desc;
    if (*expand) {
        if ((int64_t)desc->C * 4 > 0x7FFFFFFF) return false;
        bound->C = desc->C * 4;
    }
    return conv_geom(bound, &g);
}
// The dense problem that is actually contracted: with vSPARQ on, 12 expanded channels per group of four.
bool sparse24_geometry(const sparq_conv_desc* desc, const sparq_mode* mode, sparq_conv_desc* eff, bool* expand) {
    ConvGeom g;
    if (!sparse24_bound(desc, mode, eff, expand) || !conv_geom(eff, &g)) return false;
    if (*expand) eff->C = (int)sparse24_channels(desc->C, desc->KH * desc->KW, g.M);
    return conv_geom(eff, &g);
}
const sparq_mode kNoPairPlain = {8, 1, 0, 0};
// The trim of the contracted layer (a padded copy's pre-pass does it where there is one; single activations either way).
TrimKind sparse24_kind(const ConvGeom& g, const sparq_mode* mode) { return g.fold ? kTrimNone : trim_kind(mode); }

// The staging wavefronts expand what they load where a tile's patch is small beside its taps (each patch pixel is then worked out
// once per channel tile, which the matrix instructions of its taps have to cover) or where there are tiles for every CU, so that the
// expanded tensor would be written to memory and read back.  Elsewhere it is written first.  Of 200 drawn layers of more than 32
// patch pixels per tap: up to 50 of them in units of 64 channels 1.24 x faster than written (59, one slower, 0.94 x; 39 x 39 x 192 ->
// 608 1x7 75 -> 58 us); beyond, from 8192 pixels on 1.36 x (45, none slower; 51 x 51 x 272 -> 128 7x1, 7803 pixels 36 against 39, and
// fewer pixels down to 0.59 x: a strided 7x1 on 196 pixels 37 against 63); 1x1 layers in wider units 1.6 x from there on, 0.6-1.2 x below.
// `pl`: the plan of the expanded layer.
bool expands_while_staging(const sparq_conv_desc& desc, const ConvPlan& pl) {
    return sparse24_blocked(desc.C) && sparse_plan(pl, kTrimNone) && (pl.npix <= (pl.cbs == 1 ? 50 : 32) * desc.KH * desc.KW || pl.pg.M >= 8192);
}

// Layout of the buffer sparq_pack_weights_sparse24 fills: the dense packed tiles of the contracted problem, room
// to decompress into, then the same weights as operands of the sparse matrix instruction (kept bytes, positions)
// when the contracted problem's taps are 64-byte aligned (otherwise those two parts are empty).
struct Sparse24Layout { size_t tiles, dense, vals, pos; bool sparse; };
Sparse24Layout sparse24_layout(const sparq_conv_desc& eff) {
    ConvGeom g;
    conv_geom(&eff, &g);
    Sparse24Layout L;
    L.tiles = (size_t)round_up((int64_t)g.packed_bytes, 256);
    L.dense = (size_t)round_up((int64_t)eff.N * eff.KH * eff.KW * eff.C, 256);
    L.sparse = !g.fold && g.Cq % kStepK == 0;
    L.vals = L.sparse ? (size_t)round_up((int64_t)g.Kp * g.Np / 2, 256) : 0;
    L.pos = L.sparse ? (size_t)round_up((int64_t)g.Kp * g.Np / 8, 256) : 0;
    return L;
}
}  // namespace

extern "C" size_t sparq_sparse24_packed_bytes(const sparq_conv_desc* desc, const sparq_mode* mode) {
    sparq_conv_desc bound;
    bool expand;
    if (!sparse24_bound(desc, mode, &bound, &expand)) return 0;
    const Sparse24Layout L = sparse24_layout(bound);
    return L.tiles + L.dense + L.vals + L.pos;
}

extern "C" sparq_status sparq_pack_weights_sparse24(const int8_t* w_vals, const uint8_t* w_idx, const sparq_conv_desc* desc,
                                                    const sparq_mode* mode, void* packed, size_t packed_bytes, void* stream) {
    sparq_conv_desc eff;
    bool expand;
    if (!w_vals || !w_idx || !packed || !sparse24_geometry(desc, mode, &eff, &expand) || !aligned(packed, 256)) return SPARQ_EINVAL;
    if (packed_bytes < sparq_sparse24_packed_bytes(desc, mode)) return SPARQ_EWORKSPACE;
    const Sparse24Layout L = sparse24_layout(eff);
    int8_t* dense = static_cast<int8_t*>(packed) + L.tiles;
    sparq_status st = launch_sparse24_expand_weights(w_vals, w_idx, dense, (int64_t)desc->N * desc->KH * desc->KW, desc->C, eff.C,
                                                     static_cast<hipStream_t>(stream));
    if (st != SPARQ_OK) return st;
    st = sparq_pack_weights(dense, &eff, packed, L.tiles, stream);
    if (st != SPARQ_OK || !L.sparse) return st;
    ConvGeom g;
    conv_geom(&eff, &g);
    uint8_t* vals = static_cast<uint8_t*>(packed) + L.tiles + L.dense;
    return launch_sparse24_pack_operand(dense, vals, reinterpret_cast<uint32_t*>(vals + L.vals), eff.N, g.Np, eff.KH * eff.KW,
                                        eff.C, g.Cq, static_cast<hipStream_t>(stream));
}

extern "C" size_t sparq_sparse24_workspace_bytes(const sparq_conv_desc* desc, const sparq_mode* mode) {
    sparq_conv_desc bound;
    bool expand;
    if (!sparse24_bound(desc, mode, &bound, &expand)) return 0;
    if (!expand) return sparq_workspace_bytes(desc, mode);
    return (size_t)round_up((int64_t)bound.B * bound.H * bound.W * bound.C, 256) + sparq_workspace_bytes(&bound, &kNoPairPlain);
}

extern "C" sparq_status sparq_conv_gemm_sparse24(const uint8_t* x, const void* packed, const sparq_conv_desc* desc,
                                                 const sparq_mode* mode, int32_t* acc, const float* scale, float* out,
                                                 void* workspace, size_t workspace_bytes, void* stream) {
    sparq_conv_desc eff;
    bool expand;
    if (!x || !packed || (!acc && !out) || !sparse24_geometry(desc, mode, &eff, &expand)) return SPARQ_EINVAL;
    const Sparse24Layout L = sparse24_layout(eff);
    const uint8_t* sp_vals = static_cast<const uint8_t*>(packed) + L.tiles + L.dense;
    ConvGeom ge;
    conv_geom(&eff, &ge);
    const sparq_mode* emode = expand ? &kNoPairPlain : mode;
    bool dense;
    const ConvPlan plan = make_sparse_plan(ge, current_tuning(), expand, (int64_t)desc->KH * desc->KW * desc->C,
                                           sparse24_kind(ge, emode), &dense);
    SparseOperand sp_op;
    sp_op.vals = L.sparse && !dense ? sp_vals : nullptr;
    sp_op.pos = reinterpret_cast<const uint32_t*>(sp_vals + L.vals);
    sp_op.plan = &plan;
    if (!expand)      // nothing depends on the partner: the decompressed weights, the ordinary path
        return conv_launch(x, packed, desc, mode, acc, scale, out, nullptr, nullptr, workspace, workspace_bytes, stream, &sp_op);
    if (!aligned(x, 4) || !workspace || !aligned(workspace, 256)) return SPARQ_EINVAL;
    if (workspace_bytes < sparq_sparse24_workspace_bytes(desc, mode)) return SPARQ_EWORKSPACE;
    const int64_t pixels = (int64_t)desc->B * desc->H * desc->W;
    if (pixels * desc->C * 4 >= (int64_t)kInvalidOffset) return SPARQ_EUNSUPPORTED;
    if (sp_op.vals && aligned(x, 16) && expands_while_staging(*desc, plan)) {
        SparseOperand fused = sp_op;
        fused.expand_mode = mode;
        fused.x_channels = desc->C;
        const sparq_status st = conv_launch(x, packed, &eff, &kNoPairPlain, acc, scale, out, nullptr, nullptr, workspace,
                                            workspace_bytes, stream, &fused);
        if (st != SPARQ_EUNSUPPORTED) return st;
    }
    const size_t x_room = (size_t)round_up(pixels * eff.C, 256);
    uint8_t* xe = static_cast<uint8_t*>(workspace);
    const sparq_status st = launch_sparse24_expand_act(x, xe, pixels, desc->C, eff.C, mode, static_cast<hipStream_t>(stream));
    if (st != SPARQ_OK) return st;
    return conv_launch(xe, packed, &eff, &kNoPairPlain, acc, scale, out, nullptr, nullptr, xe + x_room,
                       workspace_bytes - x_room, stream, &sp_op);
}

extern "C" sparq_status sparq_sparse24_plan(const sparq_conv_desc* desc, const sparq_mode* mode, char* text, size_t text_bytes) {
    sparq_conv_desc eff;
    bool expand;
    if (!text || text_bytes == 0 || !sparse24_geometry(desc, mode, &eff, &expand)) return SPARQ_EINVAL;
    const sparq_mode* m = expand ? &kNoPairPlain : mode;
    ConvGeom g;
    conv_geom(&eff, &g);
    const TrimKind kind = sparse24_kind(g, m);
    bool dense;
    const ConvPlan pl = make_sparse_plan(g, current_tuning(), expand, (int64_t)desc->KH * desc->KW * desc->C, kind, &dense);
    char line[200];
    const sparq_status st = plan_text(&eff, m, line, sizeof(line), &pl, false);
    if (st != SPARQ_OK) return st;
    const bool smfmac = !dense && sparse24_layout(eff).sparse && sparse_plan(pl, kind);
    snprintf(text, text_bytes, "%s%s%s%s", line, expand ? " expanded_x4" : "",
             expand && smfmac && expands_while_staging(*desc, pl) ? " expanded_while_staging" : "", smfmac ? " sparse_mfma" : " dense_mfma");
    return SPARQ_OK;
}

extern "C" sparq_status sparq_conv_gemm_u8(const uint8_t* x, const void* packed_w, const sparq_conv_desc* desc,
                                           const sparq_mode* mode, const float* factor, uint8_t* y,
                                           const sparq_mode* out_mode, void* workspace, size_t workspace_bytes,
                                           void* stream) {
    if (!factor || !y) return SPARQ_EINVAL;
    return conv_launch(x, packed_w, desc, mode, nullptr, factor, nullptr, y, out_mode, workspace, workspace_bytes, stream);
}
