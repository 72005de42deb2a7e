// The workgroup tiles of the matrix kernel of hb_conv2d, hb_down2 and hb_up2: what each one covers, stages and keeps in
// LDS.  Host arithmetic only, also for tests that run without a GPU.
#pragma once
#include <stddef.h>
#include <stdint.h>

#include "hb.h"

namespace hb {

enum T2Mode { kT2Conv, kT2Down, kT2Up };
enum T2Shape { kT2Row, kT2Block, kT2Stack, kT2Flat, kT2FlatPair };   // of a workgroup's waves, see T2Geom
struct T2Tile { T2Shape shape; int nw; };     // of a call; nw: tiles of 16 columns per wave

constexpr size_t kT2LdsOfCu = 160 << 10, kT2LdsGrain = 1280;          // of a compute unit; LDS is given out in these pieces

// workgroups of so much LDS that a compute unit holds
inline size_t t2_resident(size_t lds) { return kT2LdsOfCu / ((lds + kT2LdsGrain - 1) / kT2LdsGrain * kT2LdsGrain); }

// kT2Row: the waves beside each other.  kT2Block and kT2Stack (narrow outputs): two by two, or one
// below the other.  kT2Flat (outputs of few rows): the N index of a product is 8 row pairs x 4 runs of tiles beside each other instead
// of 32 row pairs.  16 x 200000, 3 x 3 / 32 x 32 taps: 14.3 / 45 us with the tall tile, 10.2 / 17 with this one.
// kT2FlatPair: two waves of that kind, where the LDS of four leaves a compute unit a single workgroup.
template <int MODE, int NK, int NW, T2Shape SHAPE>
struct T2Geom {
    static constexpr int kPairs = SHAPE == kT2Flat || SHAPE == kT2FlatPair ? 8 : 32, kBeside = 32 / kPairs;  // row pairs, runs of tiles in N
    static constexpr int kWx = SHAPE == kT2Stack ? 1 : SHAPE == kT2Block || SHAPE == kT2FlatPair ? 2 : 4;   // waves of a workgroup, across ...
    static constexpr int kWy = SHAPE == kT2Stack ? 4 : SHAPE == kT2Block ? 2 : 1;                     // ... and down
    static constexpr int kThreads = 64 * kWx * kWy;
    static constexpr int kOccupancy = MODE == kT2Conv ? (NW > 2 ? 2 : 3) : MODE == kT2Down ? 2 : NK > 1 ? 3 : 4;   // waves per SIMD
    static constexpr int kStride = MODE == kT2Conv ? 2 : MODE == kT2Down ? 4 : 1;   // input rows per n
    static constexpr int kTileStep = MODE == kT2Conv ? 16 : MODE == kT2Down ? 32 : 8;
    static constexpr int kCols = 16 * NW * kBeside * kWx, kRows = 2 * kPairs * kWy;   // output tile
    static constexpr int kChunks = (kTileStep * (NW * kBeside * kWx - 1) + 16 * NK) / 8;      // of 8 staged pixels per row
    static constexpr int kPitch = 8 * (kChunks | 1);
    static constexpr int kPatch = 32 * (16 * NW + 4);                     // floats per wave, see the stores
    // window chunks of a wave: distinct multiples of 8 pixels at which a fragment starts
    static constexpr int kUnit = MODE == kT2Up ? 8 : 16;
    static constexpr int kFrags = (kTileStep * (NW - 1) + 16 * (NK - 1)) / kUnit + 1;
    static constexpr int kMaxSteps = MODE == kT2Conv ? HB_MAX_TAPS_CONV2D + 1 : MODE == kT2Down ? HB_MAX_TAPS_CONV2D + 2 : HB_MAX_TAPS_CONV2D / 2;
    static constexpr int kPieces = ((kStride * (kPairs * kWy - 1) + kMaxSteps) * kChunks + kThreads - 1) / kThreads;   // staged per thread
    // Weight table.  A lane's eight weights start at position 8h - (its column's shift) + kPad, 1 (conv, up) or 2 (down)
    // apart, so a row is kept in kCopies copies of kCopy taps, each shifted by kShift, and every run starts on 8 bytes
    // (down: 16).  Pitches: the lanes served together fall into different banks (conv: blocks of 8 dwords at 0, 40, 16, 56 and, for
    // the row above, 32 further; up: of 4 dwords at 0, 20, 40, 60 plus 16 and 32; down: of 16 at 0, 48, 32, 16).
    // Narrow and flat tiles of hb_down2 with many taps keep two copies on 8-byte starts: 14 KB less, so that a compute unit holds two
    // workgroups (to 32 x 56000, 28 x 28 taps 21.0 -> 16.1 us).  The others are faster with four (by 2 % on average).
    static constexpr int kCopies = MODE == kT2Down && (SHAPE == kT2FlatPair || (SHAPE != kT2Row && NK == 4)) ? 2 : 4, kShift = MODE == kT2Down ? 2 : 1, kPad = MODE == kT2Conv ? 15 : MODE == kT2Down ? 30 : 7;
    static constexpr int kCopy = MODE == kT2Conv ? 80 : MODE == kT2Down ? 96 : 40, kTabRow = kCopies == 2 ? 224 : kCopies * kCopy;
    // Zero rows of the table, above and below the taps: a step reads row s - dy or s - 2 dy.  With two for hb_conv2d as well,
    // and the image's last section as long as the others, a compute unit held two workgroups of the 64 x 128 tile instead of
    // three from 31 kernel rows on (2449 x 2432, 32 x 32 taps 24.8 -> 21.5 us).
    static constexpr int kZeroRows = MODE == kT2Conv ? 1 : 2;
    static int steps(int kh) { return MODE == kT2Conv ? kh + 1 : MODE == kT2Down ? kh + 2 : kh / 2; }
    static int rows(int kh) { return kStride * (kPairs * kWy - 1) + steps(kh); }
    static int srows(int kh) { return (rows(kh) + kStride - 1) / kStride; }
    static int tab_rows(int kh) { return MODE == kT2Up ? 2 * kh : kh + 2 * kZeroRows; }
    static size_t image_bytes(int kh) {                                   // up to the last row that is staged, in the last section
        const size_t img = ((size_t)(kStride - 1) * srows(kh) + (rows(kh) - kStride) / kStride + 1) * kPitch * 2, patch = (size_t)kWx * kWy * kPatch * 4;
        return img > patch ? img : patch;
    }
    static size_t lds_bytes(int kh) { return image_bytes(kh) + (size_t)tab_rows(kh) * kTabRow * 2; }
};

inline int64_t t2_ceil(int a, int b) { return a / b + (a % b != 0); }

// Which flat tile hb_down2 takes: above these kernel rows two workgroups of four waves no longer fit a compute unit (to 16 x
// 41000, 32 x 32 taps 20.7 us, with two waves each 15.0).
inline T2Shape t2_down_flat(int nk, int kh) { return kh > (nk == 4 ? 30 : 25) ? kT2FlatPair : kT2Flat; }

// The flat tile for outputs of few rows, where the tall ones' last 64 rows would be a quarter empty or more.
//  - hb_down2: to 32 x 40000 / 48 x 70000 / 80 x 70000 with 16 x 16 taps 12.0 / 20.4 / 31.1 us, tall 15.4 / 23.0 / 37.9; to 48 x 32768 12.7, tall
//    11.7; to 32 x 20000 with 3 x 18 8.5, tall 8.0.
//  - hb_up2: to 66 x 131072 with 4 x 4 taps / 48 x 56000 with 32 x 32 8.5 / 9.1 us, tall 11.8 / 9.4; to 64 x 88000 with 32 x 32 tall is the faster
//    by 20 %.  Up to 18 taps across also for 49 to 63 rows (60 x 76000, 10 x 10: 7.3, tall 7.9); 2 x 56000, 4 x 4 4.8, tall 4.4.
//  - hb_conv2d: both have 8192 outputs, three tall or two flat workgroups fit a compute unit, and what a call takes follows the
//    most that one compute unit gets, `tall` and `flat`.  Many taps: from 3 : 2 on (80 x 49400, 32 x 32, 4 : 2: 18.1 us, tall 26.4; 80 x
//    70000, 5 : 3: 27.2, 31.5; 34 x 88000, 3 : 3: 27.0, 21.1); fewer: from 2 : 1 on, where the tall ones need three, or 5 : 3 (16 x
//    98600, 16 x 16, 4 : 1: 10.5, 13.7; 66 x 70000, 16 x 16, 5 : 3: 15.7, 24.1); less than 8 rows of taps, or
//    many rounds of both, as measured (48 x 200000, 3 x 3: 17.3, 20.4).
inline bool t2_flat(T2Mode mode, int nk, int kh, int Ho, int Wo, int units) {
    const bool partly = Ho <= 48 || (Ho > 64 && Ho <= 96);
    if (mode == kT2Up) return (partly || (nk == 1 && Ho < 64)) && Wo > (nk == 1 && Ho <= 32 ? 256 : 192) * units;
    if (mode == kT2Down) return Ho <= 32 ? Wo > (nk == 4 ? 128 : 96) * units : partly && Ho <= 80 && Wo > 192 * units && t2_down_flat(nk, kh) == kT2Flat;
    const int64_t tall = (t2_ceil(Ho, 64) * t2_ceil(Wo, 128) + units - 1) / units, flat = (t2_ceil(Ho, 16) * t2_ceil(Wo, 512) + units - 1) / units;
    if (nk == 3 && kh >= 20 ? 2 * tall >= 3 * flat : kh >= 8 && tall >= 3 && (tall >= 2 * flat || (tall >= 5 && 3 * tall >= 5 * flat))) return Ho <= 96;
    return (Ho <= 48 && Wo > 384 * units) || (Ho <= 96 && tall >= 7 && 4 * tall >= 5 * flat);
}

// hb_down2 and hb_up2.  Sizes are rows x columns.  The tile is 64 x 64 (hb_down2) or 64 x 128, but for outputs of few rows, see
// above, and narrow ones, of which it would leave half of the waves or more without work, where their rows still fill the chip:
//  - hb_down2: 256 x 16 for at most 16 columns (131072 x 8 outputs, 16 x 16 taps 13.2 us, 64 x 64 34.2; 262144 x 4, 32 x 32 43 and
//    85), and 128 x 32 up to 160 where that leaves fewer columns empty (63550 x 17, 16 x 16 12.6 and 20.6; 43691 x 24 12.3 and 17.6).
//  - hb_up2: 128 x 64 for at most 64 columns (524288 x 32 outputs, 32 x 32 taps 30.2 us, 64 x 128 44.2).
inline T2Shape t2_resample_tile(T2Mode mode, int nk, int kh, int Ho, int Wo, int units) {
    if (t2_ceil(Ho, 64) > units) {
        if (mode == kT2Up && Wo <= 64) return kT2Block;
        if (mode == kT2Down && Wo <= 16) return kT2Stack;
        if (mode == kT2Down && Wo <= 160 && 32 * t2_ceil(Wo, 32) < 64 * t2_ceil(Wo, 64)) return kT2Block;
    }
    if (!t2_flat(mode, nk, kh, Ho, Wo, units)) return kT2Row;
    return mode == kT2Down ? t2_down_flat(nk, kh) : kT2Flat;
}

// hb_conv2d, tiles in rows x columns.  `pieces`: output rows start inside 64-byte pieces of a line.
//  - 64 x 128 is the general tile (4096 x 4096, 3 x 3 / 11 x 11 / 20 x 20 / 32 x 32 taps 19.3 / 21.3 / 34.8 / 52.9 us, with the widest
//    21.5 / 25.9 / 37.9 / 53.8; 4000 x 4000, 32 x 32 51.0, 55.8).
//  - 64 x 256 writes fewer partial pieces, which counts where stores take longer than products (4000 x 4001, 3 x 3 / 16 x 16 /
//    28 x 5 / 32 x 32: 30.2 / 37.5 / 42.9 / 55.7 us, general 38.9 / 43.2 / 52.6 / 53.0) and its columns are used (32513 x 258, 24 x 24: 44,
//    general 34; 64527 x 65, 3 x 3: 24, general 12).  A compute unit holds two of its workgroups and three of the general
//    ones, so it also takes more than one round of work, and nearly two for the tallest kernels (1500 x 5985, 576 tiles, 3 x 3 /
//    16 x 16 / 28 x 5: 21.1 / 26.1 / 31.9, general 22.9 / 27.8 / 29.2; 3000 x 2977, 564 tiles, 3 x 3: 23.6, general 22.3).
//  - 64 x 64 where the others leave compute units idle (300 x 200, 32 x 32: 9.8, general 12.0; 1500 x 1500, 9 x 9: 7.7, 8.3).
//    Also where it has fewer empty columns (87381 x 48, 3 x 3 / 32 x 32: 8.9 / 23.2, general 15.1 / 32.4; 52428 x 160, 9 x 9: 16.4, 18.4),
//    unless the partial pieces of a low kernel cost more (32513 x 129, 3 x 3: 15.6, general 13.4).
//  - 128 x 32, two by two waves, for outputs of at most 32 columns, which leave the others' waves idle (524288 x 8, 3 x 3 / 32 x 32
//    taps 18.3 / 54 us, 64 x 64 29 / 85, general 47 / 120; 131072 x 32: 8.1 / 20.1, 10.5 / 28, 13.8 / 34), and enough rows to fill the
//    chip twice (9362 x 28, 9 x 9: 6.0, 64 x 64 5.8).  Or 128 x 64, two by two waves, for the columns that those fill (131072 x 64, 3 x 3 / 32 x
//    32: 11.2 / 32.1, 64 x 64 12.6 / 35.3; 49152 x 64, 3 x 3 7.7 and 7.1; 149796 x 56 20.2 and 16.7).
inline T2Tile t2_conv_tile(int Ho, int Wo, int kh, int nk, bool pieces, int units) {
    if (Wo <= 32 && t2_ceil(Ho, 64) > units) return {kT2Block, 1};
    if (Wo > 56 && Wo <= 64 && t2_ceil(Ho, 128) >= 2 * units) return {kT2Block, 2};
    if (t2_flat(kT2Conv, nk, kh, Ho, Wo, units)) return {kT2Flat, 2};
    const int64_t wide = t2_ceil(Ho, 64) * t2_ceil(Wo, 256);
    if (pieces && Wo > 768 && kh <= (wide >= 15 * units / 4 ? 29 : wide >= 9 * units / 4 ? 18 : 0)) return {kT2Row, 4};
    const bool half_used = Wo <= 64 || (Wo > 128 && Wo <= 192 && (!pieces || kh >= 16));
    return {kT2Row, !half_used && t2_ceil(Ho, 64) * t2_ceil(Wo, 128) >= units * 5 / 4 ? 2 : 1};
}

}  // namespace hb
