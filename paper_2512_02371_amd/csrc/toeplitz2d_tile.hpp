// The workgroup tiles of the matrix kernel of hb_conv2d, hb_down2 and hb_up2: what each one covers, stages and keeps in
// LDS.  Host arithmetic only, also for tests that run without a GPU.
#pragma once
#include <stddef.h>

#include "hb.h"

namespace hb {

enum T2Mode { kT2Conv, kT2Down, kT2Up };

constexpr size_t kT2LdsOfCu = 160 << 10, kT2LdsGrain = 1280;          // of a compute unit; LDS is given out in these pieces

// workgroups of so much LDS that a compute unit holds
inline size_t t2_resident(size_t lds) { return kT2LdsOfCu / ((lds + kT2LdsGrain - 1) / kT2LdsGrain * kT2LdsGrain); }

// SHORT (outputs of few rows): the N index of a product is 8 row pairs x 4 runs of tiles beside each other instead
// of 32 row pairs.  16 x 200000, 3 x 3 / 32 x 32 taps: 14.3 / 45 us with the tall tile, 10.2 / 17 with this one.
template <int MODE, int NK, int NW, bool SHORT>
struct T2Geom {
    static constexpr int kPairs = SHORT ? 8 : 32, kBeside = 32 / kPairs;  // row pairs, runs of tiles in N
    static constexpr int kWx = 4;                                         // waves of a workgroup, beside each other
    static constexpr int kThreads = 64 * kWx;
    static constexpr int kOccupancy = MODE == kT2Conv ? (NW > 2 ? 2 : 3) : MODE == kT2Down ? 2 : NK > 1 ? 3 : 4;   // waves per SIMD
    static constexpr int kStride = MODE == kT2Conv ? 2 : MODE == kT2Down ? 4 : 1;   // input rows per n
    static constexpr int kTileStep = MODE == kT2Conv ? 16 : MODE == kT2Down ? 32 : 8;
    static constexpr int kCols = 16 * NW * kBeside * kWx, kRows = 2 * kPairs;         // output tile
    static constexpr int kChunks = (kTileStep * (NW * kBeside * kWx - 1) + 16 * NK) / 8;      // of 8 staged pixels per row
    static constexpr int kPitch = 8 * (kChunks | 1);
    static constexpr int kPatch = 32 * (16 * NW + 4);                     // floats per wave, see the stores
    // window chunks of a wave: distinct multiples of 8 pixels at which a fragment starts
    static constexpr int kUnit = MODE == kT2Up ? 8 : 16;
    static constexpr int kFrags = (kTileStep * (NW - 1) + 16 * (NK - 1)) / kUnit + 1;
    static constexpr int kMaxSteps = MODE == kT2Conv ? HB_MAX_TAPS_CONV2D + 1 : MODE == kT2Down ? HB_MAX_TAPS_CONV2D + 2 : HB_MAX_TAPS_CONV2D / 2;
    static constexpr int kPieces = ((kStride * (kPairs - 1) + kMaxSteps) * kChunks + kThreads - 1) / kThreads;   // staged per thread
    // Weight table.  A lane's eight weights start at position 8h - (its column's shift) + kPad, 1 (conv, up) or 2 (down)
    // apart, so a row is kept in kCopies copies of kCopy taps, each shifted by kShift, and every run starts on 8 bytes
    // (down: 16).  Pitches: the lanes served together fall into different banks (conv: blocks of 8 dwords at 0, 40, 16, 56 and, for
    // the row above, 32 further; up: of 4 dwords at 0, 20, 40, 60 plus 16 and 32; down: of 16 at 0, 48, 32, 16).
    static constexpr int kCopies = 4, kShift = MODE == kT2Down ? 2 : 1, kPad = MODE == kT2Conv ? 15 : MODE == kT2Down ? 30 : 7;
    static constexpr int kCopy = MODE == kT2Conv ? 80 : MODE == kT2Down ? 96 : 40, kTabRow = kCopies * kCopy;
    // Zero rows of the table, above and below the taps: a step reads row s - dy or s - 2 dy.  With two for hb_conv2d as well,
    // and the image's last section as long as the others, a compute unit held two workgroups of the 64 x 128 tile instead of
    // three from 31 kernel rows on (2449 x 2432, 32 x 32 taps 24.8 -> 21.5 us).
    static constexpr int kZeroRows = MODE == kT2Conv ? 1 : 2;
    static int steps(int kh) { return MODE == kT2Conv ? kh + 1 : MODE == kT2Down ? kh + 2 : kh / 2; }
    static int rows(int kh) { return kStride * (kPairs - 1) + steps(kh); }
    static int srows(int kh) { return (rows(kh) + kStride - 1) / kStride; }
    static int tab_rows(int kh) { return MODE == kT2Up ? 2 * kh : kh + 2 * kZeroRows; }
    static size_t image_bytes(int kh) {                                   // up to the last row that is staged, in the last section
        const size_t img = ((size_t)(kStride - 1) * srows(kh) + (rows(kh) - kStride) / kStride + 1) * kPitch * 2, patch = (size_t)kWx * kPatch * 4;
        return img > patch ? img : patch;
    }
    static size_t lds_bytes(int kh) { return image_bytes(kh) + (size_t)tab_rows(kh) * kTabRow * 2; }
};

}  // namespace hb
