// Which kernel the filters of one window along x take in hb_sepblur.  Host arithmetic alone, so that a test can compile it with the
// host's compiler.
#pragma once
#include <stdint.h>

#ifndef HB_SEP_TILES
#define HB_SEP_TILES 2        // 16-column tiles per wave strip
#endif

namespace hb {

constexpr int kSepStrip = 16 * HB_SEP_TILES;              // columns of a wave
constexpr int kSepMarchCols = 4 * kSepStrip;              // of a workgroup of the march
constexpr int64_t kSepMarchShortMax = 24 << 20;           // outputs
constexpr int sep_wide_rows(int nt) { return nt < 4 ? 64 : 80; }          // fewer are a shallow image where the row is long

struct SepCall {
    int H, W;
    int nt;                // row tiles a step needs, (taps down + 30) / 16
    bool even;             // the input starts on a whole dword, and so does every row
    bool lines;            // every row of the output starts a 128-byte line
    int cu;                // compute units
};

// The march serves the filters of one window too: its loads are whole rows of pixels, not 16 rows of 64 bytes, its coefficients arrive
// while the first rows do, and the runs of its four strips meet in one L2 where rows of the output start inside 128-byte lines.  256 x 256,
// 16 x 16 / 9 x 45 taps 5.2 / 6.1 -> 3.4 / 4.2 us, 1024 x 1024 5.9 / 7.0 -> 4.6 / 6.1, 2160 x 3840 11.4 / 13.1 -> 10.7 / 12.0, 4096 x 4096 19.1 / 20.9 -> 17.7 / 18.9,
// 2047 x 2045, 9 x 45 taps 15.3 -> 10.4, 8191 x 8191 151 / 166 -> 120 / 102.  The kernel that requests all its row tiles up front is the faster one
//  - in large images, where the march's lines are no longer put together in time or its requests no longer spread over the
//    memory (8192 x 8192, 16 x 16 / 9 x 45 taps 62 / 66 us, the march 67 / 70, 8190 x 8190, 16 x 16 117 and 125), unless input rows start
//    between dwords or there are many row tiles a step (8192 x 8192, 9 x 64 taps 75, 72; 8190 x 8190, 9 x 45 132, 125);
//  - in images of a few rows, most of whose march is the row tiles ahead of the first (16 x 16, 64 taps down 3.7 us and 4.6, 16 x 300000, 9 x 30 taps
//    9.6 and 10.0; 17 x 128 3.8 and 3.6; 28 x 288, 44 taps 4.0 and 4.4; odd rows 29 x 24, 41 taps 4.0 and 4.6, but 32 x 100 5.5 and 4.8), longer ones where the row is long (17 x 40000, 16 x 16 taps 3.9 and 5.1, 33 x 300000 12.6
//    and 15.7, 48 x 40000, 9 x 64 taps 6.6 and 7.1, 84 x 27920, 50 taps 7.1 and 8.3, 26 x 31499, 37 taps 5.8 and 7.2; 16 x 16 5.5 and 5.1, 96 x 40000, 9 x 45 8.6 and 7.9);
//  - with five row tiles a step, where the march's segments are two steps and two workgroups on every unit (1080 x 1920, 9 x 64 taps 7.5 and 7.8);
//  - in tall narrow images, whose columns leave much of the march's 128 idle, once there is more than a round of its workgroups (12872 x 159, 41 taps 8.1
//    and 10.6, 10773 x 32, 55 taps 5.9 and 7.1, 8629 x 192, 22 taps 6.0 and 6.9; 14921 x 149, 19 taps 8.9 and 10.2; below that 0.7 to 0.9 of the time everywhere);
//    beyond 3 M pixels, and in lower images of four row tiles that start inside lines, the march gains again (11097 x 444, 57 taps 14.2 and 11.2, 5177 x 129, 49 taps 8.7 and 7.7).
inline bool sep_marches(const SepCall& c) {
    const int64_t all = (int64_t)((c.H + 15) / 16) * ((c.W + kSepMarchCols - 1) / kSepMarchCols);
    const bool large = (int64_t)c.H * c.W > kSepMarchShortMax && c.even && c.nt <= (c.lines ? 4 : 3);
    const int few = c.nt == 5 ? 32 : c.nt == 4 ? (c.even || c.W <= kSepStrip ? 32 : 24) : c.lines ? 16 : 0;
    const bool wide = c.lines && c.H < sep_wide_rows(c.nt) && c.W > 64 * c.cu;
    // with four or five row tiles a step from more than one round of workgroups on
    const int shallow = c.nt == 5 ? (c.even ? 112 : 56) : c.nt == 4 ? (c.even ? 48 : 32) : 0;
    const bool long_rows = c.H <= shallow && 2 * all > (c.nt == 5 || c.even ? 3 : 2) * c.cu;
    const bool pairs = c.lines && c.nt == 5 && all > 3 * c.cu && all <= 4 * c.cu;
    const int64_t strips = (c.W + kSepStrip - 1) / kSepStrip, marched = 4 * ((strips + 3) / 4);
    const bool idle = c.even && (c.lines || c.nt == 5 || (c.nt == 4 && c.H > 6400)) && (int64_t)c.H * c.W <= (11 << 18) && all > (c.nt <= 2 ? 4 : 2) * c.cu &&
                      all <= 12 * c.cu && 100 * marched >= (c.nt >= 4 ? 110 : 116) * strips;
    return !(large || wide || long_rows || pairs || idle || c.H <= few);
}

}  // namespace hb
