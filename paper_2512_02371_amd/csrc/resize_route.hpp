// Which kernels a call of hb_resize takes.  Host arithmetic alone, so that a test can compile it with the host's compiler.
#pragma once
#include <math.h>
#include <stdint.h>

namespace hb {

constexpr int kRzChunks = 12;                 // chunks of 32 columns whose coefficients are kept in LDS
constexpr int kRzMinWidth = 8;                // of an image
// A workgroup's waves own the same columns, either one below the other, each with its own T, or (SHARED, for
// outputs too small to fill the chip that way) all the same 16 rows: the input rows are dealt among them.
template <bool SHARED>
struct RzGeom {
    static constexpr int kWaves = SHARED ? 8 : 4;
    static constexpr int kRows = SHARED ? 512 : 160;      // input rows whose horizontal results T holds at a time
    static constexpr int kPitch = kRows + 40;             // halves per xo: 32 rows beyond, and an odd multiple of 16 bytes
};

struct RzCall {
    int C, H, W, Ho, Wo, band_y, band_x;
    int64_t in_pitch;
    bool even;             // every plane starts on a whole dword, and the rows' pitch is even
    bool lines;            // every row of the output starts a 128-byte line
    int cu;                // compute units
};
struct RzRoute {
    bool one_launch;
    bool apart;            // ... and reads even and odd rows apart
    int groups;            // of 16 output rows per wave; 0: the waves of a workgroup share one
};

inline RzRoute rz_route(const RzCall& c) {
    const auto ceil16 = [](int n) { return (n + 15) / 16; };
    // What a group of n outputs spans of an axis when its starts advance by the scale
    const auto span = [](int n, int n_in, int n_out, int band) { return (double)((n_out < n ? n_out : n) - 1) * n_in / n_out + band + 1; };
    const double span_x = span(16, c.W, c.Wo, c.band_x), span_y = span(16, c.H, c.Ho, c.band_y);
    const int groups = ceil16(c.Ho), ngx = ceil16(c.Wo);
    const int64_t waves = (int64_t)c.C * ngx * groups;                    // of one group each
    const int64_t pixels = (int64_t)c.C * c.H * c.W;
    RzRoute r;
    // Groups of 16 output rows per wave: more share more, while the rows they need fit the wave's LDS and the
    // chip keeps two waves per SIMD (2048 x 2048 from 4096 x 4096: 34 / 29 / 27 us with 1 / 2 / 4; 450 x 450 x 3 from
    // 2048 x 2048: 19 / 29 / 37).  Under one wave per SIMD the waves of a workgroup share one group (256 x 256 from
    // 4096 x 4096: 20 us against 92), under two where its rows do not fit a wave's LDS at once (512 x 512 from
    // 8192 x 8192: 56 against 96; at two 256 x 2048 from 4096 x 4096 33 with a group per wave, 41 shared), and
    // where one group is all there is (64 x 240 x 4096 -> 12 x 600 68 against 121).
    const bool tall = span_y > RzGeom<false>::kRows;
    const auto good = [&](int q) { return waves >= 8 * q * c.cu && 16.0 * q * c.H / c.Ho + c.band_y <= RzGeom<false>::kRows; };
    const bool shared = waves < (tall ? 8 : 4) * c.cu || (tall && groups == 1);
    r.groups = shared ? 0 : good(4) ? 4 : good(2) ? 2 : 1;

    // Rows that start on odd samples are read at a fraction of the rate.  Of an odd pitch that is every second row, and the one-launch
    // kernel can read even and odd rows apart (8 planes of 2048 rows at a pitch of 2049, factors 4 / 9: 57 / two launches 54 -> 44 / 40 us;
    // 1947 x 6281 -> 214 x 690 28.9 -> 18.9; 4095 x 4095 -> 900 45 -> 29; 8 x 787 x 5325 -> 164 x 7830 122 -> 82), but
    //  - only groups whose rows fit T and whose windows lie inside the row; the others take its general loop, with three waves
    //    per SIMD instead of four (16 x 3012 x 89 -> 1799 x 60 11 -> 18, 8 x 5171 x 155 -> 1697 x 54 15 -> 19).  Beyond 12 M pixels the other windows are
    //    worth it (3 x 5459 x 4520 -> 3329 x 5014), if they cost no round as well (16 x 4166 x 311 -> 5190 x 35 30 -> 42);
    //  - a group per wave costs it a round of workgroups where three to a unit are nearly twice as many as four (1266 x 1483 -> 876 x 1026 7.3 -> 8.9,
    //    16 x 273 x 532 -> 42 x 823 13.0 -> 16), which it is worth with more than one chunk a window (1 x 1611 x 2997 -> 1803 x 1624 19.3 -> 16.0, 3 x 413 x
    //    2815 -> 281 x 858 14.6 -> 11.0), if that is not for the sample further left alone, and in large images (1 x 4313 x 3334 -> 1434 x 1108 32 -> 23);
    //  - few windows of many chunks, which the loop for more than four takes, are better off with two launches (16 x 1277 x 1311 -> 180 x 86 43 -> 53,
    //    3 x 3632 x 1409 -> 545 x 145 38 -> 55);
    //  - of shared groups large images gain (8 x 3907 x 465 -> 659 x 78 25 -> 18), others with more than one to a unit (586 x 2559 -> 67 x 4036 16 -> 12),
    //    few waves and small images do not (2 x 600 x 603 -> 40 18.6, 19.2; 217 x 2189 -> 198 x 176 8.2 -> 9.9), nor where half of the windows or more
    //    reach over the row's ends (16 x 4295 x 284 -> 271 x 17 49 -> 55), or long windows have no more rows than the 32 that one wave takes at a time (603 x 5703 ->
    //    425 x 448 12.5 -> 16).
    // Of 6215 random calls of odd pitches one in a hundred is more than 8 % slower so than the better way.
    const bool would_be_two = pixels > (6 << 20) && span_y > 120;         // of odd rows, see below
    const double rows = span(16 * (r.groups > 1 ? r.groups : 1), c.H, c.Ho, c.band_y) - 1;
    const bool fits = rows <= (shared ? RzGeom<true>::kRows : RzGeom<false>::kRows) && span_x + 1 <= 32 * kRzChunks;
    const int nk = (int)(span_x + 32) / 32, nk_plain = (int)(span_x + 30.5) / 32;      // chunks of a window, with the sample further left and without
    const double step = 16.0 * c.W / c.Wo;                // columns from group to group
    const double inside = (floor((c.W - 32 * nk + c.band_x / 2.0 + 1) / step) - ceil((c.band_x / 2.0 + 1) / step) + 1) / ngx;
    const int64_t wgs = r.groups ? (int64_t)c.C * ngx * ((groups + 4 * r.groups - 1) / (4 * r.groups)) : waves;
    const auto rounds = [&](int per_cu) { return (wgs + per_cu * c.cu - 1) / (per_cu * c.cu); };
    bool gains;
    if (shared) gains = inside > 0.54 && (rows > 32 || nk <= 4) && (pixels > (6 << 20) || (waves > c.cu && pixels > (1 << 19) && (inside > 0.8 || pixels > (2 << 20)) &&
                                                                                         (nk <= 5 || pixels > (1 << 20))));
    else if (would_be_two && ngx <= 12 && nk > 6) gains = false;
    else if (4 * rounds(3) < 7 * rounds(4)) gains = pixels > (12 << 20) || inside > 0.5;
    else gains = inside > 0.5 && (pixels > (12 << 20) || (nk > 1 && nk == nk_plain));
    r.apart = (c.in_pitch & 1) && fits && gains;

    // The one-launch kernel keeps the coefficients of kRzChunks chunks; wider spans it takes chunk by chunk, each one a
    // round trip, once for every group of rows that needs them.  That pays only while a group spans few rows and the
    // waves are few (2048 x 2048 -> 1024 x 26 28 us, two launches 60; -> 26 x 26 460 against 99, 16 x 1024 x 1024 -> 500 x 40
    // 63 against 37).
    // Nor does it pay where the rows of a group are so many that few workgroups pass over most of the image (2832 x 3696
    // -> 55 x 210, 370 x 1081 pixels a group: 84 us, two launches 64; 127 x 1655 47 against 77).
    // It reads a row for every group of outputs that needs it: large images of odd rows that are not taken apart take two launches
    // (16 planes of 2048 rows at a pitch of 2049 -> 228 x 228 97 us, in one 135 and, apart, 159; 3 x 4000 x 4001 -> 444 x 2667 126, 136, 140), but
    // for odd pitches whose groups are shared (16 x 5140 x 115 -> 506 x 8 29, in one 16) or have windows of one chunk (16 x 473 x 4430 -> 60 x 4397 118, 88, but
    // 1 x 1101 x 5825 -> 70 x 6899 41, 50).
    const bool odd_rows = !r.apart && !c.even && !((c.in_pitch & 1) && (shared || (nk == 1 && c.Wo <= c.W)));
    // Large enlargements are bound by their stores, of 64-byte runs here and 256-byte runs there (3 x 2048 x 2048 to three
    // times the size 222 us, two launches 170); where rows start inside 128-byte lines neither run is whole (227 against 246).
    const bool line_stores = (double)c.Ho * c.Wo >= 2.0 * c.H * c.W && (int64_t)c.C * c.Ho * c.Wo > (16 << 20) && c.lines;
    // One or two groups of rows as wide as the image leave a wave with a long walk and nothing to share (32 x 200 x 4096 -> 4
    // x 4000 183 us, two launches 96; 8 x 514 x 8160 -> 30 x 4720 81 against 74); narrow results have fewer products in each
    // row's pass (64 x 240 x 4096 -> 12 x 600 68 against 82, 12 x 1600 118 against 104).
    const bool few_groups = tall && groups <= 2 && waves >= 8 * c.cu && 4 * (int64_t)c.Wo >= c.W;
    r.one_launch = c.W >= kRzMinWidth && (span_x <= 32 * kRzChunks ? span_x * span_y <= 3.2e5 : span_y <= 128 && waves <= 2 * c.cu) &&
                   !line_stores && !few_groups && !(odd_rows && would_be_two);
    return r;
}

}  // namespace hb
