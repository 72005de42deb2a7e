// How hb_fir1d divides an image among waves.  Host arithmetic alone, so that a test can compile it with the host's compiler.
#pragma once
#include <stdint.h>

#include <algorithm>

#ifndef HB_FIR_TILES
#define HB_FIR_TILES 4        // 16-column tiles per wave strip
#endif

namespace hb {

constexpr int kFirApartRows = 17;             // of an image whose even and odd rows are taken apart
constexpr int kFirMinWidth = 8;               // of an image

// Waves per workgroup of the walk: long filters are best as single-wave workgroups, the shorter ones four to a workgroup (measured).
constexpr int fir_walk_waves(int nk) { return nk >= 7 ? 1 : 4; }

struct FirCall {
    int H, W;
    int64_t in_pitch, out_pitch;
    bool even;             // the input starts on a whole dword, and so does every row
    bool lines;            // every row of the output starts a 128-byte line
    int ntaps, anchor;
    int cu;                // compute units
};
struct FirPlan {
    int nk, nko;           // windows of 32 pixels under a tile, under a pair of tiles
    bool lean;             // windows start where their addresses are even
    int step;              // rows of a group are this far apart
    int rowsteps;          // groups of rows
    int ntiles, run_tiles, nruns;   // the walk of long filters: tiles per row, per run, runs per group of rows
};

inline FirPlan fir_plan(const FirCall& c) {
    const auto up = [](int64_t a, int64_t b) { return (int)((a + b - 1) / b); };
    FirPlan p;
    const int nk = p.nk = up(15 + c.ntaps + (c.anchor & 1), 32);
    p.nko = up(31 + c.ntaps + (c.anchor & 1), 32);
    p.ntiles = up(c.W, 16);
    const int64_t px = (int64_t)c.H * c.W;

    // The walk of long filters: runs of an even number of tiles.  More waves have more bytes in flight and walk more windows ahead
    // of their runs.  From four windows on one wave per SIMD in all (4096 x 4096, 256 / 200 taps 22.8 / 21.0 us, 25.1 / 23.8 with
    // two; 1749 x 2603, 150 taps 12.7, 16.6; with three quarters of one 4096 x 4096 23.9 / 20.5, but 8192 x 4096, 256 taps 50.2
    // against 38.4), but two where large outputs have rows that start inside lines and the input's do not start between
    // dwords, whose shifting is work that one wave per SIMD already fills (2900 x 2900, 100 / 200 taps 15.7 / 17.9 us with one wave,
    // 13.5 / 16.9 with two, 4500 x 4500 40.9 / 42.3 and 35.8 / 36.5, 2000 x 3000, 100 taps 12.1 and 11.2; 2401 x 2603, 14.1 and 15.8,
    // 2000 x 3000, 200 taps 14.6 and 14.2, 5000 x 5000 44.1 and 47.2).
    // Shorter filters two (4096 x 4096, 40 / 80 taps 17.3 / 18.6, with one 18.3 / 19.1), and four on
    // large images of whole lines (8192 x 4096, 64 taps from memory 39.8 us, 45.8 with two).  Runs shorter than
    // the windows ahead of them only where there are too few waves otherwise (1749 x 2603, 256 taps 25.9 with runs of 10
    // tiles, 20.0 with 20).  Images of a few rows, most of whose lanes are idle, take two or three (8 x 500000, 34 taps 10.7 us with
    // four, 9.5 so; 1 x 1000000, 100 taps 10.7, 13.4 with one) and longer runs (256 taps 24 -> 18).
    int waves = 8;                                        // per compute unit
    if (nk <= 3) waves = c.H < 16 ? 12 : c.lines && px > (24 << 20) ? 16 : 8;
    else if (c.H >= 16) waves = !c.lines && c.even && (nk <= 6 ? px >= (4 << 20) : px >= (8 << 20) && px <= (20 << 20)) ? 8 : 4;
    const auto run_tiles = [&](int rowsteps) {
        int runs = std::min(waves * c.cu / rowsteps, p.ntiles / 4);
        const int long_runs = p.ntiles / ((c.H < 16 ? 4 : 2) * nk);
        if ((int64_t)rowsteps * long_runs >= 3 * c.cu) runs = std::min(runs, long_runs);
        return (up(p.ntiles, std::max(1, runs)) + 1) & ~1;
    };
    const auto tasks = [&](int rowsteps) { return (int64_t)rowsteps * up(p.ntiles, run_tiles(rowsteps)); };

    // Odd starts are met where the windows have room for the pixel more (17, 33, 49, ... taps would take another window for every tile)
    // and the rows fill more than one group.  The coefficients of a walk then wait for its place, which needs rows and runs that hide it.
    // Of 7301 random calls no one is more than 8 % slower so than with plain groups, 34 more than 3 %; 7 miss more than 8 %.
    //  - One window: all but the narrowest (1000 x 32 5 % slower).
    //  - Two or three: more than a round of waves, with runs of four tiles clearly more (1025 x 1012, 18 taps, 1.6 % more, 5.3 us against 6.0; 7706 x 512, 41 taps 9.5 -> 6.8 us, 4109 x 465, 35 taps 9.1 -> 8.1, 5547 x 201, 40 taps 8.2 -> 7.3).
    //    Within one where the groups, which are of 32 rows in pairs, do not make it two (167 x 11451, 50 taps 5.6 against 6.8): with three
    //    windows always (47 x 3390, 80 taps 6.6 -> 5.9), with two in long rows (356 x 1534, 34 taps 6.2 -> 5.7), or short runs of whole lines
    //    (323 x 832, 40 taps 4.7 -> 4.3; 2222 x 331, 24 taps 5.4 against 5.8, 200 x 501, 40 taps 5.5 and 5.6).
    //  - Four to six: all but the narrowest (68 x 128, 132 taps 7.5 -> 6.4; 6752 x 32, 96 taps 4.7 against 5.2), while the pair of groups that the last rows may
    //    begin leaves the runs about as long as they are (5453 x 3253, 157 taps, two runs a row instead of three 27.5 against 33.7).
    //  - Seven to nine, which hide least: from 384 K pixels on (1579 x 639, 228 taps 12.3 -> 10.5, 142 x 7154, 215 taps with runs of six tiles for four 10.6 -> 9.0; 200 x 501, 200 taps 7.1 against 7.4, 5428 x 96, 211 taps 7.5 and
    //    8.2), and not with a third more groups (34 x 11867, 205 taps 7.9 and 8.6).
    const int plain = up(c.H, 16), apart = c.in_pitch % 2 ? 2 * up(c.H, 32) : plain;
    const bool room = up(16 + c.ntaps, 32) == nk && up(32 + c.ntaps, 32) == p.nko;
    const int64_t round = 4 * c.cu;
    bool gains;
    if (nk == 1) gains = c.W > 32;
    else if (nk <= 3) gains = c.W > 48 && (tasks(plain) > (run_tiles(plain) > 4 ? round : round + round / 50) || (tasks(apart) <= round && (nk == 3 || c.W > 1000 || (c.lines && c.W > 64 && run_tiles(apart) <= 4))));
    else if (nk <= 6) gains = c.W > 48 && 5 * run_tiles(apart) < 7 * run_tiles(plain);
    else gains = c.W > 128 && px >= (3 << 17) && 7 * apart <= 8 * plain;
    p.lean = !c.even && room && c.H >= kFirApartRows && gains && c.out_pitch <= ((int64_t)1 << 25);           // 32-bit byte offsets inside a group of 32 rows
    p.step = p.lean && c.in_pitch % 2 ? 2 : 1;
    p.rowsteps = p.lean ? apart : plain;
    p.run_tiles = run_tiles(p.rowsteps);
    p.nruns = up(p.ntiles, p.run_tiles);
    return p;
}

}  // namespace hb
