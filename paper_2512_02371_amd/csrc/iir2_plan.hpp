// Which signals hb_iir2 takes in one launch, a workgroup per channel.  Host arithmetic alone, so that a test can compile it with the host's compiler.
#pragma once
#include <stdint.h>

namespace hb {

constexpr int kIirAhead = 4;                  // tiles of 512 samples that a wave has in flight
constexpr int kIirChannelWaves = 16;          // of a channel's workgroup

// While each channel has a compute unit to itself: runs of up to four tiles, or eight where
// most units have one (T = 2500 .. 16384, 1 to 256 channels 10.2 us, 6.9 so; 32768, 1 / 64 / 256 channels 10.4 / 10.4 / 14.8, 8.4 / 9.0 /
// 12.4; 65536, 64 / 100 / 200 channels 10.7 / 14.0 / 21.9, 12.9 / 12.9 / 17.7; 400 x 8192 10.3, 11.9).  One to 16 channels owe
// this to the host, which takes 9.4 us for two launches: their kernels, replayed from a graph, take 6.5 us for 32768 samples, this one 7.9.
// Signals that start between dwords cost one compute unit more than they cost many: with few channels only up to 38 tiles
// (2 / 16 x 18433 8.3 / 8.6 us, two launches 8.6 / 8.8, 16387 7.9 / 8.2 and 8.4 / 8.6, 20001 9.1 / 9.5 and 8.6 / 8.9, 24575 10.6 / 11.0 and 8.6 / 8.8), up to three
// tiles a run from a tenth of the units on (31 x 20001 9.6 and 10.8; 24 x 9.6 and 8.6), and a little below, where two launches have clearly more than a wave per
// SIMD (25 x 22532 10.5 and 11.2; 25 x 20744 9.8 and 9.1, 23 x 24000 11.1 and 10.6), four from an eighth (32 x 32767 12.0 and 11.4),
// and up to eight only from three channels to four units on (160 x 40001 / 50001 16.6 / 18.0 and 18.4 / 20.0, 200 x 18.2 / 21.8 and 18.8 / 20.1).
inline bool iir_one_launch(int64_t C, int64_t ntiles, bool even, int cu) {
    if (C > cu || ntiles <= kIirAhead) return false;
    const int most = (even ? 2 * C >= cu : 4 * C >= 3 * cu) ? 8 : even || 8 * C >= cu ? 4 : 3;        // tiles a run
    if (most == 3 && (11 * C < cu || (10 * C < cu && 5 * C * ntiles <= 21 * cu))) return ntiles <= 38;
    return ntiles <= most * kIirChannelWaves;
}

}  // namespace hb
