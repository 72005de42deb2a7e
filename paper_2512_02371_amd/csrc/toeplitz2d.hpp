// The matrix kernel shared by the stages with an arbitrary 2-D kernel (hb_conv2d, hb_down2, hb_up2).
//
// A workgroup stages the clamped input pixels under its output tile in LDS, and every kernel row is then a
// product of Toeplitz weights with rows of that LDS image: v_mfma_f32_32x32x16_f16 with
//     A[m][k]   the weights, m = 16 output columns x 2 neighbouring output rows dy
//     B[k][n]   pixel k of the window in input row kStride n + s, n = 0 .. 31
//     D[m][n]   output columns x output rows 2n + dy
// summed over the row offsets s that either dy needs and over the window in chunks of 16 pixels.  One step s
// gives output row 2n + dy its kernel row s - dy (hb_conv2d), s - 2 dy (hb_down2) or 2s + dy (hb_up2); the rows
// of the weight table that do not exist are zero.  Why this tile: 16 columns with a window of 16 + kw - 1 pixels
// waste the least of the K = 16 chunks (47 of 48 pixels at kw = 32, 2/3 of the products useful; 32 columns 1/2),
// and putting two output rows into M costs one more step s (3 %) instead of half the products.
// Before, a wave kept input rows in registers and added every product, shifted by its kernel row, into the
// output with lane shifts, and those additions took as long as the products.  4096 x 4096, back to back:
// hb_conv2d 3 x 3 / 16 x 16 / 32 x 32 32.2 / 43.8 / 78 -> 23.0 / 33.3 / 56 us, hb_down2 + hb_up2 of 16 x 16 60 -> 42.6
// (kernels 21 + 18); a copy of the same bytes takes 18 and 23.  At 32 x 32 the matrix units are busy 45 % of the time
// (24 of 56 us), the LDS 40 %: what is left is the load and the store phase of the two workgroups a compute unit
// holds.
//
// The window of tile w is the one of tile w - 1 moved by kTileStep pixels, so the chunks are shared:
// per step a wave reads NK weight fragments and about NW + NK chunks for NW NK products.  The LDS rows that one
// read touches are consecutive (rows are dealt to kStride sections) at a pitch of an odd multiple of 16
// bytes: no bank conflicts (an even one doubles them).  Weights come from a zero-padded table of the taps, kept
// twice, one half shifted by a tap, so that every run of eight starts on a 4-byte address (a table of all
// fragments would take 100 KB).  Chains of products end after two steps and are added up outside the matrix unit:
// error of 32 x 32 taps against fp64 8.5e-8, with chains of 16 steps 1.6e-7, for 2 us less.
#pragma once
#include <algorithm>

#include "hb_device.hpp"

namespace hb {

enum T2Mode { kT2Conv, kT2Down, kT2Up };

struct T2Args {
    const half_t* in;
    float* out;
    int H, W;                                 // input
    int Ho, Wo;                               // output
    int64_t in_pitch, out_pitch;
    int kh, kw, ay, ax;
    int ncol, nrow, ntiles, per_wg;           // workgroup tiles across, down and in all; tiles of one workgroup
    int stream;                               // non-temporal stores
    int steps, srows, rows;                   // row offsets s; LDS rows per section, input rows staged
    uint16_t taps[HB_MAX_TAPS_CONV2D * HB_MAX_TAPS_CONV2D];   // kh x kw, row-major
};

typedef u32x4 u32x4_u __attribute__((aligned(4)));

constexpr int kT2MinWidth = 8;                // of an image
constexpr int kT2Pad = 32;                    // zero taps left of a table row (down: window position - 2 * 15)
constexpr int kT2Copy = 112;                  // taps per copy: up to position 63, and so that the reads of the
constexpr int kT2TabRow = 2 * kT2Copy;        // copies and of neighbouring rows fall into different banks
constexpr int kT2ZeroRows = 2;                // above and below the taps

// SHORT (outputs of few rows): the N index of a product is 8 row pairs x 4 runs of tiles beside each other instead
// of 32 row pairs, and a workgroup's waves lie beside each other.  24 x 100000, 3 x 3 / 32 x 32 taps: 18.0 / 41 us with the
// tall tile, 10.5 / 22 with this one.
template <int MODE, int NK, int NW, bool SHORT>
struct T2Geom {
    static constexpr int kPairs = SHORT ? 8 : 32, kBeside = 32 / kPairs;  // row pairs, runs of tiles in N
    static constexpr int kWy = MODE == kT2Down || SHORT ? 1 : 2;          // waves of a workgroup
    static constexpr int kWx = (MODE == kT2Down ? 2 : 4) / kWy;
    static constexpr int kThreads = 64 * kWx * kWy;
    // The walk over several tiles pays where loads and stores bound the kernel.  hb_conv2d keeps the wider tile instead:
    // fewer LDS reads per product, and no registers left to load ahead.
    static constexpr bool kWalk = MODE != kT2Conv;
    static constexpr int kOccupancy = MODE == kT2Conv ? (NW > 2 ? 2 : 3) : MODE == kT2Down ? 2 : NK > 1 ? 3 : 4;   // waves per SIMD
    static constexpr int kStride = MODE == kT2Conv ? 2 : MODE == kT2Down ? 4 : 1;   // input rows per n
    static constexpr int kTileStep = MODE == kT2Conv ? 16 : MODE == kT2Down ? 32 : 8;
    static constexpr int kCols = 16 * NW * kBeside * kWx, kRows = 2 * kPairs * kWy;         // output tile
    static constexpr int kChunks = (kTileStep * (NW * kBeside * kWx - 1) + 16 * NK) / 8;      // of 8 staged pixels per row
    static constexpr int kPitch = 8 * (kChunks | 1);
    static constexpr int kPatch = 32 * (16 * NW + 4);                     // floats per wave, see the stores
    // window chunks of a wave: distinct multiples of 8 pixels at which a fragment starts
    static constexpr int kUnit = MODE == kT2Up ? 8 : 16;
    static constexpr int kFrags = (kTileStep * (NW - 1) + 16 * (NK - 1)) / kUnit + 1;
    static constexpr int kMaxSteps = MODE == kT2Conv ? HB_MAX_TAPS_CONV2D + 1 : MODE == kT2Down ? HB_MAX_TAPS_CONV2D + 2 : HB_MAX_TAPS_CONV2D / 2;
    static constexpr int kPieces = ((kStride * (kPairs * kWy - 1) + kMaxSteps) * kChunks + kThreads - 1) / kThreads;   // staged per thread
    static int steps(int kh) { return MODE == kT2Conv ? kh + 1 : MODE == kT2Down ? kh + 2 : kh / 2; }
    static int rows(int kh) { return kStride * (kPairs * kWy - 1) + steps(kh); }
    static int srows(int kh) { return (rows(kh) + kStride - 1) / kStride; }
    static int tab_rows(int kh) { return MODE == kT2Up ? 2 * kh : kh + 2 * kT2ZeroRows; }
    static size_t image_bytes(int kh) {
        const size_t img = (size_t)kStride * srows(kh) * kPitch * 2, patch = (size_t)kWx * kWy * kPatch * 4;
        return img > patch ? img : patch;
    }
    static size_t lds_bytes(int kh) { return image_bytes(kh) + (size_t)tab_rows(kh) * kT2TabRow * 2; }
};

template <int MODE, int NK, int NW, bool SHORT>
__global__ void __launch_bounds__((T2Geom<MODE, NK, NW, SHORT>::kThreads), (T2Geom<MODE, NK, NW, SHORT>::kOccupancy)) toeplitz2d_mfma_kernel(T2Args p, int table_offset) {
    using G = T2Geom<MODE, NK, NW, SHORT>;
    extern __shared__ __attribute__((aligned(16))) char s_dyn[];
    half_t* const s_px = reinterpret_cast<half_t*>(s_dyn);
    half_t* const s_tab = reinterpret_cast<half_t*>(s_dyn + table_offset);
    // the taps come from the kernel arguments in one round trip (the table built straight from there, one gather
    // after the other, took 10 us)
    __shared__ __attribute__((aligned(16))) uint16_t s_taps[HB_MAX_TAPS_CONV2D * HB_MAX_TAPS_CONV2D];

    const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int c = lane & 31, h = lane >> 5;
    const int wx = wv % G::kWx, wy = wv / G::kWx;
    // a workgroup takes per_wg tiles, one below the other, and every XCD one contiguous run of them: neighbours
    // share their halo pixels in one L2
    const int first = xcd_contiguous(blockIdx.x, gridDim.x) * p.per_wg, last = min(first + p.per_wg, p.ntiles);

    // The pixels under a tile's windows, both indices clamped: pieces of eight, what reaches over a row's ends
    // requested from an address inside and shifted into place on its way to LDS.  Piece u of a thread is piece
    // tid + kThreads u of the tile, its row and column kept by addition; past the end the last row's repeat.
    half8 ahead[G::kPieces];
    const int r_first = tid / G::kChunks, ch_first = tid - r_first * G::kChunks;
    auto next_piece = [](int& r, int& ch) {
        r += G::kThreads / G::kChunks;
        ch += G::kThreads % G::kChunks;
        if (ch >= G::kChunks) {
            ch -= G::kChunks;
            ++r;
        }
    };
    auto tile_origin = [&](int t, int& x, int& y) {       // of its pixels
        const int ct = t / p.nrow, rt = t - ct * p.nrow;
        x = (MODE == kT2Conv ? G::kCols * ct : MODE == kT2Down ? 2 * G::kCols * ct : G::kCols / 2 * ct) - p.ax;
        y = (MODE == kT2Conv ? G::kRows * rt : MODE == kT2Down ? 2 * G::kRows * rt : G::kRows / 2 * rt) - p.ay;
    };
    auto request = [&](int t) {
        int x, y, r = r_first, ch = ch_first;
        tile_origin(t, x, y);
#pragma unroll
        for (int u = 0; u < G::kPieces; ++u, next_piece(r, ch)) {
            const int row = clampi(y + min(r, p.rows - 1), 0, p.H - 1);
            ahead[u] = ldg8(p.in, 2u * ((uint32_t)row * (uint32_t)p.in_pitch + (uint32_t)clampi(x + 8 * ch, 0, p.W - 8)));
        }
    };
    auto deliver = [&](int t) {
        int x, y, r = r_first, ch = ch_first;
        tile_origin(t, x, y);
        const bool inside = x >= 0 && x + 8 * G::kChunks <= p.W;          // uniform
        if (!inside) {
#pragma unroll
            for (int u = 0; u < G::kPieces; ++u, next_piece(r, ch)) {
                ahead[u] = shift_in_from_right(ahead[u], max(x + 8 * ch - (p.W - 8), 0));
                ahead[u] = shift_in_from_left(ahead[u], max(-x - 8 * ch, 0));
            }
            r = r_first, ch = ch_first;
        }
#pragma unroll
        for (int u = 0; u < G::kPieces; ++u, next_piece(r, ch)) {
            const int rl = min(r, p.rows - 1);
            *reinterpret_cast<half8*>(s_px + ((rl % G::kStride) * p.srows + rl / G::kStride) * G::kPitch + 8 * ch) = ahead[u];
        }
    };

    for (int i = 8 * tid; i < p.kh * p.kw; i += 8 * G::kThreads)
        *reinterpret_cast<u32x4*>(s_taps + i) = *reinterpret_cast<const u32x4_u*>(p.taps + i);
    request(first);
    lds_barrier();
    // weight table: conv / down row r holds kernel row r - kT2ZeroRows; up row 2 (2s + dy) + dx holds the taps
    // 2t + dx of kernel row 2s + dy
    const int tab_rows = MODE == kT2Up ? 2 * p.kh : p.kh + 2 * kT2ZeroRows;
    for (int i = tid; i < tab_rows * (kT2TabRow / 8); i += G::kThreads) {
        const int r = i / (kT2TabRow / 8), j = 8 * (i - r * (kT2TabRow / 8));
        const int t0 = (j >= kT2Copy ? j - kT2Copy + 1 : j) - kT2Pad;
        const int ry = MODE == kT2Up ? r >> 1 : r - kT2ZeroRows;
        half8 v;
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            const int t = t0 + k, rx = MODE == kT2Up ? 2 * t + (r & 1) : t;
            const bool live = ry >= 0 && ry < p.kh && t >= 0 && rx < p.kw;
            const uint16_t tap = s_taps[live ? ry * p.kw + rx : 0];
            v[k] = live ? __builtin_bit_cast(half_t, tap) : (half_t)0;
        }
        *reinterpret_cast<half8*>(s_tab + 8 * i) = v;
    }
    deliver(first);
    lds_barrier();

    // lane (m = c, h): eight weights from window position 16 kk + 8h on; lane (n = c, h): eight pixels from there on
    const int mx = c & 15, mdy = c >> 4;
    const int t0 = 8 * h - (MODE == kT2Conv ? mx : MODE == kT2Down ? 2 * mx : mx >> 1) + kT2Pad;
    const int row0 = MODE == kT2Conv ? kT2ZeroRows - mdy : MODE == kT2Down ? kT2ZeroRows - 2 * mdy : 2 * mdy + (mx & 1);
    const half_t* const tab = s_tab + row0 * kT2TabRow + (t0 & 1 ? kT2Copy + t0 - 1 : t0);
    const int pair = c % G::kPairs, beside = c / G::kPairs;
    const half_t* const px = s_px + (G::kPairs * wy + pair) * G::kPitch + G::kTileStep * NW * (G::kBeside * wx + beside) + 8 * h;
    // stores: lane (n = c, h) holds columns 16 w + 8 (q & 1) + 4h + r of rows 2n + q / 2; a patch turns the 32 rows of
    // one dy into runs of 64 NW bytes
    float* const patch = reinterpret_cast<float*>(s_dyn) + wv * G::kPatch;
    constexpr int kPatchPitch = 16 * NW + 4, kLanes = 4 * NW, kPer = 64 / kLanes;
    const int rr = lane / kLanes, xx = 4 * (lane - rr * kLanes);

#pragma unroll 1
    for (int tile = first; tile < last; ++tile) {
        if (G::kWalk && tile + 1 < last) request(tile + 1);           // on its way during the products
        const int ct = tile / p.nrow, rt = tile - ct * p.nrow;        // tiles run down the columns
        const int xw = G::kCols * ct + 16 * NW * G::kBeside * wx, yw = G::kRows * rt + 2 * G::kPairs * wy;    // the wave's outputs
        const bool active = xw < p.Wo && yw < p.Ho;       // uniform
        floatx16 total[NW];
#pragma unroll
        for (int w = 0; w < NW; ++w) total[w] = floatx16{};
        if (active) {
            struct Frags { half8 a[NK], b[G::kFrags]; };
            auto fetch = [&](int s, Frags& f) {
                const half_t* const trow = tab + s * (MODE == kT2Up ? 4 : 1) * kT2TabRow;
                const half_t* const prow = px + ((s % G::kStride) * p.srows + s / G::kStride) * G::kPitch;
#pragma unroll
                for (int kk = 0; kk < NK; ++kk) f.a[kk] = __builtin_bit_cast(half8, *reinterpret_cast<const u32x4_u*>(trow + 16 * kk));
#pragma unroll
                for (int u = 0; u < G::kFrags; ++u) f.b[u] = *reinterpret_cast<const half8*>(prow + G::kUnit * u);
            };
            auto products = [&](const Frags& f, floatx16 (&acc)[NW]) {
#pragma unroll
                for (int kk = 0; kk < NK; ++kk)
#pragma unroll
                    for (int w = 0; w < NW; ++w) acc[w] = mfma32x32x16(f.a[kk], f.b[(G::kTileStep * w + 16 * kk) / G::kUnit], acc[w]);
            };
            // two steps a turn, each one's fragments read during the products of the one before
            Frags even, odd;
            fetch(0, even);
#pragma unroll 1
            for (int s = 0; s < p.steps; s += 2) {
                floatx16 acc[NW];
#pragma unroll
                for (int w = 0; w < NW; ++w) acc[w] = floatx16{};
                fetch(min(s + 1, p.steps - 1), odd);
                products(even, acc);
                __builtin_amdgcn_sched_barrier(0);
                fetch(min(s + 2, p.steps - 1), even);
                if (s + 1 < p.steps) products(odd, acc);
#pragma unroll
                for (int w = 0; w < NW; ++w) total[w] += acc[w];
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        lds_barrier();                                     // the LDS image becomes the waves' store patches
        if (active) {
            const bool whole = xw + 16 * NW * G::kBeside <= p.Wo && yw + 2 * G::kPairs <= p.Ho;   // uniform
#pragma unroll
            for (int dy = 0; dy < 2; ++dy) {
#pragma unroll
                for (int w = 0; w < NW; ++w)
#pragma unroll
                    for (int j = 0; j < 2; ++j) {
                        const int q = 2 * dy + j;
                        *reinterpret_cast<floatx4*>(patch + c * kPatchPitch + 16 * w + 8 * j + 4 * h) =
                            floatx4{total[w][4 * q], total[w][4 * q + 1], total[w][4 * q + 2], total[w][4 * q + 3]};
                    }
                wave_lds_fence();
#pragma unroll
                for (int i = 0; i < 32 / kPer; ++i) {
                    const int n = kPer * i + rr, y = yw + 2 * (n % G::kPairs) + dy, x = xw + 16 * NW * (n / G::kPairs) + xx;
                    const floatx4 v = *reinterpret_cast<const floatx4*>(patch + n * kPatchPitch + xx);
                    float* const dst = p.out + (int64_t)y * p.out_pitch + x;
                    if (whole && p.stream) {
                        __builtin_nontemporal_store(v, reinterpret_cast<floatx4_u*>(dst));
                    } else if (whole) {
                        *reinterpret_cast<floatx4_u*>(dst) = v;
                    } else if (y < p.Ho) {
#pragma unroll
                        for (int k = 0; k < 4; ++k)
                            if (x + k < p.Wo) dst[k] = v[k];
                    }
                }
                wave_lds_fence();
            }
        }
        if (G::kWalk && tile + 1 < last) {
            lds_barrier();                                 // patches read
            deliver(tile + 1);
            lds_barrier();
        }
    }
}

// The short tile where most of the tall ones would be empty and they are more than one round of workgroups; below, its
// larger workgroups only take longer (8 x 4096, 16 x 16 taps 11.2 us, tall 8.1).
template <int MODE, int NK, int NW>
static bool t2_short(const T2Args& a) {
    using Tall = T2Geom<MODE, NK, NW, false>;
    return a.Ho <= (MODE == kT2Conv ? 3 * Tall::kRows / 4 : Tall::kRows / 2) && ceil_div(a.Wo, Tall::kCols) > 3 * num_cu();
}

template <int MODE, int NK, int NW, bool SHORT>
static hb_status t2_launch(T2Args& a, hipStream_t st) {
    using G = T2Geom<MODE, NK, NW, SHORT>;
    const int64_t tiles = (int64_t)ceil_div(a.Wo, G::kCols) * ceil_div(a.Ho, G::kRows);
    if (tiles > 0x3fffffff) return HB_ERR_UNSUPPORTED;
    // The resampling kernels' runs of 64 and 128 bytes, where they are not whole lines, leave through the L2, which puts
    // neighbours together (4094 x 4094 and 2047 x 2047, 8 x 8 taps: 46 us, streamed 62; smaller outputs, which the
    // memory-side cache takes in, are better streamed: 1078 x 1916 17.9 against 19.6).
    a.stream = !G::kWalk || (a.out_pitch % 32 == 0 && aligned_to(a.out, 128)) || (int64_t)a.Ho * a.Wo * 4 <= (32 << 20);
    a.steps = G::steps(a.kh);
    a.rows = G::rows(a.kh);
    a.srows = G::srows(a.kh);
    a.ncol = ceil_div(a.Wo, G::kCols);
    a.nrow = ceil_div(a.Ho, G::kRows);
    a.ntiles = (int)tiles;
    const size_t lds = G::lds_bytes(a.kh);
    const auto kernel = toeplitz2d_mfma_kernel<MODE, NK, NW, SHORT>;
    if (allow_dynamic_lds(reinterpret_cast<const void*>(kernel), lds) != HB_OK) return HB_ERR_HIP;
    // as many workgroups as are resident at once
    const int64_t fit = num_cu() * std::min<int64_t>((160 << 10) / (lds + sizeof(a.taps)), 4 * G::kOccupancy / (G::kThreads / 64));
    a.per_wg = G::kWalk ? (int)((tiles + fit - 1) / fit) : 1;
    hipLaunchKernelGGL(kernel, dim3((unsigned)ceil_div(a.ntiles, a.per_wg)), dim3(G::kThreads), lds, st, a, (int)G::image_bytes(a.kh));
    return launch_status();
}

}  // namespace hb
