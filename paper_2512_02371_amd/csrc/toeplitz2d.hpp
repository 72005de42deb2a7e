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
// output with lane shifts, and those additions took as long as the products.
//
// A workgroup is four waves, in general beside each other, and makes ONE tile: while it loads or stores, the others of its
// compute unit multiply, and the dispatcher evens out what they need (walking down a column with the next tile on its way in
// registers took 23.6 us where this takes 19.5).  4096 x 4096, launches back to back, walking and now: hb_conv2d 3 x 3 / 16 x 16 /
// 32 x 32 22.9 / 32.6 / 52.9 -> 20.1 / 26.0 / 51.8 us; hb_down2 of 4 x 4 / 16 x 16 / 32 x 32 taps 20.3 / 23.6 / 42.7 -> 17.4 / 19.5 / 27.3,
// hb_up2 17.8 / 19.0 / 29.8 -> 13.1 / 16.9 / 23.0; a copy of the same bytes takes 18, 9 and 14.  What bounds them now: at 32 x 32
// conv2d the products, with the matrix units busy half of the time (0.43-0.54, clock 1.7-2.1 GHz), and the load and store phases of the
// three workgroups of a compute unit, which they only in part cover; in hb_down2 the loads that all workgroups begin with, in hb_up2
// the stores.  Which tile a call takes: toeplitz2d_tile.hpp.
//
// The window of tile w is the one of tile w - 1 moved by kTileStep pixels, so the chunks are shared:
// per step a wave reads NK weight fragments and about NW + NK chunks for NW NK products.  The LDS rows that one
// read touches are consecutive (rows are dealt to kStride sections) at a pitch of an odd multiple of 16
// bytes: no bank conflicts (an even one doubles them).  Weights come from a zero-padded table of the taps, every row
// in four shifted copies (two in some tiles of hb_down2), so that every run of eight starts on 8 or 16 bytes: a run costs 8 (two 8-byte
// pieces) or 4.8 LDS cycles, against 16 in pieces of 4 bytes (a table of all fragments would take 100 KB).  Chains of products end
// after two steps and are added up outside the matrix unit: error of 32 x 32 taps against fp64 8.5e-8, with chains of 16
// steps 1.6e-7, for 2 us less.
#pragma once
#include <algorithm>

#include "hb_device.hpp"
#include "toeplitz2d_tile.hpp"

namespace hb {

struct T2Args {
    const half_t* in;
    float* out;
    int H, W;                                 // input
    int Ho, Wo;                               // output
    int64_t in_pitch, out_pitch;
    int kh, kw, ay, ax;
    int ncol, nrow, ntiles;                   // workgroup tiles across, down and in all
    int stream;                               // non-temporal stores
    int alias;                                // the staged taps share the image's LDS
    int steps, srows, rows;                   // row offsets s; LDS rows per section, input rows staged
    uint16_t taps[HB_MAX_TAPS_CONV2D * HB_MAX_TAPS_CONV2D];   // kh x kw, row-major
};

typedef u32x4 u32x4_u __attribute__((aligned(4)));
typedef half8 half8_a8 __attribute__((aligned(8)));

constexpr int kT2MinWidth = 8;                // of an image

template <int MODE, int NK, int NW, T2Shape SHAPE>
__global__ void __launch_bounds__((T2Geom<MODE, NK, NW, SHAPE>::kThreads), (T2Geom<MODE, NK, NW, SHAPE>::kOccupancy)) toeplitz2d_mfma_kernel(T2Args p, int table_offset, int taps_offset) {
    using G = T2Geom<MODE, NK, NW, SHAPE>;
    extern __shared__ __attribute__((aligned(16))) char s_dyn[];
    half_t* const s_px = reinterpret_cast<half_t*>(s_dyn);
    half_t* const s_tab = reinterpret_cast<half_t*>(s_dyn + table_offset);
    // the taps come from the kernel arguments in one round trip (the table built straight from there, one gather
    // after the other, took 10 us)
    uint16_t* const s_taps = reinterpret_cast<uint16_t*>(s_dyn + (p.alias ? 0 : taps_offset));

    const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int c = lane & 31, h = lane >> 5, wx = wv % G::kWx, wy = wv / G::kWx;
    // Every XCD takes one contiguous run of tiles, one below the other: neighbours share their halo pixels in one L2.
    // hb_up2, bound by its stores, sweeps along the rows instead, four tiles to an XCD (4096 x 4096, 16 x 16 taps 16.4 -> 14.6 us).
    const int tile = MODE == kT2Up ? xcd_blocked(blockIdx.x, p.ntiles, 4) : xcd_contiguous(blockIdx.x, p.ntiles);
    const int ct = MODE == kT2Up ? tile % p.ncol : tile / p.nrow, rt = MODE == kT2Up ? tile / p.ncol : tile - ct * p.nrow;

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
    const int x0 = (MODE == kT2Conv ? G::kCols * ct : MODE == kT2Down ? 2 * G::kCols * ct : G::kCols / 2 * ct) - p.ax;
    const int y0 = (MODE == kT2Conv ? G::kRows * rt : MODE == kT2Down ? 2 * G::kRows * rt : G::kRows / 2 * rt) - p.ay;
    auto request = [&]() {
        int r = r_first, ch = ch_first;
#pragma unroll
        for (int u = 0; u < G::kPieces; ++u, next_piece(r, ch)) {
            const int row = clampi(y0 + min(r, p.rows - 1), 0, p.H - 1);
            ahead[u] = ldg8(p.in, 2u * ((uint32_t)row * (uint32_t)p.in_pitch + (uint32_t)clampi(x0 + 8 * ch, 0, p.W - 8)));
        }
    };
    auto deliver = [&]() {
        int r = r_first, ch = ch_first;
        const bool inside = x0 >= 0 && x0 + 8 * G::kChunks <= p.W;        // uniform
        if (!inside) {
#pragma unroll
            for (int u = 0; u < G::kPieces; ++u, next_piece(r, ch)) {
                ahead[u] = shift_in_from_right(ahead[u], max(x0 + 8 * ch - (p.W - 8), 0));
                ahead[u] = shift_in_from_left(ahead[u], max(-x0 - 8 * ch, 0));
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
    request();
    lds_barrier();
    // weight table: conv / down row r holds kernel row r - G::kZeroRows; up row 2 (2s + dy) + dx holds the taps
    // 2t + dx of kernel row 2s + dy
    const int tab_rows = MODE == kT2Up ? 2 * p.kh : p.kh + 2 * G::kZeroRows;
    for (int i = tid; i < tab_rows * (G::kCopy / 8); i += G::kThreads) {      // one run of a row in all its copies
        const int r = i / (G::kCopy / 8), j = 8 * (i - r * (G::kCopy / 8));
        const int ry = MODE == kT2Up ? r >> 1 : r - G::kZeroRows;
        half_t run[8 + G::kShift * (G::kCopies - 1)];
#pragma unroll
        for (int k = 0; k < 8 + G::kShift * (G::kCopies - 1); ++k) {
            const int t = j - G::kPad + k, rx = MODE == kT2Up ? 2 * t + (r & 1) : t;
            const bool live = ry >= 0 && ry < p.kh && t >= 0 && rx < p.kw;
            const uint16_t tap = s_taps[live ? ry * p.kw + rx : 0];
            run[k] = live ? __builtin_bit_cast(half_t, tap) : (half_t)0;
        }
#pragma unroll
        for (int q = 0; q < G::kCopies; ++q) {
            half8 v;
#pragma unroll
            for (int k = 0; k < 8; ++k) v[k] = run[k + G::kShift * q];
            *reinterpret_cast<half8*>(s_tab + r * G::kTabRow + q * G::kCopy + j) = v;
        }
    }
    if (p.alias) lds_barrier();                            // the taps lie where the image goes
    deliver();
    lds_barrier();

    // lane (m = c, h): eight weights from window position 16 kk + 8h on; lane (n = c, h): eight pixels from there on
    const int mx = c & 15, mdy = c >> 4;
    const int t0 = 8 * h - (MODE == kT2Conv ? mx : MODE == kT2Down ? 2 * mx : mx >> 1) + G::kPad, t_copy = t0 / G::kShift % G::kCopies;
    const int row0 = MODE == kT2Conv ? G::kZeroRows - mdy : MODE == kT2Down ? G::kZeroRows - 2 * mdy : 2 * mdy + (mx & 1);
    const half_t* const tab = s_tab + row0 * G::kTabRow + t_copy * G::kCopy + t0 - G::kShift * t_copy;
    const int pair = c % G::kPairs, beside = c / G::kPairs;
    const half_t* const px = s_px + (G::kPairs * wy + pair) * G::kPitch + G::kTileStep * NW * (G::kBeside * wx + beside) + 8 * h;
    // stores: lane (n = c, h) holds columns 16 w + 8 (q & 1) + 4h + r of rows 2n + q / 2; a patch turns the 32 rows of
    // one dy into runs of 64 NW bytes
    float* const patch = reinterpret_cast<float*>(s_dyn) + wv * G::kPatch;
    constexpr int kPatchPitch = 16 * NW + 4, kLanes = 4 * NW, kPer = 64 / kLanes;
    const int rr = lane / kLanes, xx = 4 * (lane - rr * kLanes);

    const int xw = G::kCols * ct + 16 * NW * G::kBeside * wx, yw = G::kRows * rt + 2 * G::kPairs * wy;    // the wave's outputs
    const bool active = xw < p.Wo && yw < p.Ho;       // uniform
    floatx16 total[NW];
#pragma unroll
    for (int w = 0; w < NW; ++w) total[w] = floatx16{};
    if (active) {
        struct Frags { half8 a[NK], b[G::kFrags]; };
        auto fetch = [&](int s, Frags& f) {
            const half_t* const trow = tab + s * (MODE == kT2Up ? 4 : 1) * G::kTabRow;
            const half_t* const prow = px + ((s % G::kStride) * p.srows + s / G::kStride) * G::kPitch;
#pragma unroll
            for (int kk = 0; kk < NK; ++kk)
                f.a[kk] = MODE == kT2Down && G::kCopies == 4 ? *reinterpret_cast<const half8*>(trow + 16 * kk) : *reinterpret_cast<const half8_a8*>(trow + 16 * kk);
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
        // Whole runs also where rows are missing, in single floats only where columns are: a tile of 36 of 64 rows stored
        // all of them that way (hb_up2 of 24 x 100000, 4 x 4 taps 19.8 -> 13.9 us, hb_conv2d of 49 x 97000, 3 x 3 13.6 -> 10.4).
        const bool columns = xw + 16 * NW * G::kBeside <= p.Wo, whole = columns && yw + 2 * G::kPairs <= p.Ho;   // uniform
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
                } else if (columns) {
                    if (y < p.Ho) {
                        if (p.stream) __builtin_nontemporal_store(v, reinterpret_cast<floatx4_u*>(dst));
                        else *reinterpret_cast<floatx4_u*>(dst) = v;
                    }
                } else if (y < p.Ho) {
#pragma unroll
                    for (int k = 0; k < 4; ++k)
                        if (x + k < p.Wo) dst[k] = v[k];
                }
            }
            wave_lds_fence();
        }
    }
}

template <int MODE, int NK, int NW, T2Shape SHAPE>
static hb_status t2_launch(T2Args& a, hipStream_t st) {
    using G = T2Geom<MODE, NK, NW, SHAPE>;
    const int64_t tiles = (int64_t)ceil_div(a.Wo, G::kCols) * ceil_div(a.Ho, G::kRows);
    if (tiles > 0x3fffffff) return HB_ERR_UNSUPPORTED;
    // The resampling kernels' runs of 64 and 128 bytes, where they are not whole lines, leave through the L2, which puts
    // neighbours together (4094 x 4094 and 2047 x 2047, 8 x 8 taps: 46 us, streamed 62; smaller outputs, which the
    // memory-side cache takes in, are better streamed: 1078 x 1916 17.9 against 19.6).
    a.stream = MODE == kT2Conv || (a.out_pitch % 32 == 0 && aligned_to(a.out, 128)) || (int64_t)a.Ho * a.Wo * 4 <= (32 << 20);
    a.steps = G::steps(a.kh);
    a.rows = G::rows(a.kh);
    a.srows = G::srows(a.kh);
    a.ncol = ceil_div(a.Wo, G::kCols);
    a.nrow = ceil_div(a.Ho, G::kRows);
    a.ntiles = (int)tiles;
    // the staged taps get LDS of their own where a compute unit holds as many workgroups with it
    const size_t shared = G::lds_bytes(a.kh), taps = ((size_t)a.kh * a.kw * 2 + 15) / 16 * 16;
    a.alias = t2_resident(shared + taps) < t2_resident(shared);
    const size_t lds = a.alias ? shared : shared + taps;
    const auto kernel = toeplitz2d_mfma_kernel<MODE, NK, NW, SHAPE>;
    if (allow_dynamic_lds(reinterpret_cast<const void*>(kernel), lds) != HB_OK) return HB_ERR_HIP;
    hipLaunchKernelGGL(kernel, dim3((unsigned)a.ntiles), dim3(G::kThreads), lds, st, a, (int)G::image_bytes(a.kh), (int)shared);
    return launch_status();
}

}  // namespace hb
