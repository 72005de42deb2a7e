// hb_resize: separable resampling by a non-integer factor with precomputed banded matrices, and
// its vector-ALU twin (Sec. V-C); hb_lanczos3_matrix builds such a matrix on the host.
//
// Each axis is one sparse matrix: row o holds `band` coefficients for the input samples
// start[o] .. start[o] + band - 1.  As in the paper the matrix is treated as block-sparse: the 16
// rows of an aligned group share one starting index (the smallest of theirs, moved down to an even
// sample or a multiple of eight) and the band is widened to cover all of them, at the price of some multiplications by
// zero.  A group of 16 outputs is then a dense 16 x (32 NK) coefficient block, and 16 image rows
// times that block is NK products of the usual kind: the image operand is 8 consecutive samples of
// one row per lane, straight from memory.
//
// Both passes run in one launch (but for large factors, see below).  A wave owns 16 output columns x 16 GY output rows: it applies the
// horizontal matrix to 16 input rows at a time and leaves the result, rounded to fp16, TRANSPOSED in its piece of
// LDS, T[xo][y], where the vertical pass finds its contraction index y contiguous: out^T = T * coef_y^T ends with
// a lane owning four consecutive columns of a row.  (The vector-ALU twin keeps two launches with T in the
// workspace.)
#include <math.h>

#include "hb_device.hpp"
#include "hb_host.hpp"
#include "resize_route.hpp"

namespace hb {

// One pass of the two-launch form and of the vector-ALU twin.
struct BandArgs {
    const half_t* x;                          // [planes][rows][len], row pitch x_pitch, plane stride x_plane
    void* z;                                  // [planes][nout][rows] transposed result, fp16 or fp32
    const int* start;                         // device: nout first input indices
    const half_t* coef;                       // device: nout x band coefficients
    int rows, len, nout, band, planes;
    int64_t x_pitch, x_plane, z_pitch, z_plane;
    int ngroups, nruns;                       // groups of 16 outputs; runs of kRzWaves strips per plane
};

struct ResizeArgs {
    const half_t* in;
    float* out;
    const int *start_x, *start_y;
    const half_t *coef_x, *coef_y;
    int C, H, W, Ho, Wo, band_x, band_y;
    int64_t in_pitch, in_plane, out_pitch, out_plane;
    int ngx, ngy;                             // workgroups across and down
    int first_mask;                           // of a window's first column: ~7 where rows start on 16 bytes, else ~1
};

// Coefficients t .. t + 7 of row o of an n x band matrix, zero outside [0, band).  The neighbouring rows' entries
// that the load covers are masked; only at the two ends of the matrix is it moved and shifted back.
__device__ __forceinline__ half8 rz_coef8(const half_t* m, int n, int band, int o, int t) {
    const int64_t end = (int64_t)n * band - 8, want = (int64_t)o * band + t;
    if (end < 0) {                                        // uniform: fewer than eight entries in all
        half8 f;
#pragma unroll
        for (int i = 0; i < 8; ++i) f[i] = t + i >= 0 && t + i < band ? m[(int64_t)o * band + t + i] : (half_t)0;
        return f;
    }
    const int64_t at = want < 0 ? 0 : want > end ? end : want;
    half8 v = *reinterpret_cast<const half8_u*>(m + at);
    if (at != want) {
        const int d = (int)(want - at);
        v = d > 0 ? shift_in_from_right<true>(v, d) : shift_in_from_left<true>(v, -d);
    }
    u32x4 b = __builtin_bit_cast(u32x4, v);
#pragma unroll
    for (int j = 0; j < 4; ++j)
        b[j] &= ((uint32_t)(t + 2 * j) < (uint32_t)band ? 0xffffu : 0u) | ((uint32_t)(t + 2 * j + 1) < (uint32_t)band ? 0xffff0000u : 0u);
    return __builtin_bit_cast(half8, b);
}
// Smallest lo and largest hi over the 16 lanes of a row, by rotations inside the row (against exchanges through LDS:
// 3 x 1000 x 1000 -> 900 11.5 -> 11.1 us, 4096 x 4096 -> 2048 25.8 -> 25.5).
__device__ __forceinline__ void rz_extent(int& lo, int& hi) {
#define HB_RZ_STEP(n)                                                            \
    lo = min(lo, __builtin_amdgcn_mov_dpp(lo, 0x120 + n, 0xf, 0xf, true));       \
    hi = max(hi, __builtin_amdgcn_mov_dpp(hi, 0x120 + n, 0xf, 0xf, true));
    HB_RZ_STEP(1)
    HB_RZ_STEP(2)
    HB_RZ_STEP(4)
    HB_RZ_STEP(8)
#undef HB_RZ_STEP
}

template <int I>
struct RzInt {
    static constexpr int value = I;
};

// The vertical pass over the rows that T holds from base on.  Text and not a lambda: as a lambda with two callers it has the compiler keep 10
// registers fewer of loads in flight also where there is one (16 x 2946 x 322 -> 283 x 30 18.3 us, 20.9 so; 16 x 2001 x 125 -> 364 x 22 12.3, 14.3).
#define HB_RZ_VERTICAL(base)                                                                                                                         \
    _Pragma("unroll")                                                                                                                                \
    for (int q = 0; q < GY; ++q) {                                                                                                                   \
        const int vsy = __shfl(sy, 16 * q + c, 64), vo = min(yo0 + 16 * q + c, p.Ho - 1);                                                            \
        const int first = ylo + ((__builtin_amdgcn_readlane(glo, 16 * q) - ylo) & ~7); /* 16-byte pieces of T */                                     \
        const int hi = __builtin_amdgcn_readlane(ghi, 16 * q);                                                                                       \
        /* chunks that start in this round, four coefficient loads at a time */                                                                      \
        const int k_first = max(base - first + 31, 0) / 32, k_end = min(hi - first + 31, base + kRows - first + 31) / 32;                            \
        _Pragma("unroll 1")                                                                                                                          \
        for (int k0 = k_first; k0 < k_end; k0 += 4) {                                                                                                \
            half8 f[4];                                                                                                                              \
            _Pragma("unroll")                                                                                                                        \
            for (int k = 0; k < 4; ++k)                                                                                                              \
                if (k0 + k < k_end) f[k] = rz_coef8(p.coef_y, p.Ho, p.band_y, vo, first + 32 * (k0 + k) + 8 * g - vsy);                              \
            _Pragma("unroll")                                                                                                                        \
            for (int k = 0; k < 4; ++k)                                                                                                              \
                if (k0 + k < k_end)                                                                                                                  \
                    out[q] = mfma16x16x32(*reinterpret_cast<const half8*>(rows + c * kPitch + first + 32 * (k0 + k) - base + 8 * g), f[k], out[q]);  \
        }                                                                                                                                            \
    }

// What bounds it: a wave's chain of dependent round trips (starts -> pixels and coefficients -> vertical products ->
// stores) where waves are few, and its instructions (the geometry of a group is 600 of them) where they are many: GY
// groups of rows per wave share them and the rows that neighbouring groups both need.  As two launches with T in
// memory: 3 x 2048 x 2048 -> 450 27.7 -> 19.4 us, 4096 x 4096 -> 2048 36 -> 27, -> 256 39 -> 20.
template <int GY, bool SHARED, bool ODD>
__global__ void __launch_bounds__(64 * RzGeom<SHARED>::kWaves, ODD && !SHARED ? 3 : 4) resize_mfma_kernel(ResizeArgs p) {
    constexpr int kWaves = RzGeom<SHARED>::kWaves, kRows = RzGeom<SHARED>::kRows, kPitch = RzGeom<SHARED>::kPitch;
    __shared__ __attribute__((aligned(16))) half8 s_frag[(ODD ? 2 : 1) * kRzChunks * 64];
    __shared__ __attribute__((aligned(16))) half_t s_rows[(SHARED ? 1 : kWaves) * 16 * kPitch];
    const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int c = lane & 15, g = lane >> 4;
    // workgroups side by side read overlapping pieces of the same rows: walk them back to back inside one XCD
    int wg = xcd_contiguous(blockIdx.x, gridDim.x);
    const int gx = wg % p.ngx;
    wg /= p.ngx;
    const int gy = wg % p.ngy, plane = wg / p.ngy;

    // Columns: the aligned group of 16 outputs shares its first sample and number of 32-sample chunks.  The first sample
    // is even and, where that takes no chunk more, a multiple of eight, so that loads of aligned rows are aligned
    // (3 x 2048 x 2048 -> 450 16.9 -> 15.0 us).  A
    // start below -band (above len - 1) reads nothing but the first (last) sample, and so does
    // -band (len - 1): clamping it there changes no result and bounds the span by the image.
    const int xo = min(16 * gx + c, p.Wo - 1);            // lanes beyond Wo repeat the last output and store nothing
    const int sx = clampi(p.start_x[xo], -p.band_x, p.W - 1);
    // Rows: lane c + 16 q holds the start of output row c of the wave's group q
    const int yo0 = 16 * GY * (SHARED ? gy : kWaves * gy + wv);
    const int sy = clampi(p.start_y[min(yo0 + (lane & (16 * GY - 1)), p.Ho - 1)], -p.band_y, p.H - 1);
    int xlo = sx, xhi = sx + p.band_x;
    rz_extent(xlo, xhi);
    // ODD: the rows that start on an odd sample are read from one sample further left
    xlo = (__builtin_amdgcn_readfirstlane(xlo) & ~1) - (ODD ? 1 : 0);
    xhi = __builtin_amdgcn_readfirstlane(xhi);
    const int nk = (xhi - xlo + 31) >> 5, aligned = xlo & p.first_mask;
    if (!ODD && xhi - aligned <= 32 * nk) xlo = aligned;
    int glo = sy, ghi = sy + p.band_y;                    // of the lane's group of 16 rows
    rz_extent(glo, ghi);
    int ylo = glo, yhi = ghi;
#pragma unroll
    for (int off = 16; off < 16 * GY; off <<= 1) {
        ylo = min(ylo, __shfl_xor(ylo, off, 64));
        yhi = max(yhi, __shfl_xor(yhi, off, 64));
    }
    ylo = __builtin_amdgcn_readfirstlane(ylo);
    yhi = __builtin_amdgcn_readfirstlane(yhi);

    // coefficient blocks, B-operand layout: lane (c = o, g) holds coef[o][first + 32 kk + 8g + i - start[o]]
    const int x_even = xlo + (ODD ? 1 : 0);
    auto frag_x = [&](int kk) { return rz_coef8(p.coef_x, p.Wo, p.band_x, xo, x_even + 32 * kk + 8 * g - sx); };
    for (int kk = wv; kk < min(nk, kRzChunks); kk += kWaves) s_frag[kk * 64 + lane] = frag_x(kk);
    if constexpr (ODD)
        for (int kk = kWaves - 1 - wv; kk < min(nk, kRzChunks); kk += kWaves)
            s_frag[(kRzChunks + kk) * 64 + lane] = rz_coef8(p.coef_x, p.Wo, p.band_x, xo, xlo + 32 * kk + 8 * g - sx);

    const half_t* const px = p.in + (int64_t)plane * p.in_plane;
    half_t* const rows = s_rows + (SHARED ? 0 : wv * 16 * kPitch);        // T
    floatx4 out[GY];
#pragma unroll
    for (int q = 0; q < GY; ++q) out[q] = floatx4{0.f, 0.f, 0.f, 0.f};
    auto load = [&](int y, int kk) {                      // chunk kk of row y
        const uint32_t row = (uint32_t)clampi(y, 0, p.H - 1) * (uint32_t)p.in_pitch;
        const int xs = x_even + 32 * kk, x = xs + 8 * g;
        if (xs >= 0 && xs + 32 <= p.W) return ldg8(px, 2u * (row + (uint32_t)x));     // uniform
        // Requested inside the row, then shifted into place.  The column is hidden from the compiler, which otherwise works
        // out the masks of all four chunks' shifts ahead of the loop, also for groups inside the image, and spills 40 scalar
        // registers over them (250 calls on 64 to 4096 rows and columns, factors up to 16: 6 % faster on average, none slower).
        int xe = x;
        asm volatile("" : "+v"(xe));
        const half8 v = ldg8(px, 2u * (row + (uint32_t)clampi(xe, 0, p.W - 8)));
        return shift_in_from_left(shift_in_from_right(v, max(xe - (p.W - 8), 0)), max(-xe, 0));
    };
    auto rows_ready = [&]() {
        if (SHARED) __syncthreads();
        else wave_lds_fence();
    };
    const int t_first = SHARED ? wv : 0, t_step = SHARED ? kWaves : 1;    // row tiles of this wave
    __syncthreads();
    if (yo0 >= p.Ho) return;                              // SHARED: no such workgroup

    // ODD: rows start on even and odd samples in turn, and of a row read from an odd one on every lane's 16 bytes are several cache
    // accesses.  Here the even and the odd rows of 32 are two operands, each of which is read from whole dwords with coefficients that
    // start where its window does; what they give is put together again on its way to T (3 x 1912 x 2923 -> 671 x 1025 39.3 -> 25.9 us).
    // For groups inside the rows whose rows fit T, the others take the general loop.
    auto short_loop = [&](auto chunks, int base, int tiles) {
        constexpr int NK = decltype(chunks)::value, kAhead = 2;       // units of 32 rows in flight
        const int first_odd = (int)((reinterpret_cast<uintptr_t>(px) >> 1) + (uintptr_t)(intptr_t)base) & 1;    // row base starts on an odd sample
        // (hidden from the compiler, which otherwise works out the addresses of all four loops ahead of the first)
        int l = lane;
        asm volatile("" : "+v"(l));
        const int lc = l & 15, lg = l >> 4;
        half8 f[2][NK];
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int k = 0; k < NK; ++k) f[u][k] = s_frag[((u ^ first_odd) ? kRzChunks + k : k) * 64 + l];
        half8 d[kAhead][2][NK];
        auto request = [&](int t, half8 (&to)[2][NK]) {
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                const int y = base + 32 * t + 2 * lc + u, xs = x_even - (u ^ first_odd);
                const uint32_t at = (uint32_t)clampi(y, 0, p.H - 1) * (uint32_t)p.in_pitch + (uint32_t)(xs + 8 * lg);
                const char* const q = reinterpret_cast<const char*>(px) + (uint64_t)(2u * at);
#pragma unroll
                for (int k = 0; k < NK; ++k) to[u][k] = *reinterpret_cast<const half8_u*>(q + 64 * k);
            }
        };
        const int units = tiles / 2;
#pragma unroll
        for (int a = 0; a < kAhead; ++a)
            if (t_first + a * t_step < units) request(t_first + a * t_step, d[a]);
#pragma unroll 1
        for (int t = t_first; t < units; t += kAhead * t_step) {
#pragma unroll
            for (int a = 0; a < kAhead; ++a) {
                const int ta = t + a * t_step;
                if (ta >= units) break;
                floatx4 acc[2];
#pragma unroll
                for (int u = 0; u < 2; ++u) {
                    acc[u] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                    for (int k = 0; k < NK; ++k) acc[u] = mfma16x16x32(d[a][u][k], f[u][k], acc[u]);
                }
                if (ta + kAhead * t_step < units) request(ta + kAhead * t_step, d[a]);
                half8 h;                                  // rows 8g .. 8g + 7 of the unit
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    h[2 * j] = (half_t)acc[0][j];
                    h[2 * j + 1] = (half_t)acc[1][j];
                }
                *reinterpret_cast<half8*>(rows + lc * kPitch + 32 * ta + 8 * lg) = h;
            }
        }
    };
    // The same for five chunks and more: up to four of them at a time, the next ones in flight, coefficients from LDS.
    auto long_loop = [&](int base, int tiles) {
        const int first_odd = (int)((reinterpret_cast<uintptr_t>(px) >> 1) + (uintptr_t)(intptr_t)base) & 1, units = tiles / 2;
        int l = lane;
        asm volatile("" : "+v"(l));
        const int lc = l & 15, lg = l >> 4;
        auto request = [&](int t, int k0, half8 (&to)[2][4]) {
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                const int y = base + 32 * t + 2 * lc + u, xs = x_even - (u ^ first_odd) + 32 * k0;
                const uint32_t at = (uint32_t)clampi(y, 0, p.H - 1) * (uint32_t)p.in_pitch + (uint32_t)(xs + 8 * lg);
                const char* const q = reinterpret_cast<const char*>(px) + (uint64_t)(2u * at);
#pragma unroll
                for (int k = 0; k < 4; ++k)
                    if (k0 + k < nk) to[u][k] = *reinterpret_cast<const half8_u*>(q + 64 * k);        // uniform
            }
        };
        floatx4 acc[2] = {floatx4{0.f, 0.f, 0.f, 0.f}, floatx4{0.f, 0.f, 0.f, 0.f}};
        auto use = [&](int t, int k0, const half8 (&d)[2][4]) {
#pragma unroll
            for (int k = 0; k < 4; ++k)
                if (k0 + k < nk) {
#pragma unroll
                    for (int u = 0; u < 2; ++u) acc[u] = mfma16x16x32(d[u][k], s_frag[((u ^ first_odd) * kRzChunks + k0 + k) * 64 + l], acc[u]);
                }
            if (k0 + 4 < nk) return;
            half8 h;                                      // rows 8g .. 8g + 7 of the unit
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                h[2 * j] = (half_t)acc[0][j];
                h[2 * j + 1] = (half_t)acc[1][j];
            }
            *reinterpret_cast<half8*>(rows + lc * kPitch + 32 * t + 8 * lg) = h;
            acc[0] = acc[1] = floatx4{0.f, 0.f, 0.f, 0.f};
        };
        auto advance = [&](int& t, int& k0) {
            k0 += 4;
            if (k0 >= nk) {
                k0 = 0;
                t += t_step;
            }
        };
        half8 d0[2][4], d1[2][4];
        int t = t_first, k0 = 0;
        if (t < units) request(t, k0, d0);
#pragma unroll 1
        while (t < units) {
            int tn = t, kn = k0;
            advance(tn, kn);
            if (tn < units) request(tn, kn, d1);
            use(t, k0, d0);
            if (tn >= units) break;
            t = tn;
            k0 = kn;
            advance(t, k0);
            if (t < units) request(t, k0, d0);
            use(tn, kn, d1);
        }
    };
    int from = ylo;                                       // row
    const bool short_group = ODD && xlo >= 0 && x_even + 32 * nk <= p.W && yhi - ylo <= kRows && nk <= kRzChunks;    // uniform
    if constexpr (ODD) {
        if (short_group) {
            const int base = ylo, tiles = (yhi - base + 31) / 32 * 2;
            if (!SHARED || wv == 0) *reinterpret_cast<half8*>(rows + c * kPitch + 16 * tiles + 8 * g) = half8{};
            if (nk == 1) short_loop(RzInt<1>{}, base, tiles);
            else if (nk == 2) short_loop(RzInt<2>{}, base, tiles);
            else if (nk == 3) short_loop(RzInt<3>{}, base, tiles);
            else if (nk == 4) short_loop(RzInt<4>{}, base, tiles);
            else long_loop(base, tiles);
            rows_ready();
            if (!SHARED || wv == 0) {
                HB_RZ_VERTICAL(base)
            }
            from = yhi;
        }
    }
#pragma unroll 1
    for (int base = from; base < yhi; base += kRows) {
        // T of rows base .. base + rows - 1; a chunk of the vertical pass that starts before base + kRows may reach
        // 32 rows further, real ones or, after the last, zeros
        const bool last = yhi - base <= kRows;
        const int tiles = last ? (yhi - base + 15) / 16 : (kRows + 32) / 16;
        rows_ready();                                     // the previous rows are read
        if (last && (!SHARED || wv == 0)) *reinterpret_cast<half8*>(rows + c * kPitch + 16 * tiles + 8 * g) = half8{};
        // D[m = y][n = xo]: lane (c = xo, g) holds rows 4g .. 4g + 3
        auto keep = [&](int t, const floatx4& acc) {
            *reinterpret_cast<half4*>(rows + c * kPitch + 16 * t + 4 * g) = to_half4(acc);
        };
        if (nk <= kRzChunks) {
            // up to four chunks of a tile are one piece of work; the next piece is requested before the current one
            // is multiplied
            auto request = [&](int t, int k0, half8 (&d)[4]) {
#pragma unroll
                for (int k = 0; k < 4; ++k)
                    if (k0 + k < nk) d[k] = load(base + 16 * t + c, k0 + k);          // uniform
            };
            floatx4 acc = {0.f, 0.f, 0.f, 0.f};
            half8 cur[4], nxt[4];
            int t = t_first, k0 = 0;
            if (t < tiles) request(t, 0, cur);
#pragma unroll 1
            while (t < tiles) {
                const bool end = k0 + 4 >= nk;
                const int t1 = end ? t + t_step : t, k1 = end ? 0 : k0 + 4;
                if (t1 < tiles) request(t1, k1, nxt);
#pragma unroll
                for (int k = 0; k < 4; ++k)
                    if (k0 + k < nk) acc = mfma16x16x32(cur[k], s_frag[(k0 + k) * 64 + lane], acc);
                if (end) {
                    keep(t, acc);
                    acc = floatx4{0.f, 0.f, 0.f, 0.f};
                }
                t = t1;
                k0 = k1;
#pragma unroll
                for (int k = 0; k < 4; ++k) cur[k] = nxt[k];
            }
        } else {                                          // spans of more than 384 columns: no room for the block
#pragma unroll 1
            for (int t = t_first; t < tiles; t += t_step) {
                floatx4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
                for (int kk = 0; kk < nk; ++kk) acc = mfma16x16x32(load(base + 16 * t + c, kk), frag_x(kk), acc);
                keep(t, acc);
            }
        }
        rows_ready();
        if (SHARED && wv != 0) continue;
        HB_RZ_VERTICAL(base)
    }
    if (SHARED && wv != 0) return;
    // D[m = xo][n = yo]: lane (c = yo, g) holds columns 4g .. 4g + 3 of its row
#pragma unroll
    for (int q = 0; q < GY; ++q) {
        const int yo = yo0 + 16 * q + c, x = 16 * gx + 4 * g;
        if (yo < p.Ho && x < p.Wo)
            store4_mask(p.out + (int64_t)plane * p.out_plane + (int64_t)yo * p.out_pitch, x, p.Wo, out[q]);
    }
}

#undef HB_RZ_VERTICAL

// ---------------------------------------------------------------------------
// The two-launch form for large factors: one kernel that contracts over the memory-contiguous index of its input and
// writes its result TRANSPOSED, Z[o][r] = sum_j X[r][start[o] + j] coef[o][j], run once per axis with T in the
// workspace.  A wave owns 64 rows of X and one group of 16 outputs, so the pixels of a wide span are read once per
// group whatever the rows' matrix is, by as many waves as the image has rows.
constexpr int kRzTiles = 4;                   // 16-row tiles of X per wave (64 rows r)
constexpr int kRzWaves = 2;                   // waves per workgroup: 2 strips of 64 rows, one group of 16 outputs (measured: 1, 4, 8 are slower)
constexpr int kRzMaxChunks = HB_RESIZE_MAX_SPAN / 32;

// Sixteen rows of 64 floats from the accumulators (lane (c, g): row c, columns 16 w + 4 g ..) to
// fp16 rows in memory, through the wave's LDS patch so that a row leaves as one 128-byte run.
template <int NW>
__device__ __forceinline__ void rz_store_rows_half(float* patch, half_t* dst, uint32_t pitch_elems,
                                                   const floatx4 (&acc)[NW], int lane) {
    const int c = lane & 15, g = lane >> 4;
#pragma unroll
    for (int w = 0; w < NW; ++w)
        *reinterpret_cast<floatx4*>(patch + c * RowPatch<NW>::kPitch + 16 * w + 4 * g) = acc[w];
    wave_lds_fence();
    constexpr int kLanesPerRow = 4 * NW, kRowsPerPass = 64 / kLanesPerRow;
    const int rr = lane / kLanesPerRow, xq = lane - rr * kLanesPerRow;
#pragma unroll
    for (int s = 0; s < 16 / kRowsPerPass; ++s) {
        const int row = s * kRowsPerPass + rr;
        const floatx4 v = *reinterpret_cast<const floatx4*>(patch + row * RowPatch<NW>::kPitch + 4 * xq);
        const half4 h = {(half_t)v[0], (half_t)v[1], (half_t)v[2], (half_t)v[3]};
        *reinterpret_cast<half4_u*>(dst + (size_t)row * pitch_elems + 4 * xq) = h;
    }
    wave_lds_fence();
}

template <bool OUT_HALF>
__global__ void __launch_bounds__(64 * kRzWaves) band_mfma_kernel(BandArgs p) {
    constexpr int NW = kRzTiles;
    // The coefficient block and, once the products are done, the waves' store patches share one piece
    // of LDS: with both resident a compute unit held too few workgroups to cover the grid in one round.
    constexpr int kFragBytes = kRzMaxChunks * 64 * 16, kPatchBytes = kRzWaves * RowPatch<NW>::kFloats * 4;
    __shared__ __attribute__((aligned(16))) char s_mem[kFragBytes > kPatchBytes ? kFragBytes : kPatchBytes];
    half8* s_frag = reinterpret_cast<half8*>(s_mem);
    float* s_patch = reinterpret_cast<float*>(s_mem);

    const int tid = threadIdx.x;
    const int lane = tid & 63, wv = tid >> 6;
    const int c = lane & 15, g = lane >> 4;
    // neighbouring groups read neighbouring pieces of the same rows: walk them back to back inside one XCD
    int wg = xcd_contiguous(blockIdx.x, gridDim.x);
    const int grp = wg % p.ngroups;
    wg /= p.ngroups;
    const int run = wg % p.nruns, plane = wg / p.nruns;
    const int o0 = 16 * grp;

    // geometry of the group: first sample (even) and number of 32-sample chunks.  Lane column c
    // reads the start of output o0 + c; the minimum and maximum over the 16 columns come from four
    // butterfly steps inside each row of 16 lanes, so every lane ends up with the same numbers.
    // A start below -band (above len - 1) reads nothing but the first (last) sample, and so does
    // -band (len - 1): clamping it there changes no result and bounds the span by the image.
    const int o = o0 + c;
    const bool live = o < p.nout;
    const int st = live ? clampi(p.start[o], -p.band, p.len - 1) : 0;
    int lo = live ? st : 0x7fffffff, hi = live ? st + p.band : -0x7fffffff;
#pragma unroll
    for (int off = 1; off < 16; off <<= 1) {
        lo = min(lo, __shfl_xor(lo, off, 64));
        hi = max(hi, __shfl_xor(hi, off, 64));
    }
    const int first = lo & ~1, nk_all = (hi - first + 31) / 32;

    const int r0 = 64 * (kRzWaves * run + wv);            // this wave's strip of rows
    const bool active = r0 < p.rows;
    const half_t* xpl = p.x + (size_t)plane * p.x_plane;
    const uint32_t rowbytes = (uint32_t)p.x_pitch * 2u;
    uint32_t rowoff[NW];
#pragma unroll
    for (int w = 0; w < NW; ++w) rowoff[w] = (uint32_t)min(r0 + 16 * w + c, p.rows - 1) * rowbytes;

    auto load_chunk = [&](int kk, half8 (&d)[NW]) {
        const int xs = first + 32 * kk;                   // uniform
        if (xs >= 0 && xs + 32 <= p.len) {
#pragma unroll
            for (int w = 0; w < NW; ++w) d[w] = ldg8(xpl, rowoff[w] + 2u * (uint32_t)(xs + 8 * g));
        } else {
#pragma unroll
            for (int w = 0; w < NW; ++w)
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    const int x = clampi(xs + 8 * g + i, 0, p.len - 1);
                    d[w][i] = *reinterpret_cast<const half_t*>(reinterpret_cast<const char*>(xpl) + (rowoff[w] + 2u * (uint32_t)x));
                }
        }
    };
    floatx4 acc[NW];
#pragma unroll
    for (int w = 0; w < NW; ++w) acc[w] = floatx4{0.f, 0.f, 0.f, 0.f};
    half8 bufa[NW], bufb[NW];
    // The coefficient block holds kRzMaxChunks chunks; a group that spans more (a very large factor,
    // or starts that jump inside the group) takes several rounds of block + products.
    for (int base = 0; base < nk_all; base += kRzMaxChunks) {
        const int nk = min(nk_all - base, kRzMaxChunks);
        if (base) __syncthreads();                        // every wave is done with the previous block
        // the first window chunk is requested before the coefficient block is built
        if (active) load_chunk(base, bufa);

        // coefficient block, B-operand layout: lane (c = o, g) holds B[8g + i][o] = coef[o][first + 32 kk + 8g + i - start[o]];
        // wave wv builds chunks wv, wv + kRzWaves, ...
        for (int kk = wv; kk < nk; kk += kRzWaves) {
            half8 f;
#pragma unroll
            for (int i = 0; i < 8; ++i) f[i] = (half_t)0;
            if (live) {
                const int t0 = first + 32 * (base + kk) + 8 * g - st;
                const half_t* row = p.coef + (size_t)o * p.band;
#pragma unroll
                for (int i = 0; i < 8; ++i)
                    if (t0 + i >= 0 && t0 + i < p.band) f[i] = row[t0 + i];
            }
            s_frag[kk * 64 + lane] = f;
        }
        __syncthreads();

        // two window buffers used alternately: the next chunk is in flight while this one is multiplied
        auto use_chunk = [&](int kk, const half8 (&d)[NW]) {
            const half8 f = s_frag[kk * 64 + lane];
#pragma unroll
            for (int w = 0; w < NW; ++w) acc[w] = mfma16x16x32(d[w], f, acc[w]);
        };
        for (int kk = 0; active && kk < nk; kk += 2) {
            if (kk + 1 < nk) load_chunk(base + kk + 1, bufb);
            use_chunk(kk, bufa);
            if (kk + 1 >= nk) break;
            if (kk + 2 < nk) load_chunk(base + kk + 2, bufa);
            use_chunk(kk + 1, bufb);
        }
    }
    __syncthreads();                                      // every wave is done with the coefficient block
    if (!active) return;

    // D[m = r][n = o]: lane (c = o, g) holds rows r0 + 16 w + 4 g .. + 3 = four consecutive elements of Z's row o
    float* patch = s_patch + wv * RowPatch<NW>::kFloats;
    const bool whole = o0 + 16 <= p.nout && r0 + 64 <= p.rows;
    if (OUT_HALF) {
        half_t* z = reinterpret_cast<half_t*>(p.z) + (size_t)plane * p.z_plane;
        if (whole) {
            rz_store_rows_half<NW>(patch, z + (size_t)o0 * p.z_pitch + r0, (uint32_t)p.z_pitch, acc, lane);
        } else if (o0 + c < p.nout) {
            half_t* row = z + (size_t)(o0 + c) * p.z_pitch;
#pragma unroll
            for (int w = 0; w < NW; ++w)
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const int r = r0 + 16 * w + 4 * g + j;
                    if (r < p.rows) row[r] = (half_t)acc[w][j];
                }
        }
    } else {
        float* z = reinterpret_cast<float*>(p.z) + (size_t)plane * p.z_plane;
        if (whole) {
            store_rows_via_lds<NW, true>(patch, z + (size_t)o0 * p.z_pitch + r0, (uint32_t)p.z_pitch, acc, lane);
        } else if (o0 + c < p.nout) {
            float* row = z + (size_t)(o0 + c) * p.z_pitch;
#pragma unroll
            for (int w = 0; w < NW; ++w) store4_mask(row, r0 + 16 * w + 4 * g, p.rows, acc[w]);
        }
    }
}

// Vector-ALU twin of one pass.  A workgroup takes one group of 16 outputs and 64 rows of X: the samples
// the group reads (from its smallest start on, 256 at a time, every index clamped) are staged in LDS
// with coalesced row loads; a thread owns one output o and four rows, reads a coefficient once and
// uses it for its four rows; the four results are consecutive elements of row o of the transposed Z.
constexpr int kRzvChunk = 256;                // staged samples per row and round
constexpr int kRzvPitch = kRzvChunk + 8;      // halves

template <bool OUT_HALF>
__global__ void __launch_bounds__(256) band_valu_kernel(BandArgs p) {
    __shared__ __attribute__((aligned(16))) half_t s_x[64 * kRzvPitch];
    const int tid = threadIdx.x;
    int wg = blockIdx.x;
    const int grp = wg % p.ngroups;
    wg /= p.ngroups;
    const int nblk = (p.rows + 63) / 64;
    const int blk = wg % nblk, plane = wg / nblk;
    const int r0 = 64 * blk;
    const int o = 16 * grp + (tid & 15), rq = tid >> 4;
    const bool live = o < p.nout;
    const int st = live ? clampi(p.start[o], -p.band, p.len - 1) : 0;   // same samples as the unclamped start
    int lo = live ? st : 0x7fffffff, hi = live ? st + p.band : -0x7fffffff;
#pragma unroll
    for (int off = 1; off < 16; off <<= 1) {
        lo = min(lo, __shfl_xor(lo, off, 64));
        hi = max(hi, __shfl_xor(hi, off, 64));
    }
    const half_t* xpl = p.x + (size_t)plane * p.x_plane;
    const half_t* k = p.coef + (size_t)(live ? o : 0) * p.band;
    float acc[4] = {0.f, 0.f, 0.f, 0.f};
    for (int base = lo; base < hi; base += kRzvChunk) {
        const int n = min(kRzvChunk, hi - base);          // samples of this round
        const int nch = (n + 7) / 8;
        if (base != lo) __syncthreads();                  // everyone is done with the previous round
        for (int idx = tid; idx < 64 * nch; idx += 256) {
            const int r = idx / nch, ch = idx - r * nch;
            const half_t* row = xpl + (size_t)min(r0 + r, p.rows - 1) * p.x_pitch;
            *reinterpret_cast<half8*>(&s_x[r * kRzvPitch + 8 * ch]) = load8_clamp(row, base + 8 * ch, p.len);
        }
        __syncthreads();
        if (live) {
            const int j0 = max(0, base - st), j1 = min(p.band, base + n - st);
            for (int j = j0; j < j1; ++j) {
                const float c = (float)k[j];
                const half_t* src = &s_x[4 * rq * kRzvPitch + (st + j - base)];
#pragma unroll
                for (int q = 0; q < 4; ++q) acc[q] = fmaf(c, (float)src[q * kRzvPitch], acc[q]);
            }
        }
    }
    if (!live) return;
    const int r = r0 + 4 * rq;
    if (OUT_HALF) {
        half_t* z = reinterpret_cast<half_t*>(p.z) + (size_t)plane * p.z_plane + (size_t)o * p.z_pitch;
#pragma unroll
        for (int q = 0; q < 4; ++q)
            if (r + q < p.rows) z[r + q] = (half_t)acc[q];
    } else {
        float* z = reinterpret_cast<float*>(p.z) + (size_t)plane * p.z_plane + (size_t)o * p.z_pitch;
#pragma unroll
        for (int q = 0; q < 4; ++q)
            if (r + q < p.rows) z[r + q] = acc[q];
    }
}

static int64_t rz_pitch(int H) { return ((int64_t)H + 7) & ~(int64_t)7; }

static hb_status resize_run(bool valu, const hb_half* in, float* out, void* workspace, size_t workspace_bytes,
                            int C, int H, int W, int Ho, int Wo,
                            int64_t in_pitch, int64_t in_plane, int64_t out_pitch, int64_t out_plane,
                            const int32_t* start_y, const hb_half* coef_y, int band_y,
                            const int32_t* start_x, const hb_half* coef_x, int band_x, hb_stream stream) {
    if (!in || !out || !start_y || !coef_y || !start_x || !coef_x) return HB_ERR_INVALID_ARG;
    if (C < 1 || H < 1 || W < 1 || Ho < 1 || Wo < 1) return HB_ERR_INVALID_ARG;
    if (band_y < 1 || band_x < 1 || band_y > HB_RESIZE_MAX_SPAN || band_x > HB_RESIZE_MAX_SPAN) return HB_ERR_INVALID_ARG;
    if (in_pitch < W || out_pitch < Wo) return HB_ERR_INVALID_ARG;
    if (C > 1 && (in_plane < (int64_t)H * in_pitch || out_plane < (int64_t)Ho * out_pitch)) return HB_ERR_INVALID_ARG;
    if (!aligned_to(in, 2) || !aligned_to(out, 4) || !aligned_to(start_y, 4) || !aligned_to(start_x, 4) ||
        !aligned_to(coef_y, 2) || !aligned_to(coef_x, 2))
        return HB_ERR_INVALID_ARG;
    const int64_t hp = rz_pitch(H);
    // lanes address the rows of a plane with 32-bit byte offsets
    if ((int64_t)H * in_pitch >= ((int64_t)1 << 31) || (int64_t)Wo * hp >= ((int64_t)1 << 31) ||
        (int64_t)Ho * out_pitch >= ((int64_t)1 << 30) || C > 65535)
        return HB_ERR_UNSUPPORTED;
    const size_t need = hb_resize_workspace_size(C, H, Wo);
    if (!workspace || workspace_bytes < need || !aligned_to(workspace, 256)) return HB_ERR_WORKSPACE;
    hipStream_t st = reinterpret_cast<hipStream_t>(stream);

    const RzRoute route = rz_route({C, H, W, Ho, Wo, band_y, band_x, in_pitch, in_pitch % 2 == 0 && (C == 1 || in_plane % 2 == 0) && aligned_to(in, 4),
                                    out_pitch % 32 == 0 && out_plane % 32 == 0 && aligned_to(out, 128), num_cu()});
    if (!valu && route.one_launch) {
        ResizeArgs r;
        r.in = reinterpret_cast<const half_t*>(in);
        r.out = out;
        r.start_x = start_x;
        r.start_y = start_y;
        r.coef_x = reinterpret_cast<const half_t*>(coef_x);
        r.coef_y = reinterpret_cast<const half_t*>(coef_y);
        r.C = C;
        r.H = H;
        r.W = W;
        r.Ho = Ho;
        r.Wo = Wo;
        r.band_x = band_x;
        r.band_y = band_y;
        r.in_pitch = in_pitch;
        r.in_plane = in_plane;
        r.out_pitch = out_pitch;
        r.out_plane = out_plane;
        r.ngx = ceil_div(Wo, 16);
        r.first_mask = in_pitch % 8 == 0 && (C == 1 || in_plane % 8 == 0) && aligned_to(in, 16) ? ~7 : ~1;
        const int gq = route.groups, groups = ceil_div(Ho, 16);
        r.ngy = gq ? ceil_div(groups, gq * RzGeom<false>::kWaves) : groups;
        const int64_t blocks = (int64_t)C * r.ngx * r.ngy;
        if (blocks > 0x7fffffff) return HB_ERR_UNSUPPORTED;
        const dim3 grid((unsigned)blocks), block(64 * RzGeom<false>::kWaves);
        auto launch = [&](auto odd) {
            constexpr bool ODD = decltype(odd)::value != 0;
            if (gq == 4) hipLaunchKernelGGL((resize_mfma_kernel<4, false, ODD>), grid, block, 0, st, r);
            else if (gq == 2) hipLaunchKernelGGL((resize_mfma_kernel<2, false, ODD>), grid, block, 0, st, r);
            else if (gq == 1) hipLaunchKernelGGL((resize_mfma_kernel<1, false, ODD>), grid, block, 0, st, r);
            else hipLaunchKernelGGL((resize_mfma_kernel<1, true, ODD>), grid, dim3(64 * RzGeom<true>::kWaves), 0, st, r);
        };
        if (route.apart) launch(RzInt<1>{});
        else launch(RzInt<0>{});
        return launch_status();
    }

    BandArgs a;
    // horizontal: image rows y, contraction over x, result T^T[xo][y] in fp16
    a.x = reinterpret_cast<const half_t*>(in);
    a.z = workspace;
    a.start = start_x;
    a.coef = reinterpret_cast<const half_t*>(coef_x);
    a.rows = H;
    a.len = W;
    a.nout = Wo;
    a.band = band_x;
    a.planes = C;
    a.x_pitch = in_pitch;
    a.x_plane = in_plane;
    a.z_pitch = hp;
    a.z_plane = (int64_t)Wo * hp;
    BandArgs b;
    // vertical: rows of T^T, contraction over y, result out[yo][xo] in fp32
    b.x = reinterpret_cast<const half_t*>(workspace);
    b.z = out;
    b.start = start_y;
    b.coef = reinterpret_cast<const half_t*>(coef_y);
    b.rows = Wo;
    b.len = H;
    b.nout = Ho;
    b.band = band_y;
    b.planes = C;
    b.x_pitch = hp;
    b.x_plane = (int64_t)Wo * hp;
    b.z_pitch = out_pitch;
    b.z_plane = out_plane;
    const bool matrix = !valu && W >= kRzMinWidth;
    for (BandArgs* q : {&a, &b}) {
        q->ngroups = ceil_div(q->nout, 16);
        q->nruns = ceil_div(q->rows, 64 * kRzWaves);
        const int64_t blocks = (int64_t)q->planes * q->ngroups * (matrix ? q->nruns : ceil_div(q->rows, 64));
        if (blocks > 0x7fffffff) return HB_ERR_UNSUPPORTED;
        const dim3 grid((unsigned)blocks), block(matrix ? 64 * kRzWaves : 256);
        if (matrix && q == &a) hipLaunchKernelGGL(band_mfma_kernel<true>, grid, block, 0, st, *q);
        else if (matrix) hipLaunchKernelGGL(band_mfma_kernel<false>, grid, block, 0, st, *q);
        else if (q == &a) hipLaunchKernelGGL(band_valu_kernel<true>, grid, block, 0, st, *q);
        else hipLaunchKernelGGL(band_valu_kernel<false>, grid, block, 0, st, *q);
        const hb_status s = launch_status();
        if (s != HB_OK) return s;
    }
    return HB_OK;
}

}  // namespace hb

extern "C" size_t hb_resize_workspace_size(int C, int H, int Wo) {
    if (C < 1 || H < 1 || Wo < 1) return 0;
    return (size_t)C * (size_t)Wo * (size_t)hb::rz_pitch(H) * sizeof(uint16_t);
}

extern "C" hb_status hb_resize(const hb_half* in, float* out, void* workspace, size_t workspace_bytes,
                               int C, int H, int W, int Ho, int Wo,
                               int64_t in_pitch, int64_t in_plane, int64_t out_pitch, int64_t out_plane,
                               const int32_t* start_y, const hb_half* coef_y, int band_y,
                               const int32_t* start_x, const hb_half* coef_x, int band_x, hb_stream stream) {
    return hb::resize_run(false, in, out, workspace, workspace_bytes, C, H, W, Ho, Wo, in_pitch, in_plane, out_pitch,
                          out_plane, start_y, coef_y, band_y, start_x, coef_x, band_x, stream);
}

extern "C" hb_status hb_resize_valu(const hb_half* in, float* out, void* workspace, size_t workspace_bytes,
                                    int C, int H, int W, int Ho, int Wo,
                                    int64_t in_pitch, int64_t in_plane, int64_t out_pitch, int64_t out_plane,
                                    const int32_t* start_y, const hb_half* coef_y, int band_y,
                                    const int32_t* start_x, const hb_half* coef_x, int band_x, hb_stream stream) {
    return hb::resize_run(true, in, out, workspace, workspace_bytes, C, H, W, Ho, Wo, in_pitch, in_plane, out_pitch,
                          out_plane, start_y, coef_y, band_y, start_x, coef_x, band_x, stream);
}

extern "C" int hb_lanczos3_band(int n_in, int n_out) {
    if (n_in < 1 || n_out < 1 || n_out > n_in) return 0;
    return (int)floor(6.0 * (double)n_in / (double)n_out) + 1;
}

extern "C" hb_status hb_lanczos3_matrix(int n_in, int n_out, int32_t* start_host, hb_half* coef_host) {
    const int band = hb_lanczos3_band(n_in, n_out);
    if (band == 0 || !start_host || !coef_host) return HB_ERR_INVALID_ARG;
    if (band > HB_RESIZE_MAX_SPAN) return HB_ERR_UNSUPPORTED;
    const double pi = 3.14159265358979323846, scale = (double)n_in / (double)n_out;
    double w[HB_RESIZE_MAX_SPAN];
    for (int o = 0; o < n_out; ++o) {
        const double centre = (o + 0.5) * scale - 0.5;
        const int first = (int)ceil(centre - 3.0 * scale);
        double sum = 0.0;
        for (int j = 0; j < band; ++j) {
            const double x = ((double)(first + j) - centre) / scale;
            double v = 0.0;
            if (fabs(x) < 3.0) v = x == 0.0 ? 1.0 : (sin(pi * x) / (pi * x)) * (sin(pi * x / 3.0) / (pi * x / 3.0));
            w[j] = v;
            sum += v;
        }
        start_host[o] = first;
        for (int j = 0; j < band; ++j) coef_host[(size_t)o * band + j] = hb::float_to_half_bits((float)(w[j] / sum));
    }
    return HB_OK;
}
