// hb_pyr_level: one Laplacian-pyramid level (2x down, 2x up, residual) with strided-Toeplitz and
// two-phase coefficient matrices (Sec. V-B), and its vector-ALU twin.
//
// MFMA formulation.  w = [1,4,6,4,1]/16.  Per axis the level is two linear maps, A_down(n, u) = w[u - 2n + 2]
// and the phase matrix A_up(x, n) (even outputs (1,6,1)/8 on D[q-1..q+1], odd outputs (1,1)/2 on
// D[q..q+1]), so what is subtracted from the image is
//     U = C_y * in * C_x^T,   C = A_up * A_down,
// a band matrix of two alternating rows, [1,4,12,28,38,28,12,4,1]/128 and [1,4,7,8,7,4,1]/32, whose entries
// are exact in fp16.  The border rules (pixel index clamped in A_down, D index clamped in A_up) only change
// the entries of the first three and the last four rows of C, which stay multiples of 1/128.  So a level is
// ONE pair of chained Toeplitz products per 16 x 16 output tile, as in hb_sepblur, instead of four:
//   row pass      T1[y][n] = sum_k P[y][k] * C_x[n][k]        P = 32 pixels of a row from x0 - 8 on
//   column pass   R'[n][m] = in'[n][m] - sum_k T1h[k][n] * C_y[m][k]    k = 32 image rows from y0 - 8 on
// The original pixels reach the column pass through the same registers: a 0/1 selection product copies
// them into accumulator layout (exactly), and a second one, with the rows shifted by the window's 8,
// seeds the accumulator.  The coarser level, when it is wanted, shares both passes' operands: 32 pixels
// give 8 D columns of a 16-column tile, two tiles (and two row steps) fill one D tile.
//
// Geometry.  A wave owns 64 columns x 16 NS rows and requests every pixel it needs before its first
// product (NS + 1 row tiles): it lives for one memory round trip plus its arithmetic, and what keeps the
// memory busy is the number of such waves.  Windows that reach over the image border load from an address
// moved inside the row; what lies outside has weight zero.
#include "hb_device.hpp"
#include "hb_host.hpp"

namespace hb {

struct PyrArgs {
    const half_t* in;
    float* res;
    half_t* down;      // may be null
    int H, W, Hd, Wd;
    int64_t in_pitch, res_pitch, down_pitch;
    int nct, ntasks;   // 64-column strips; strips x segments of 16 NS rows
};

// Rows of C and of A_down as zero-padded runs, in 1/128: entry kPyrPad + t is the weight of pixel x + t (of pixel
// 2n + t for A_down), of pixel t at the left / top border, of pixel n - 1 + t at the right / bottom one.  A
// fragment is eight (or twice four) consecutive entries of the row that its output column selects.
constexpr int kPyrPad = 40, kPyrRow = 96;
constexpr int kPyrStd = 0, kPyrLeft = 2, kPyrRight = 5, kPyrDown = 9, kPyrDownLeft = 10, kPyrDownRight = 11, kPyrRows = 12;
struct PyrTable { uint16_t v[kPyrRows * kPyrRow]; };

// fp16 bits of v / 128, 0 <= v <= 128
constexpr uint16_t pyr_half_bits(int v) {
    if (v == 0) return 0;
    int k = 0;
    while ((v >> (k + 1)) != 0) ++k;
    return (uint16_t)(((k - 7 + 15) << 10) | ((v << (10 - k)) & 0x3ff));
}
// 16 * weight of pixel u in D sample n (pixel index clamped to [0, len - 1])
constexpr int pyr_down_weight(int n, int u, int len) {
    constexpr int w[5] = {1, 4, 6, 4, 1};
    int s = 0;
    for (int t = 0; t < 5; ++t) {
        int q = 2 * n + t - 2;
        q = q < 0 ? 0 : (q > len - 1 ? len - 1 : q);
        if (q == u) s += w[t];
    }
    return s;
}
// 128 * weight of pixel u in output x of U (D index clamped as well)
constexpr int pyr_weight(int x, int u, int len) {
    constexpr int up[2][3] = {{1, 6, 1}, {0, 4, 4}};
    int s = 0;
    for (int d = -1; d <= 1; ++d) {
        int n = (x >> 1) + d;
        n = n < 0 ? 0 : (n > len / 2 - 1 ? len / 2 - 1 : n);
        s += up[x & 1][d + 1] * pyr_down_weight(n, u, len);
    }
    return s;
}
constexpr PyrTable pyr_make_table() {
    constexpr int L = 64;                                 // any length whose two borders do not meet
    PyrTable t{};
    for (int u = 0; u < L; ++u) {
        for (int e = 0; e < 2; ++e) {                     // outputs 32 and 33: away from both borders
            const int w = pyr_weight(L / 2 + e, u, L), o = u - (L / 2 + e) + kPyrPad;
            if (w) t.v[(kPyrStd + e) * kPyrRow + o] = pyr_half_bits(w);
        }
        for (int x = 0; x < 3; ++x)
            if (u < kPyrRow - kPyrPad) t.v[(kPyrLeft + x) * kPyrRow + u + kPyrPad] = pyr_half_bits(pyr_weight(x, u, L));
        for (int d = 0; d < 4; ++d)
            if (u - (L - 1) + kPyrPad >= 0)
                t.v[(kPyrRight + d) * kPyrRow + u - (L - 1) + kPyrPad] = pyr_half_bits(pyr_weight(L - 1 - d, u, L));
        const int dw = pyr_down_weight(L / 4, u, L), dl = pyr_down_weight(0, u, L), dr = pyr_down_weight(L / 2 - 1, u, L);
        if (dw) t.v[kPyrDown * kPyrRow + u - L / 2 + kPyrPad] = pyr_half_bits(8 * dw);
        if (dl) t.v[kPyrDownLeft * kPyrRow + u + kPyrPad] = pyr_half_bits(8 * dl);
        if (dr) t.v[kPyrDownRight * kPyrRow + u - (L - 1) + kPyrPad] = pyr_half_bits(8 * dr);
    }
    return t;
}
__device__ const PyrTable kPyrTable = pyr_make_table();
// Borders that do not meet: row 2 of C reads pixel 6, row n - 4 reads pixel n - 8 and up.
constexpr int kPyrMinSide = 8;

// Entry of the table from which the weights of pixels u, u + 1, ... in output x (of an axis of n) run.
__device__ __forceinline__ const uint16_t* pyr_run(int x, int u, int n) {
    const bool left = x <= 2, right = x >= n - 4 && x < n;
    const int row = left ? kPyrLeft + x : right ? kPyrRight + (n - 1 - x) : kPyrStd + (x & 1);
    const int off = left ? u : right ? u - (n - 1) : u - x;
    return kPyrTable.v + row * kPyrRow + kPyrPad + off;
}
// ... and in D sample m
__device__ __forceinline__ const uint16_t* pyr_down_run(int m, int u, int n) {
    const bool left = m == 0, right = m == n / 2 - 1;
    const int row = left ? kPyrDownLeft : right ? kPyrDownRight : kPyrDown;
    const int off = left ? u : right ? u - (n - 1) : u - 2 * m;
    return kPyrTable.v + row * kPyrRow + kPyrPad + off;
}
__device__ __forceinline__ half8 pyr_natural(const uint16_t* run) { return *reinterpret_cast<const half8_u*>(run); }
// chained slot order: slots 8g + 0..3 and 8g + 4..7 are 16 rows apart
__device__ __forceinline__ half8 pyr_chained(const uint16_t* run) {
    return join(*reinterpret_cast<const half4_u*>(run), *reinterpret_cast<const half4_u*>(run + 16));
}
__device__ __forceinline__ half8 pyr_negated(half8 v) {
    u32x4 b = __builtin_bit_cast(u32x4, v);
    b ^= 0x80008000u;
    return __builtin_bit_cast(half8, b);
}

// 16-column tiles per strip.  Two: 122 registers, four waves per SIMD (8192 x 8192 with the coarser level
// 96 us, 4096 x 4096 22.3); four (256-byte runs, 196 registers, two waves) 99 / 24.0.
constexpr int kPyrNW = 2;

// One task: 16 NW columns x 16 NS rows from (x0, Y0).  INSIDE: every window and every output column of the
// strip lies inside the image (rows may still reach over the top and bottom).
template <int NS, int NW, bool INSIDE, bool STREAM, bool DOWN>
__device__ __forceinline__ void pyr_task(const PyrArgs& p, float* patch, int x0, int Y0, int lane) {
    constexpr int NV = NW / 2, NL = NS + 1;
    const int c = lane & 15, g = lane >> 4;
    const half8 z8 = {0, 0, 0, 0, 0, 0, 0, 0};
    const floatx4 zero = {0.f, 0.f, 0.f, 0.f};

    half8 px[NL][NW];
#pragma unroll
    for (int q = 0; q < NL; ++q) {
        const half_t* row = p.in + (int64_t)clampi(Y0 - 8 + 16 * q + c, 0, p.H - 1) * p.in_pitch;
#pragma unroll
        for (int w = 0; w < NW; ++w) {
            const int xs = x0 - 8 + 16 * w + 8 * g;
            px[q][w] = *reinterpret_cast<const half8_u*>(row + (INSIDE ? xs : clampi(xs, 0, p.W - 8)));
        }
    }
    // coefficients only now: a wave that waited for them first would put a memory round trip in front of
    // its pixel requests
    __builtin_amdgcn_sched_barrier(0);
    // Weights of tile w for the row pass, and for the D columns 16 v + c under the strip: tile 2v gives those of the
    // lanes c < 8, tile 2v + 1 the others (away from the borders the same numbers, eight lanes on).  Away from the
    // borders every tile has the same weights: column 32 stands for any.
    constexpr int NF = INSIDE ? 1 : NW;
    half8 bx[NF], bd[NF];
#pragma unroll
    for (int w = 0; w < NF; ++w) {
        const int xt = INSIDE ? 32 : x0 + 16 * w, n = INSIDE ? 1 << 20 : p.W;
        bx[w] = pyr_natural(pyr_run(xt + c, xt - 8 + 8 * g, n));
        if (DOWN) bd[w] = pyr_natural(pyr_down_run(xt / 2 + (c & 7), xt - 8 + 8 * g, n));
    }
    half8 selx, sely;                                     // pixels 8 .. 23 of the window; rows 8 .. 23 of it
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        selx[i] = (half_t)(8 * g + i == c + 8 ? 1.f : 0.f);
        sely[i] = (half_t)(krow32(g, i) == c + 8 ? 1.f : 0.f);
    }
    // column-pass weights of row step R; of D, a step has eight rows, so two steps share a tile of 16
    auto column_weights = [&](int R, int n) { return pyr_negated(pyr_chained(pyr_run(R + c, R - 8 + 4 * g, n))); };
    auto down_column_weights = [&](int R, int n) { return pyr_chained(pyr_down_run(R / 2 + (c & 7), R - 8 + 4 * g, n)); };
    auto half_lanes = [&](half8 f, int u) { return (c >= 8) == (bool)u ? f : z8; };
    const bool edge = Y0 == 0 || Y0 + 16 * NS + 4 > p.H;  // uniform
    const half8 by0 = column_weights(32, 1 << 20);
    half8 bm0;
    if (DOWN) bm0 = down_column_weights(32, 1 << 20);

    half4 T[2][NW], X[2][NW], Td[2][NV];                  // row tiles q - 1 and q: row-filtered, copied, D columns
    floatx4 D[NV];
#pragma unroll
    for (int q = 0; q < NL; ++q) {
        __builtin_amdgcn_sched_barrier(0);                // row tile by row tile: keeps few results live at a time
#pragma unroll
        for (int w = 0; w < NW; ++w) {
            if (!INSIDE) {
                const int xs = x0 - 8 + 16 * w + 8 * g;
                px[q][w] = shift_in_from_right(px[q][w], xs - clampi(xs, 0, p.W - 8));
            }
            T[q & 1][w] = to_half4(mfma16x16x32(px[q][w], bx[INSIDE ? 0 : w], zero));
            X[q & 1][w] = to_half4(mfma16x16x32(px[q][w], selx, zero));
        }
        if (DOWN) {
#pragma unroll
            for (int v = 0; v < NV; ++v) {
                floatx4 d = mfma16x16x32(px[q][2 * v], half_lanes(bd[INSIDE ? 0 : 2 * v], 0), zero);
                d = mfma16x16x32(px[q][2 * v + 1], half_lanes(bd[INSIDE ? 0 : 2 * v + 1], 1), d);
                Td[q & 1][v] = to_half4(d);
            }
        }
        if (q == 0) continue;
        const int s = q - 1, R = Y0 + 16 * s;             // output rows R .. R + 15, window rows R - 8 .. R + 23
        if (R >= p.H) break;                              // uniform
        half8 by = by0, bm;
        if (DOWN) bm = bm0;
        if (edge && (R == 0 || R + 20 > p.H)) {           // uniform
            by = column_weights(R, p.H);
            if (DOWN) bm = down_column_weights(R, p.H);
        }
        floatx4 acc[NW];
#pragma unroll
        for (int w = 0; w < NW; ++w) {
            acc[w] = mfma16x16x32(join(X[s & 1][w], X[q & 1][w]), sely, zero);
            acc[w] = mfma16x16x32(join(T[s & 1][w], T[q & 1][w]), by, acc[w]);
        }
        if (INSIDE && R + 16 <= p.H)
            store_rows_via_lds<NW, STREAM>(patch, p.res + (int64_t)R * p.res_pitch + x0, (uint32_t)p.res_pitch, acc, lane);
        else
            store_rows_via_lds_masked<NW, STREAM>(patch, p.res + (int64_t)R * p.res_pitch + x0, p.res_pitch, acc, lane, p.H - R, p.W - x0);
        if (DOWN) {
#pragma unroll
            for (int v = 0; v < NV; ++v)
                D[v] = mfma16x16x32(join(Td[s & 1][v], Td[q & 1][v]), half_lanes(bm, s & 1), (s & 1) ? D[v] : zero);
            if ((s & 1) || R + 16 >= p.H) {
                // D rows m0 + lane column, m0 that of the pair's first step; 16 bytes per lane, 32 NV bytes
                // of a row together.  Plain stores: the next level reads them
                const int m0 = (R - 16 * (s & 1)) / 2;
                half_t* const dp = reinterpret_cast<half_t*>(patch);
                constexpr int kPitch = 16 * NV + 8, kLanes = 2 * NV;
#pragma unroll
                for (int v = 0; v < NV; ++v) *reinterpret_cast<half4*>(dp + c * kPitch + 16 * v + 4 * g) = to_half4(D[v]);
                wave_lds_fence();
                const int dr = lane / kLanes, n = 8 * (lane - kLanes * dr);
                if (NV == 2 || dr < 16) {
                    const half8 dv = *reinterpret_cast<const half8*>(dp + dr * kPitch + n);
                    half_t* const dst = p.down + (int64_t)(m0 + dr) * p.down_pitch + x0 / 2 + n;
                    const int rows = min(p.Hd - m0, (s & 1) ? 16 : 8), cols = p.Wd - x0 / 2 - n;
                    if (dr < rows) {
                        if (INSIDE || cols >= 8) {
                            *reinterpret_cast<half8_u*>(dst) = dv;
                        } else {
#pragma unroll
                            for (int i = 0; i < 8; ++i)
                                if (i < cols) dst[i] = dv[i];
                        }
                    }
                }
                wave_lds_fence();
            }
        }
    }
}

template <int NS, bool STREAM, bool DOWN>
__global__ void __launch_bounds__(256, 4) pyr_mfma_kernel(PyrArgs p) {
    __shared__ __attribute__((aligned(16))) float s_patch[4][RowPatch<kPyrNW>::kFloats];
    const int lane = threadIdx.x & 63;
    // of every 32 workgroups an XCD takes four neighbours: the chip sweeps through the image in launch
    // order and neighbouring tasks meet in one L2
    const int task = __builtin_amdgcn_readfirstlane(xcd_blocked(blockIdx.x, gridDim.x, 4) * 4 + (threadIdx.x >> 6));
    if (task >= p.ntasks) return;
    const int seg = task / p.nct, ct = task - seg * p.nct;
    const int x0 = 16 * kPyrNW * ct, Y0 = 16 * NS * seg;
    float* patch = s_patch[threadIdx.x >> 6];
    if (x0 > 0 && x0 + 16 * kPyrNW + 8 <= p.W) {
        pyr_task<NS, kPyrNW, true, STREAM, DOWN>(p, patch, x0, Y0, lane);
    } else {
        // border strips two row steps at a time: with weights per tile the whole task's registers would cost every
        // strip a wave per SIMD
#pragma unroll 1
        for (int y = Y0; y < min(Y0 + 16 * NS, p.H); y += 32) {
            int l = lane;                                 // nothing lane-dependent is kept from turn to turn
            asm volatile("" : "+v"(l));
            pyr_task<2, kPyrNW, false, STREAM, DOWN>(p, patch, x0, y, l);
        }
    }
}

// ---------------------------------------------------------------------------
// Vector-ALU twin: a 32 x 64 output tile per workgroup, every stage through LDS with
// plain fp32 FMAs.  D is rounded to fp16 as in the MFMA path; the D tile is gathered at
// clamped D indices, which is the definition's border rule verbatim.
constexpr int kPTH = 32, kPTW = 64;
constexpr int kPRows = kPTH + 7;             // image rows 2(M-1)-2 .. 2(M+16)+2
constexpr int kPPitch = 88;                  // image columns X0-8 .. X0+79
constexpr int kPDR = kPTH / 2 + 2, kPDC = kPTW / 2 + 2;

__global__ void __launch_bounds__(256) pyr_valu_kernel(PyrArgs p) {
    __shared__ half_t s_px[kPRows * kPPitch];
    __shared__ float s_hx[kPRows * (kPDC + 1)];
    __shared__ half_t s_d[kPDR * (kPDC + 2)];
    __shared__ float s_u1[kPDR * (kPTW + 4)];
    const float wt[5] = {0.0625f, 0.25f, 0.375f, 0.25f, 0.0625f};
    const int nctv = (p.W + kPTW - 1) / kPTW;
    const int rt = blockIdx.x / nctv, ct = blockIdx.x - rt * nctv;
    const int X0 = ct * kPTW, R0 = rt * kPTH;
    const int xs = X0 - 8, ys = R0 - 4;
    for (int idx = threadIdx.x; idx < kPRows * (kPPitch / 8); idx += 256) {
        const int r = idx / (kPPitch / 8), ch = idx - r * (kPPitch / 8);
        const half_t* row = p.in + (int64_t)clampi(ys + r, 0, p.H - 1) * p.in_pitch;
        *reinterpret_cast<half8*>(&s_px[r * kPPitch + 8 * ch]) = load8_clamp(row, xs + 8 * ch, p.W);
    }
    __syncthreads();
    // down along x at the (clamped) D columns this tile's up pass reads
    for (int idx = threadIdx.x; idx < kPRows * kPDC; idx += 256) {
        const int r = idx / kPDC, j = idx - r * kPDC;
        const int dc = clampi(X0 / 2 - 1 + j, 0, p.Wd - 1);
        float acc = 0.f;
#pragma unroll
        for (int k = 0; k < 5; ++k)
            acc = fmaf(wt[k], (float)s_px[r * kPPitch + clampi(2 * dc + k - 2, 0, p.W - 1) - xs], acc);
        s_hx[r * (kPDC + 1) + j] = acc;
    }
    __syncthreads();
    // down along y -> D (fp16), optional store of the D samples under this tile
    for (int idx = threadIdx.x; idx < kPDR * kPDC; idx += 256) {
        const int i = idx / kPDC, j = idx - i * kPDC;
        const int dr = clampi(R0 / 2 - 1 + i, 0, p.Hd - 1);
        float acc = 0.f;
#pragma unroll
        for (int k = 0; k < 5; ++k)
            acc = fmaf(wt[k], s_hx[(clampi(2 * dr + k - 2, 0, p.H - 1) - ys) * (kPDC + 1) + j], acc);
        const half_t dv = (half_t)acc;
        s_d[i * (kPDC + 2) + j] = dv;
        if (p.down && i >= 1 && i <= kPTH / 2 && j >= 1 && j <= kPTW / 2) {
            const int m = R0 / 2 - 1 + i, n = X0 / 2 - 1 + j;
            if (m < p.Hd && n < p.Wd) p.down[(int64_t)m * p.down_pitch + n] = dv;
        }
    }
    __syncthreads();
    // up along x
    for (int idx = threadIdx.x; idx < kPDR * kPTW; idx += 256) {
        const int i = idx / kPTW, x = idx - i * kPTW;
        const half_t* d = &s_d[i * (kPDC + 2) + (x >> 1)];       // d[0] = D[q-1], d[1] = D[q], d[2] = D[q+1]
        s_u1[i * (kPTW + 4) + x] = (x & 1) ? 0.5f * ((float)d[1] + (float)d[2])
                                           : 0.125f * ((float)d[0] + (float)d[2]) + 0.75f * (float)d[1];
    }
    __syncthreads();
    // up along y, residual; four consecutive columns per thread
    for (int idx = threadIdx.x; idx < kPTH * (kPTW / 4); idx += 256) {
        const int y = idx / (kPTW / 4), cg = idx - y * (kPTW / 4);
        const int yo = R0 + y, xo = X0 + 4 * cg;
        if (yo >= p.H || xo >= p.W) continue;
        const float* u = &s_u1[(y >> 1) * (kPTW + 4) + 4 * cg];  // rows q-1, q, q+1
        const half_t* px = &s_px[(y + 4) * kPPitch + 4 * cg + 8];
        floatx4 rv;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const float a = u[v], b = u[(kPTW + 4) + v], cc = u[2 * (kPTW + 4) + v];
            const float up = (y & 1) ? 0.5f * (b + cc) : 0.125f * (a + cc) + 0.75f * b;
            rv[v] = (float)px[v] - up;
        }
        store4_mask(p.res + (int64_t)yo * p.res_pitch, xo, p.W, rv);
    }
}

static hb_status pyr_prepare(PyrArgs& a, const hb_half* in, float* res, hb_half* down,
                             int H, int W, int64_t in_pitch, int64_t res_pitch, int64_t down_pitch) {
    hb_status s = check_image(in, res, H, W, in_pitch, res_pitch);
    if (s != HB_OK) return s;
    if ((H & 1) || (W & 1)) return HB_ERR_INVALID_ARG;
    if (down && (down_pitch < W / 2 || !aligned_to(down, 2))) return HB_ERR_INVALID_ARG;
    if (down && down_pitch > ((int64_t)1 << 26)) return HB_ERR_UNSUPPORTED;
    a.in = reinterpret_cast<const half_t*>(in);
    a.res = res;
    a.down = reinterpret_cast<half_t*>(down);
    a.H = H;
    a.W = W;
    a.Hd = H / 2;
    a.Wd = W / 2;
    a.in_pitch = in_pitch;
    a.res_pitch = res_pitch;
    a.down_pitch = down_pitch;
    a.nct = a.ntasks = 0;
    return HB_OK;
}

template <int NS>
static hb_status pyr_launch(PyrArgs& a, hipStream_t st) {
    const int64_t ntasks = (int64_t)a.nct * ceil_div(a.H, 16 * NS);
    if (ntasks > 0x7fffffff - 4) return HB_ERR_UNSUPPORTED;
    a.ntasks = (int)ntasks;
    const dim3 grid((unsigned)((ntasks + 3) / 4));
    if (a.down) hipLaunchKernelGGL((pyr_mfma_kernel<NS, true, true>), grid, dim3(256), 0, st, a);
    else hipLaunchKernelGGL((pyr_mfma_kernel<NS, true, false>), grid, dim3(256), 0, st, a);
    return launch_status();
}

}  // namespace hb

extern "C" hb_status hb_pyr_level_valu(const hb_half* in, float* residual, hb_half* down_or_null,
                                       int H, int W, int64_t in_pitch, int64_t res_pitch, int64_t down_pitch,
                                       hb_stream stream);

extern "C" hb_status hb_pyr_level(const hb_half* in, float* residual, hb_half* down_or_null,
                                  int H, int W, int64_t in_pitch, int64_t res_pitch, int64_t down_pitch,
                                  hb_stream stream) {
    using namespace hb;
    PyrArgs a;
    hb_status s = pyr_prepare(a, in, residual, down_or_null, H, W, in_pitch, res_pitch, down_pitch);
    if (s != HB_OK) return s;
    if (W < kPyrMinSide || H < kPyrMinSide)   // the two borders' rows of C meet: vector-ALU kernel
        return hb_pyr_level_valu(in, residual, down_or_null, H, W, in_pitch, res_pitch, down_pitch, stream);
    hipStream_t st = reinterpret_cast<hipStream_t>(stream);
    a.nct = ceil_div(W, 16 * kPyrNW);
    // Long tasks re-read fewer rows (NS + 1 row tiles for NS), short ones fill the chip and end together: NS = 4 /
    // NS = 2 measured 96 / 111 us on 8192 x 8192 (32768 long tasks), 22.3 / 25.3 on 4096 x 4096 (8192), 18.2 / 16.1
    // on 3002 x 2710 (3995), the same on 2048 x 2048 (2048).
    if ((int64_t)a.nct * ceil_div(H, 64) >= 24 * num_cu()) return pyr_launch<4>(a, st);
    return pyr_launch<2>(a, st);
}

extern "C" hb_status hb_pyr_level_valu(const hb_half* in, float* residual, hb_half* down_or_null,
                                       int H, int W, int64_t in_pitch, int64_t res_pitch, int64_t down_pitch,
                                       hb_stream stream) {
    using namespace hb;
    PyrArgs a;
    hb_status s = pyr_prepare(a, in, residual, down_or_null, H, W, in_pitch, res_pitch, down_pitch);
    if (s != HB_OK) return s;
    const int64_t blocks = (int64_t)ceil_div(H, kPTH) * ceil_div(W, kPTW);
    if (blocks > 0x7fffffff) return HB_ERR_UNSUPPORTED;
    hipLaunchKernelGGL(pyr_valu_kernel, dim3((unsigned)blocks), dim3(256), 0,
                       reinterpret_cast<hipStream_t>(stream), a);
    return launch_status();
}
