// hb_pyr_level: one Laplacian-pyramid level as four chained products with strided-Toeplitz and two-phase
// coefficient matrices (Sec. V-B), and its vector-ALU twin.
//
// MFMA formulation.  w = [1,4,6,4,1]/16, A_down(n, u) = w[u - 2n + 2], A_up(x, n) the two phases of 2w (even outputs
// (1,6,1)/8 on D[q-1..q+1], odd outputs (1,1)/2 on D[q..q+1]).  Every product contracts over the index that the
// accumulator before it holds per lane, so the chain of one 16 x 16 output tile at (R, x0) stays in registers:
//   1 down, x   T1[y][n]  = sum_k P[y][k]  * A_down[n][k]     P = 32 pixels of a row from x0 - 8 on
//   2 down, y   D'[n][m]  = sum_k T1[k][n] * A_down[m][k]     k = 32 image rows from R - 8 on
//   3 up, x     U1[m][x]  = sum_k D[m][k]  * A_up[x][k]
//   4 up, y     R'[x][y]  = in'[x][y] - sum_k U1[k][x] * A_up[y][k]
// T1, D and U1 are rounded to fp16, which is what makes them operands; D is the coarser level itself, so that the
// residual belongs to the image that `down` receives: residual + up(down) gives the input back up to the rounding of
// U1.  (One product with the band matrix A_up A_down per axis, without D in between, takes half the roundings and
// loses exactly that.)  Each tile has 16 x 16 slots of D, slot i for sample (x0 or R) / 2 - 4 + i: slots 3 .. 12 feed
// the tile's outputs, 4 .. 11 are the samples under it.  The other slots' windows are cut off by the 32 pixels
// and meet zero weights.
// The original pixels reach the last product through the same registers: a 0/1 selection product copies them into
// accumulator layout (exactly), and they fill the half of the last product's K = 32 that U1's 16 rows leave free.
//
// Border rules.  Pixel indices are clamped at the load (rows per lane; columns requested from an address inside the
// row and shifted into place), so A_down has no border.  D indices are clamped in A_up: its entries there are
// sums of the plain ones, multiples of 1/8.
//
// Geometry.  A wave owns 32 columns x 16 NS rows and requests every pixel it needs before its first
// product (NS + 1 row tiles): it lives for one memory round trip plus its arithmetic, and what keeps the
// memory busy is the number of such waves.  8192 x 8192 with the coarser level 96 us, a copy of the bytes 73 to 79;
// 1024 x 1024 5.9, the rate of the host's launches.
#include "hb_device.hpp"
#include "hb_host.hpp"

namespace hb {

struct PyrArgs {
    const half_t* in;
    float* res;
    half_t* down;      // may be null
    int H, W, Hd, Wd;
    int64_t in_pitch, res_pitch, down_pitch;
    int nct, ntasks;   // 32-column strips; strips x segments of 16 NS rows
};

// w and the two phases of 2w as zero-padded runs: entry kPyrPad + t of a row is its weight t.  A fragment is eight (or
// twice four) consecutive entries.
constexpr int kPyrPad = 32, kPyrRow = 72;
struct PyrTable { uint16_t w[kPyrRow], up[2][kPyrRow]; };
constexpr uint16_t kPyr16th = 0x2c00, kPyr8th = 0x3000, kPyr4th = 0x3400, kPyr3_8ths = 0x3600, kPyrHalf = 0x3800, kPyr3_4ths = 0x3a00;
constexpr PyrTable pyr_make_table() {
    constexpr uint16_t w[5] = {kPyr16th, kPyr4th, kPyr3_8ths, kPyr4th, kPyr16th};
    constexpr uint16_t up[2][3] = {{kPyr8th, kPyr3_4ths, kPyr8th}, {0, kPyrHalf, kPyrHalf}};
    PyrTable t{};
    for (int i = 0; i < 5; ++i) t.w[kPyrPad + i] = w[i];
    for (int ph = 0; ph < 2; ++ph)
        for (int i = 0; i < 3; ++i) t.up[ph][kPyrPad + i] = up[ph][i];
    return t;
}
__device__ const PyrTable kPyrTable = pyr_make_table();

__device__ __forceinline__ half4 pyr_run4(const uint16_t* row, int t) { return *reinterpret_cast<const half4_u*>(row + kPyrPad + t); }
__device__ __forceinline__ half8 pyr_run8(const uint16_t* row, int t) { return *reinterpret_cast<const half8_u*>(row + kPyrPad + t); }
// A_up, output lane c, D slots 4g .. 4g + 3, away from the borders: output c is phase c % 2 of slot 4 + c / 2 ...
__device__ __forceinline__ half4 pyr_up(int c, int g) { return pyr_run4(kPyrTable.up[c & 1], 4 * g - 3 - (c >> 1)); }
// ... and with the D index clamped, for the outputs from x0 on (even) and n samples of D.
__device__ __forceinline__ half4 pyr_up_clamped(int x0, int n, int c, int g) {
    const int q = (x0 >> 1) + (c >> 1), first = (x0 >> 1) - 4 + 4 * g;
    half4 r;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        float s = 0.f;
#pragma unroll
        for (int d = -1; d <= 1; ++d) {
            const float v = (c & 1) ? (d < 0 ? 0.f : 0.5f) : (d == 0 ? 0.75f : 0.125f);
            s += clampi(q + d, 0, n - 1) == first + i ? v : 0.f;
        }
        r[i] = (half_t)s;
    }
    return r;
}

// Images narrower than this run the vector-ALU kernel, which keeps the row-filtered pixels and U along x in fp32.
constexpr int kPyrMinWidth = 48;

// 16-column tiles per strip.  Two: at most 106 registers, four waves per SIMD.
constexpr int kPyrNW = 2;

// One task: 16 NW columns x 16 NS rows from (x0, Y0).  INSIDE: every window and every output column of the
// strip lies inside the image and no D index along x is clamped (rows may still reach over the top and bottom).
template <int NS, int NW, bool INSIDE, bool DOWN>
__device__ __forceinline__ void pyr_task(const PyrArgs& p, float* patch, int x0, int Y0, int lane) {
    constexpr int NL = NS + 1;
    const int c = lane & 15, g = lane >> 4;
    const half4 z4 = {0, 0, 0, 0};
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
    const half8 down_x = pyr_run8(kPyrTable.w, 8 * g - 2 * c + 2);
    const half8 down_y = join(pyr_run4(kPyrTable.w, 4 * g - 2 * c + 2), pyr_run4(kPyrTable.w, 4 * g - 2 * c + 18));
    half4 up_x[INSIDE ? 1 : NW];
#pragma unroll
    for (int w = 0; w < (INSIDE ? 1 : NW); ++w) up_x[w] = INSIDE ? pyr_up(c, g) : pyr_up_clamped(x0 + 16 * w, p.Wd, c, g);
    const half4 up_y0 = -pyr_up(c, g);
    half8 selx;                                           // pixels 8 .. 23 of the window
    half4 sely;                                           // rows 8 .. 23 of it, lane (c, g) holding 16 (g < 2) + 4g + i
#pragma unroll
    for (int i = 0; i < 8; ++i) selx[i] = (half_t)(8 * g + i == c + 8 ? 1.f : 0.f);
#pragma unroll
    for (int i = 0; i < 4; ++i) sely[i] = (half_t)(4 * g + i + (g < 2 ? 16 : 0) == c + 8 ? 1.f : 0.f);

    half4 T[2][NW], X[2][NW], D[2][NW];                   // row tiles q - 1 and q: down along x, copied; D of two steps
#pragma unroll
    for (int q = 0; q < NL; ++q) {
        __builtin_amdgcn_sched_barrier(0);                // row tile by row tile: keeps few results live at a time
#pragma unroll
        for (int w = 0; w < NW; ++w) {
            if (!INSIDE) {
                const int xs = x0 - 8 + 16 * w + 8 * g;
                px[q][w] = shift_in_from_right(px[q][w], max(xs - (p.W - 8), 0));
                px[q][w] = shift_in_from_left(px[q][w], max(-xs, 0));
            }
            T[q & 1][w] = to_half4(mfma16x16x32(px[q][w], down_x, zero));
            X[q & 1][w] = to_half4(mfma16x16x32(px[q][w], selx, zero));
        }
        if (q == 0) continue;
        const int s = q - 1, R = Y0 + 16 * s;             // output rows R .. R + 15, window rows R - 8 .. R + 23
        if (R >= p.H) break;                              // uniform
        half4 up_y = up_y0;
        if (R == 0 || R + 18 > p.H) up_y = -pyr_up_clamped(R, p.Hd, c, g);   // uniform
        floatx4 acc[NW];
#pragma unroll
        for (int w = 0; w < NW; ++w) {
            D[s & 1][w] = to_half4(mfma16x16x32(join(T[s & 1][w], T[q & 1][w]), down_y, zero));
            const half4 u = to_half4(mfma16x16x32(join(D[s & 1][w], z4), join(up_x[INSIDE ? 0 : w], z4), zero));
            acc[w] = mfma16x16x32(join(u, g < 2 ? X[q & 1][w] : X[s & 1][w]), join(up_y, sely), zero);
        }
        if (INSIDE && R + 16 <= p.H)
            store_rows_via_lds<NW, true>(patch, p.res + (int64_t)R * p.res_pitch + x0, (uint32_t)p.res_pitch, acc, lane);
        else
            store_rows_via_lds_masked<NW, true>(patch, p.res + (int64_t)R * p.res_pitch + x0, p.res_pitch, acc, lane, p.H - R, p.W - x0);
        if (DOWN && ((s & 1) || R + 16 >= p.H)) {
            // the 8 rows of D under each of two steps, eight columns per tile: lane (c, g) holds row slot c, column
            // slots 4g .. 4g + 3.  16 bytes per lane, 16 NW bytes of a row together.  Plain stores: the next level reads them
            const int m0 = (R - 16 * (s & 1)) / 2;
            half_t* const dp = reinterpret_cast<half_t*>(patch);
            constexpr int kPitch = 8 * NW + 8;
            if (c >= 4 && c < 12 && (g == 1 || g == 2)) {
#pragma unroll
                for (int w = 0; w < NW; ++w) {
                    half_t* const q4 = dp + (c - 4) * kPitch + 8 * w + 4 * (g - 1);
                    *reinterpret_cast<half4*>(q4) = D[0][w];
                    if (s & 1) *reinterpret_cast<half4*>(q4 + 8 * kPitch) = D[1][w];
                }
            }
            wave_lds_fence();
            const int dr = lane / NW, n = 8 * (lane - NW * dr);
            const int rows = min(p.Hd - m0, (s & 1) ? 16 : 8), cols = p.Wd - x0 / 2 - n;
            if (dr < rows) {
                const half8 dv = *reinterpret_cast<const half8*>(dp + dr * kPitch + n);
                half_t* const dst = p.down + (int64_t)(m0 + dr) * p.down_pitch + x0 / 2 + n;
                if (INSIDE || cols >= 8) {
                    *reinterpret_cast<half8_u*>(dst) = dv;
                } else {
#pragma unroll
                    for (int i = 0; i < 8; ++i)
                        if (i < cols) dst[i] = dv[i];
                }
            }
            wave_lds_fence();
        }
    }
}

template <int NS, bool DOWN>
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
        pyr_task<NS, kPyrNW, true, DOWN>(p, patch, x0, Y0, lane);
    } else {
        // border strips two row steps at a time: with weights per tile the whole task's registers would cost every
        // strip a wave per SIMD
#pragma unroll 1
        for (int y = Y0; y < min(Y0 + 16 * NS, p.H); y += 32) {
            int l = lane;                                 // nothing lane-dependent is kept from turn to turn
            asm volatile("" : "+v"(l));
            pyr_task<2, kPyrNW, false, DOWN>(p, patch, x0, y, l);
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
    if (a.down) hipLaunchKernelGGL((pyr_mfma_kernel<NS, true>), grid, dim3(256), 0, st, a);
    else hipLaunchKernelGGL((pyr_mfma_kernel<NS, false>), grid, dim3(256), 0, st, a);
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
    if (W < kPyrMinWidth)
        return hb_pyr_level_valu(in, residual, down_or_null, H, W, in_pitch, res_pitch, down_pitch, stream);
    hipStream_t st = reinterpret_cast<hipStream_t>(stream);
    a.nct = ceil_div(W, 16 * kPyrNW);
    // Long tasks re-read fewer rows (NS + 1 row tiles for NS), short ones fill the chip and end together: NS = 4 /
    // NS = 2 measured 96 / 104 us on 8192 x 8192 (32768 long tasks), 27.3 / 27.6 on 4096 x 4096 (8192), 17.6 / 16.1
    // on 3002 x 2710 (3995), 8.5 / 7.9 on 2048 x 2048 (2048).
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
