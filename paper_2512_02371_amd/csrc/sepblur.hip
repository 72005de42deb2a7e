// hb_sepblur: separable 2-D blur as two chained Toeplitz products per tile
// (Sec. V-A), and its vector-ALU twin.
//
// MFMA formulation.  A wave owns a strip of HB_SEP_TILES 16-column tiles and goes
// down it in steps of 16 rows.
//   row pass     T1[m][n] = sum_k P[m][k] * Bx[k][n]     m = image row, n = column, k = pixel
//                P = the 32*NKX pixels from x0 - ax - e on (e = ax & 1: even, dword-aligned
//                window start),   Bx[k][n] = taps_x[k - n - e]
//   column pass  O'[m][n] = sum_k T1h[m][k] * By[k][n]   m = column, n = output row, k = window row
//                By[k][n] = taps_y[window_row(k) - n]
// The row-pass accumulator holds, per lane, four consecutive ROWS of one column,
// which is exactly the operand layout of a product that contracts over rows: two
// stacked accumulators, rounded to fp16 (the stage's fp16 intermediate), are the
// K = 32 A-operand of the column pass without leaving the registers.  The paper
// handles the second axis with a serial loop over r_y; separability turns it into
// this second Toeplitz product with the roles of image and coefficients swapped.
// The column-pass accumulator holds four consecutive COLUMNS of one row per lane,
// so results leave with one 16-byte store per lane.
//
// The window rows of output rows [R, R+16) are [R - ay, R - ay + 15 + Ty - 1]; row
// tiles are laid on the grid R - ay + 16 q, so a step consumes NT = (Ty + 30) / 16
// consecutive tiles and produces one new tile.  Rows outside the image repeat the
// edge row: clamping the image row index at the load is the same as clamping the
// index of the row-filtered intermediate, because the row pass treats rows
// independently.
#include "hb_device.hpp"
#include "hb_host.hpp"
#include "sepblur_plan.hpp"
#include <algorithm>

namespace hb {

struct SepArgs {
    const half_t* in;
    float* out;
    int H, W;
    int64_t in_pitch, out_pitch;
    int Tx, ax, Ty, ay;
    int nct, nseg;     // strips (of 128 columns for the marching kernel) x segments
    int steps;         // 16-row steps per segment
    int c0, c1;        // strips whose windows and tiles lie inside the row
    Taps tx, ty;
};

// Coefficient fragments, read from the tap tables in the kernel arguments: coefx[kk] = B operand of the
// row pass, Bx[32 kk + 8g + i][c]; coefy[j] = B operand of the column pass in the chained slot order.
template <int NKX, int NK>
__device__ __forceinline__ void sep_fragments(const SepArgs& p, int c, int g, half8 (&coefx)[NKX], half8 (&coefy)[NK]) {
    const int e = p.ax & 1;
#pragma unroll
    for (int kk = 0; kk < NKX; ++kk) coefx[kk] = tap_run(p.tx.tab, 32 * kk + 8 * g - c - e);
#pragma unroll
    for (int j = 0; j < NK; ++j)
#pragma unroll
        for (int i = 0; i < 8; ++i) coefy[j][i] = tap_at(p.ty.tab, 32 * j + krow32(g, i) - c);
}

// One window per tile (up to 17 taps along x).  A wave requests ALL its row tiles before the
// first product.  It then lives for one memory round trip plus its arithmetic, and what keeps
// the memory system busy is the number of such waves in flight (the dispatcher refills as they
// leave) rather than a chain of dependent steps inside one long-lived wave, each waiting for the
// one tile it has in flight.  INSIDE: every window of the strip lies inside the row and every tile is full.
// The other strips load what reaches over the row's ends from an address moved inside and shift it into
// place in registers, which is the column clamp itself (with the clamp folded into per-tile coefficients
// instead, whose tables every lane gathered from the kernel arguments, a border strip took 15 us whatever the
// image size).  Rows are clamped per lane and rows beyond the image are not stored.
template <int NT, int NS, bool INSIDE>
__device__ __forceinline__ void sep_task(const SepArgs& p, float* patch, int x0, int Y0, int xw, int lane) {
    constexpr int NW = HB_SEP_TILES, NL = NS + NT - 1, NK = (NT + 1) / 2;
    const int c = lane & 15, g = lane >> 4;
    const half_t* src = p.in + (INSIDE ? x0 - xw : 0);    // uniform; lanes add row * pitch + 8g
    half8 px[NL][NW];
#pragma unroll
    for (int q = 0; q < NL; ++q) {
        const int yr = clampi(Y0 - p.ay + 16 * q + c, 0, p.H - 1);
        const uint32_t off = (uint32_t)yr * (uint32_t)p.in_pitch * 2u;
#pragma unroll
        for (int w = 0; w < NW; ++w) {
            const int xs = 16 * w + 8 * g;
            px[q][w] = ldg8(src, off + 2u * (uint32_t)(INSIDE ? xs : clampi(x0 - xw + xs, 0, p.W - 8)));
        }
    }
    // The tap tables are read only now: a wave that waited for them first would put a memory round
    // trip in front of its pixel requests.
    __builtin_amdgcn_sched_barrier(0);
    half8 coefx[1], coefy[NK];
    sep_fragments<1, NK>(p, c, g, coefx, coefy);
    half4 h[NL][NW];                                      // row-filtered tiles, rounded to fp16
#pragma unroll
    for (int q = 0; q < NL; ++q) {
#pragma unroll
        for (int w = 0; w < NW; ++w) {
            half8 v = px[q][w];
            if (!INSIDE) {
                const int xs = x0 - xw + 16 * w + 8 * g;
                v = shift_in_from_right(v, max(xs - (p.W - 8), 0));
                v = shift_in_from_left(v, max(-xs, 0));
            }
            const floatx4 zero = {0.f, 0.f, 0.f, 0.f};
            h[q][w] = to_half4(mfma16x16x32(v, coefx[0], zero));
        }
        if (q < NT - 1) continue;
        const int s = q - (NT - 1), R = Y0 + 16 * s;      // output step completed by this tile
        if (R >= p.H) break;                              // uniform
        floatx4 acc[NW];
#pragma unroll
        for (int w = 0; w < NW; ++w) {
            acc[w] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int j = 0; j < NK; ++j) {
                const half4 lo = h[s + 2 * j][w];
                const half4 hi = (2 * j + 1 < NT) ? h[s + 2 * j + 1][w] : half4{0, 0, 0, 0};
                acc[w] = mfma16x16x32(join(lo, hi), coefy[j], acc[w]);
            }
        }
        float* const dst = p.out + (int64_t)R * p.out_pitch + x0;
        if (INSIDE && R + 16 <= p.H) store_rows_via_lds<NW, true>(patch, dst, (uint32_t)p.out_pitch, acc, lane);
        else store_rows_via_lds_masked<NW, true>(patch, dst, p.out_pitch, acc, lane, p.H - R, p.W - x0);
    }
}
constexpr int kSepMinWidth = 8;               // of an image for those loads

template <int NT, int NS>
__global__ void __launch_bounds__(256) sepblur_mfma_kernel(SepArgs p) {
    __shared__ __attribute__((aligned(16))) float s_patch[4][RowPatch<HB_SEP_TILES>::kFloats];
    const int lane = threadIdx.x & 63;
    const int xw = p.ax + (p.ax & 1);         // window start, left of the tile
    // of every 32 workgroups an XCD takes four neighbours (measured on 4096 x 4096 / 8192 x 8192: this
    // order 24.1 / 84.7 us, one contiguous eighth of the tasks per XCD 24.2 / 97.7, plain order 26.4 / 87.3)
    const int task = __builtin_amdgcn_readfirstlane(xcd_blocked(blockIdx.x, gridDim.x, 4) * 4 + (threadIdx.x >> 6));
    if (task >= p.nct * p.nseg) return;
    const int seg = task / p.nct, ct = task - seg * p.nct;
    const int x0 = 16 * HB_SEP_TILES * ct, Y0 = 16 * NS * seg;
    float* patch = s_patch[threadIdx.x >> 6];
    if (ct >= p.c0 && ct < p.c1) sep_task<NT, NS, true>(p, patch, x0, Y0, xw, lane);
    else sep_task<NT, NS, false>(p, patch, x0, Y0, xw, lane);
}

// Two or three windows per tile (18 to 64 taps along x).  Straight from memory every pixel would be requested
// NKX times along x, by loads that touch 16 rows each; here a workgroup of four strips marches down 128
// columns, the pixels under them pass through LDS (two row tiles, clamped when they are requested; row pitch an
// odd multiple of 16 bytes: conflict-free), and the windows are LDS reads.  Three row tiles are in flight
// in registers; NT filtered ones are kept.  128 registers, four workgroups per compute unit (three: 29 us
// instead of 19 at 4096 x 4096, 31 taps).  4096 x 4096 with 31 / 64 taps 28.2 / 41.7 -> 19.0 / 22.3 us, a copy of the
// same bytes 18.3; all its pixels staged before the first product, four workgroups of 64 rows deep, 34.6 / 53.
constexpr int kSepAhead = 3;
template <int NKX>
struct SepMarch {
    static constexpr int kChunks = (kSepMarchCols - 16 + 32 * NKX) / 8;   // of 8 pixels, per row
    static constexpr int kPitch = 8 * (kChunks | 1);
};
template <int NKX, int NT, bool FULL>
__device__ __forceinline__ void sep_march(const SepArgs& p, half_t* s_px, float* patch, int x0, int Y0, int nsteps, int lane, int wv) {
    using S = SepMarch<NKX>;
    constexpr int NW = HB_SEP_TILES, NK = (NT + 1) / 2, kPieces = (16 * S::kChunks + 255) / 256;
    const int c = lane & 15, g = lane >> 4, tid = threadIdx.x;
    const int xw = x0 - p.ax - (p.ax & 1);                // first pixel staged
    const half_t* const src = p.in + (FULL ? xw : 0);
    const int ntiles = nsteps + NT - 1;
    int prow[kPieces], pcol[kPieces];
#pragma unroll
    for (int u = 0; u < kPieces; ++u) {
        const int i = min(tid + 256 * u, 16 * S::kChunks - 1);        // the last threads repeat the last piece
        prow[u] = i / S::kChunks;
        pcol[u] = 8 * (i - prow[u] * S::kChunks);
    }
    auto load_tile = [&](int q, half8 (&v)[kPieces]) {
#pragma unroll
        for (int u = 0; u < kPieces; ++u) {
            const int yr = clampi(Y0 - p.ay + 16 * min(q, ntiles - 1) + prow[u], 0, p.H - 1);
            const uint32_t off = (uint32_t)yr * (uint32_t)p.in_pitch + (uint32_t)(FULL ? pcol[u] : clampi(xw + pcol[u], 0, p.W - 8));
            v[u] = ldg8(src, 2u * off);
        }
    };
    half8 ahead[kSepAhead][kPieces];
#pragma unroll
    for (int d = 0; d < kSepAhead; ++d) load_tile(d, ahead[d]);
    half8 coefx[NKX], coefy[NK];
    sep_fragments<NKX, NK>(p, c, g, coefx, coefy);
    half4 h[NT][NW];                                      // row-filtered tiles q - NT + 1 .. q, rounded to fp16
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int w = 0; w < NW; ++w) h[t][w] = half4{0, 0, 0, 0};
    auto tile = [&](int q) {
        half_t* const buf = s_px + (q & 1) * 16 * S::kPitch;
#pragma unroll
        for (int u = 0; u < kPieces; ++u) {
            half8 v = ahead[0][u];
            if (!FULL) {                                  // see sep_task
                v = shift_in_from_right(v, max(xw + pcol[u] - (p.W - 8), 0));
                v = shift_in_from_left(v, max(-xw - pcol[u], 0));
            }
            *reinterpret_cast<half8*>(buf + prow[u] * S::kPitch + pcol[u]) = v;
        }
#pragma unroll
        for (int d = 0; d + 1 < kSepAhead; ++d)
#pragma unroll
            for (int u = 0; u < kPieces; ++u) ahead[d][u] = ahead[d + 1][u];
        load_tile(q + kSepAhead, ahead[kSepAhead - 1]);
        lds_barrier();                                // also: nobody reads the other buffer any more
#pragma unroll
        for (int t = 0; t + 1 < NT; ++t)
#pragma unroll
            for (int w = 0; w < NW; ++w) h[t][w] = h[t + 1][w];
        const half_t* const px = buf + c * S::kPitch + 16 * NW * wv + 8 * g;
#pragma unroll
        for (int w = 0; w < NW; ++w) {
            floatx4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int kk = 0; kk < NKX; ++kk)
                acc = mfma16x16x32(*reinterpret_cast<const half8*>(px + 16 * w + 32 * kk), coefx[kk], acc);
            h[NT - 1][w] = to_half4(acc);
        }
    };
#pragma unroll
    for (int q = 0; q < NT - 1; ++q) tile(q);
#pragma unroll 1
    for (int s = 0; s < nsteps; ++s) {
        tile(s + NT - 1);
        const int R = Y0 + 16 * s;
        floatx4 acc[NW];
#pragma unroll
        for (int w = 0; w < NW; ++w) {
            acc[w] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int j = 0; j < NK; ++j)
                acc[w] = mfma16x16x32(join(h[2 * j][w], 2 * j + 1 < NT ? h[2 * j + 1 < NT ? 2 * j + 1 : 0][w] : half4{0, 0, 0, 0}), coefy[j], acc[w]);
        }
        const int x = x0 + 16 * NW * wv;
        float* const dst = p.out + (int64_t)R * p.out_pitch + x;
        if (FULL) store_rows_via_lds<NW, true>(patch, dst, (uint32_t)p.out_pitch, acc, lane);
        else if (x < p.W) store_rows_via_lds_masked<NW, true>(patch, dst, p.out_pitch, acc, lane, p.H - R, p.W - x);
    }
}

template <int NKX, int NT>
__global__ void __launch_bounds__(256, 4) sepblur_march_mfma_kernel(SepArgs p) {
    using S = SepMarch<NKX>;
    __shared__ __attribute__((aligned(16))) half_t s_px[2 * 16 * S::kPitch];
    __shared__ __attribute__((aligned(16))) float s_patch[4][RowPatch<HB_SEP_TILES>::kFloats];
    const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int task = xcd_blocked(blockIdx.x, gridDim.x, 4);
    const int seg = task / p.nct, ct = task - seg * p.nct;
    const int x0 = kSepMarchCols * ct, Y0 = 16 * p.steps * seg;
    const int nsteps = min(p.steps, (p.H - Y0 + 15) / 16);
    const int xw = x0 - p.ax - (p.ax & 1);
    if (xw >= 0 && xw + 8 * S::kChunks <= p.W && Y0 + 16 * nsteps <= p.H)
        sep_march<NKX, NT, true>(p, s_px, s_patch[wv], x0, Y0, nsteps, lane, wv);
    else
        sep_march<NKX, NT, false>(p, s_px, s_patch[wv], x0, Y0, nsteps, lane, wv);
}

// ---------------------------------------------------------------------------
// Vector-ALU twin: 32 x 64 output tile per workgroup; pixels with halo in LDS (column and row indices
// clamped, the definition's border rule verbatim), row pass to an LDS intermediate (rounded to fp16 like
// the matrix kernel's, kept as fp32), column pass from it.  Both passes are register-blocked: a thread
// owns 8 consecutive outputs of a row (of a column) and reads 8 taps and 8 new samples per 64 FMAs.
// Taps are padded with zeros to a multiple of 8.
constexpr int kVTH = 32, kVTW = 64;
constexpr int kVRows = kVTH + HB_MAX_TAPS;              // 96: rows the column pass may touch
constexpr int kVPxPitch = kVTW + HB_MAX_TAPS + 8;       // 136 halves

__global__ void __launch_bounds__(256) sepblur_valu_kernel(SepArgs p) {
    __shared__ __attribute__((aligned(16))) half_t s_px[kVRows * kVPxPitch];
    __shared__ __attribute__((aligned(16))) float s_tmp[kVRows * kVTW];
    __shared__ __attribute__((aligned(16))) float s_kx[HB_MAX_TAPS], s_ky[HB_MAX_TAPS];
    static_assert(HB_MAX_TAPS % 8 == 0, "taps are processed eight at a time");
    if (threadIdx.x < HB_MAX_TAPS) {
        s_kx[threadIdx.x] = (int)threadIdx.x < p.Tx ? (float)tap_at(p.tx.tab, threadIdx.x) : 0.f;
        s_ky[threadIdx.x] = (int)threadIdx.x < p.Ty ? (float)tap_at(p.ty.tab, threadIdx.x) : 0.f;
    }
    const int nctv = (p.W + kVTW - 1) / kVTW;
    const int rt = blockIdx.x / nctv, ct = blockIdx.x - rt * nctv;
    const int x0 = ct * kVTW, y0 = rt * kVTH;
    const int txp = (p.Tx + 7) & ~7, typ = (p.Ty + 7) & ~7;
    const int nrows = kVTH + p.Ty - 1;                     // image rows under the tile
    // staged pixel (r, j) = in[clampH(y0 - ay + r)][clampW(x0 - ax + j)], j < 64 + txp covers every window
    const int nch = (kVTW + txp) / 8;
    for (int idx = threadIdx.x; idx < nrows * nch; idx += 256) {
        const int r = idx / nch, ch = idx - r * nch;
        const half_t* row = p.in + (int64_t)clampi(y0 - p.ay + r, 0, p.H - 1) * p.in_pitch;
        *reinterpret_cast<half8*>(&s_px[r * kVPxPitch + 8 * ch]) = load8_clamp(row, x0 - p.ax + 8 * ch, p.W);
    }
    __syncthreads();
    // row pass: thread = 8 consecutive columns of one staged row
    for (int idx = threadIdx.x; idx < nrows * (kVTW / 8); idx += 256) {
        const int r = idx >> 3, xl = 8 * (idx & 7);
        const half8* src = reinterpret_cast<const half8*>(&s_px[r * kVPxPitch + xl]);
        float acc[8], w[16];
#pragma unroll
        for (int q = 0; q < 8; ++q) acc[q] = 0.f;
        {
            const half8 v = src[0];
#pragma unroll
            for (int i = 0; i < 8; ++i) w[i] = (float)v[i];
        }
        for (int tb = 0; tb < txp; tb += 8) {
            const half8 v = src[tb / 8 + 1];
            const floatx4 ka = *reinterpret_cast<const floatx4*>(&s_kx[tb]), kb = *reinterpret_cast<const floatx4*>(&s_kx[tb + 4]);
#pragma unroll
            for (int i = 0; i < 8; ++i) w[8 + i] = (float)v[i];
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const float kv = i < 4 ? ka[i] : kb[i - 4];
#pragma unroll
                for (int q = 0; q < 8; ++q) acc[q] = fmaf(kv, w[q + i], acc[q]);
            }
#pragma unroll
            for (int i = 0; i < 8; ++i) w[i] = w[8 + i];
        }
        floatx4* dst = reinterpret_cast<floatx4*>(&s_tmp[r * kVTW + xl]);
        dst[0] = floatx4{(float)(half_t)acc[0], (float)(half_t)acc[1], (float)(half_t)acc[2], (float)(half_t)acc[3]};
        dst[1] = floatx4{(float)(half_t)acc[4], (float)(half_t)acc[5], (float)(half_t)acc[6], (float)(half_t)acc[7]};
    }
    // rows only the zero taps reach
    for (int idx = nrows * kVTW + threadIdx.x; idx < (kVTH + typ) * kVTW; idx += 256) s_tmp[idx] = 0.f;
    __syncthreads();
    // column pass: thread = 8 consecutive rows of one column
    const int x = threadIdx.x & 63, r0 = 8 * (threadIdx.x >> 6);
    if (x0 + x >= p.W || y0 + r0 >= p.H) return;
    float acc[8], w[16];
#pragma unroll
    for (int q = 0; q < 8; ++q) acc[q] = 0.f;
#pragma unroll
    for (int i = 0; i < 8; ++i) w[i] = s_tmp[(r0 + i) * kVTW + x];
    for (int tb = 0; tb < typ; tb += 8) {
        const floatx4 ka = *reinterpret_cast<const floatx4*>(&s_ky[tb]), kb = *reinterpret_cast<const floatx4*>(&s_ky[tb + 4]);
#pragma unroll
        for (int i = 0; i < 8; ++i) w[8 + i] = s_tmp[(r0 + tb + 8 + i) * kVTW + x];
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const float kv = i < 4 ? ka[i] : kb[i - 4];
#pragma unroll
            for (int q = 0; q < 8; ++q) acc[q] = fmaf(kv, w[q + i], acc[q]);
        }
#pragma unroll
        for (int i = 0; i < 8; ++i) w[i] = w[8 + i];
    }
#pragma unroll
    for (int q = 0; q < 8; ++q)
        if (y0 + r0 + q < p.H) p.out[(int64_t)(y0 + r0 + q) * p.out_pitch + x0 + x] = acc[q];
}

static hb_status sep_prepare(SepArgs& a, const hb_half* in, float* out, int H, int W,
                             int64_t in_pitch, int64_t out_pitch,
                             const hb_half* tx, int ntx, int ax, const hb_half* ty, int nty, int ay) {
    hb_status s = check_image(in, out, H, W, in_pitch, out_pitch);
    if (s != HB_OK) return s;
    // lanes address rows with 32-bit byte offsets from the image base
    if ((int64_t)H * in_pitch >= ((int64_t)1 << 31) || (int64_t)H * out_pitch >= ((int64_t)1 << 30)) return HB_ERR_UNSUPPORTED;
    if ((s = check_taps(tx, ntx, ax)) != HB_OK) return s;
    if ((s = check_taps(ty, nty, ay)) != HB_OK) return s;
    a.in = reinterpret_cast<const half_t*>(in);
    a.out = out;
    a.H = H;
    a.W = W;
    a.in_pitch = in_pitch;
    a.out_pitch = out_pitch;
    a.Tx = ntx;
    a.ax = ax;
    a.Ty = nty;
    a.ay = ay;
    a.nct = a.nseg = a.steps = a.c0 = a.c1 = 0;
    a.tx = pack_taps(tx, ntx);
    a.ty = pack_taps(ty, nty);
    return HB_OK;
}

template <class K>
static hb_status sep_launch(K kernel, hipStream_t st, SepArgs& a, int ns, int cols, int per_wg) {
    a.nct = ceil_div(a.W, cols);
    a.steps = ns;
    a.nseg = ceil_div(a.H, 16 * ns);
    const int64_t tasks = (int64_t)a.nct * a.nseg;
    if (tasks > 0x7fffffff) return HB_ERR_UNSUPPORTED;
    hipLaunchKernelGGL(kernel, dim3((unsigned)((tasks + per_wg - 1) / per_wg)), dim3(256), 0, st, a);
    return launch_status();
}
// One window per tile, where the march is slower: see sep_marches.  4 steps per task, 8 where NT - 1 = 3 extra row tiles weigh
// more and its waves are not too few (8192 x 8192, 16 taps down: 62 us with 4, 68 with 8; 9036 x 9, 38 taps 7.2 with 4, 10.6 with 8), 2 where the rows end after two (16 x 300000, 16 / 64 taps 9.2 and 12.7 us with 4 and
// 2 before, 8.3 and 12.7 with 2).
template <int NT>
static hb_status sep_launch_one_window(hipStream_t st, SepArgs& a) {
    // a strip is interior when all its windows lie inside the row and its tiles are full
    constexpr int cols = 16 * HB_SEP_TILES;
    const int xw = a.ax + (a.ax & 1), nct = ceil_div(a.W, cols);
    const int after = cols - 16 - xw + 32;
    interior_range(nct, cols, xw, after > cols ? after : cols, a.W, a.c0, a.c1);
    if (a.H <= 32) return sep_launch(sepblur_mfma_kernel<NT, 2>, st, a, 2, cols, 4);
    if constexpr (NT == 4) {
        if (a.H >= sep_wide_rows(NT) && 2 * (int64_t)ceil_div(a.H, 128) * nct >= 15 * num_cu()) return sep_launch(sepblur_mfma_kernel<NT, 8>, st, a, 8, cols, 4);
    }
    return sep_launch(sepblur_mfma_kernel<NT, 4>, st, a, 4, cols, 4);
}
// Row tiles (steps) of a segment of the march.  Every segment requests and filters NT - 1 row tiles ahead of its own, so
// long ones save work: as long as leaves two workgroups per compute unit (1079 x 1917, 31 / 60 taps 7.4 / 8.8 us, with
// the four that are resident 8.7 / 11.3; 2048 x 2048, 31 / 64 taps 8.6 / 10.3 and 9.4 / 11.9; with one 9.1 / 10.5), of eight steps
// at most (8192 x 4096, 48 taps: 36 us with 8 steps, 42 with 16).  From about ten steps per unit (`all` in all columns) up to where
// both rules give eight, something else weighs more:
//  - Output rows of whole lines, or of half lines under more than 17 taps down: three or four workgroups a unit hide more
//    of each other's loads (3072 x 3072, 31 / 48 / 64 taps 12.8 / 13.1 / 14.3 us, with two 14.1 / 14.3 / 15.9; 2160 x 3840, 40 x 5 taps 10.8 and 11.9;
//    1500 x 6000, 31 / 64 taps 13.7 / 14.8 and 14.3 / 16.3; 3600 x 3600, 48 taps 18.6 and 19.7).
//  - Other rows: two or three steps.  The parts of a line that two workgroups write meet in the L2 only while these keep in step,
//    which they do for a few rows, and with short filters that weighs more in smaller images too (3000 x 3000, 16 / 31 / 48 taps 13.6 /
//    16.7 / 17.1 us, with eight steps 17.5 / 18.3 / 18.8; 1800 x 1808, 16 taps 6.7, with four 7.0; 2000 x 3000, 16 x 33 taps 10.9, with six 11.9; 2700 x
//    1500, 31 taps 9.3, with four 9.9).  Where input rows start between dwords a row tile costs more: only in large images, and three
//    (3333 x 3333, 5 / 31 / 48 taps 20.1 / 20.7 / 21.8, with eight 23.7 / 24.4 / 24.4; 64 taps 23.9 with five, 25.0 with three; 1801 x 1811, 5 / 31 taps
//    9.1 / 10.4 with two, 8.1 / 9.7 with the four that two workgroups a unit give; 2401 x 2603 14.0 / 15.0 and 13.2 / 14.3).
static int sep_march_steps(const SepArgs& a, int nkx, int nt, bool lines) {
    const int64_t cu = num_cu(), rowsteps = ceil_div(a.H, 16), nct = ceil_div(a.W, kSepMarchCols), all = rowsteps * nct;
    auto steps_for = [&](int64_t wgs) { return (int)std::min<int64_t>((all + wgs - 1) / wgs, 8); };
    const int two = steps_for(2 * cu);
    const bool half_lines = a.out_pitch % 16 == 0 && aligned_to(a.out, 64), even = a.in_pitch % 2 == 0 && aligned_to(a.in, 4);
    if (all <= 4 * cu || all > 28 * cu) return two;
    if (lines || (half_lines && nt > 2)) {
        if (nt <= 3) return all > (nt == 3 ? 10 : 8) * cu ? steps_for(4 * cu) : two;
        return all > 24 * cu ? steps_for(4 * cu) : all > 16 * cu ? steps_for(3 * cu) : two;
    }
    if (!even) return all <= 16 * cu ? two : nt <= 4 ? 3 : 5;
    const int few = all > 20 * cu ? 3 : 2;
    if (nt <= 2) return half_lines && nkx >= 2 && all <= 8 * cu ? two : few;
    if (all > 24 * cu) return steps_for(4 * cu);
    if (all > 16 * cu) return nt == 3 ? few : nt == 4 ? 3 : two;
    if (nt > 3 || (all > 8 * cu && all <= 10 * cu)) return two;
    if (all > 10 * cu) return nkx == 1 ? 2 : two;
    return 8 * nct * ((rowsteps + two - 1) / two) >= 15 * cu ? 2 : two;       // nearly two workgroups to every unit
}
template <int NT>
static hb_status sep_launch_nt(int nkx, hipStream_t st, SepArgs& a) {
    const bool lines = a.out_pitch % 32 == 0 && aligned_to(a.out, 128);
    if (nkx == 1 && !sep_marches({a.H, a.W, NT, a.in_pitch % 2 == 0 && aligned_to(a.in, 4), lines, num_cu()})) return sep_launch_one_window<NT>(st, a);
    const int steps = sep_march_steps(a, nkx, NT, lines);
    if (nkx == 1) return sep_launch(sepblur_march_mfma_kernel<1, NT>, st, a, steps, kSepMarchCols, 1);
    if (nkx == 2) return sep_launch(sepblur_march_mfma_kernel<2, NT>, st, a, steps, kSepMarchCols, 1);
    return sep_launch(sepblur_march_mfma_kernel<3, NT>, st, a, steps, kSepMarchCols, 1);
}

}  // namespace hb

extern "C" hb_status hb_sepblur_valu(const hb_half* in, float* out, int H, int W,
                                     int64_t in_pitch, int64_t out_pitch,
                                     const hb_half* taps_x_host, int ntaps_x, int anchor_x,
                                     const hb_half* taps_y_host, int ntaps_y, int anchor_y, hb_stream stream);

extern "C" hb_status hb_sepblur(const hb_half* in, float* out, int H, int W,
                                int64_t in_pitch, int64_t out_pitch,
                                const hb_half* taps_x_host, int ntaps_x, int anchor_x,
                                const hb_half* taps_y_host, int ntaps_y, int anchor_y, hb_stream stream) {
    using namespace hb;
    SepArgs a;
    hb_status s = sep_prepare(a, in, out, H, W, in_pitch, out_pitch, taps_x_host, ntaps_x, anchor_x,
                              taps_y_host, ntaps_y, anchor_y);
    if (s != HB_OK) return s;
    const int nkx = ceil_div(15 + ntaps_x + (anchor_x & 1), 32);          // 1 .. 3
    if (W < kSepMinWidth)
        return hb_sepblur_valu(in, out, H, W, in_pitch, out_pitch, taps_x_host, ntaps_x, anchor_x,
                               taps_y_host, ntaps_y, anchor_y, stream);
    hipStream_t st = reinterpret_cast<hipStream_t>(stream);
    switch ((ntaps_y + 30) / 16) {
        case 1: return sep_launch_nt<1>(nkx, st, a);
        case 2: return sep_launch_nt<2>(nkx, st, a);
        case 3: return sep_launch_nt<3>(nkx, st, a);
        case 4: return sep_launch_nt<4>(nkx, st, a);
        default: return sep_launch_nt<5>(nkx, st, a);
    }
}

extern "C" hb_status hb_sepblur_valu(const hb_half* in, float* out, int H, int W,
                                     int64_t in_pitch, int64_t out_pitch,
                                     const hb_half* taps_x_host, int ntaps_x, int anchor_x,
                                     const hb_half* taps_y_host, int ntaps_y, int anchor_y, hb_stream stream) {
    using namespace hb;
    SepArgs a;
    hb_status s = sep_prepare(a, in, out, H, W, in_pitch, out_pitch, taps_x_host, ntaps_x, anchor_x,
                              taps_y_host, ntaps_y, anchor_y);
    if (s != HB_OK) return s;
    const int64_t blocks = (int64_t)ceil_div(H, kVTH) * ceil_div(W, kVTW);
    if (blocks > 0x7fffffff) return HB_ERR_UNSUPPORTED;
    hipLaunchKernelGGL(sepblur_valu_kernel, dim3((unsigned)blocks), dim3(256), 0,
                       reinterpret_cast<hipStream_t>(stream), a);
    return launch_status();
}
