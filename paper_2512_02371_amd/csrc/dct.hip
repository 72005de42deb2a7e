// hb_dct_denoise: transform-domain coring on overlapping windowed 16 x 16 tiles, and its
// vector-ALU twin (Sec. V-E): window, DCT down the columns and along the rows, small bins set to
// zero, the two inverse transforms, window again; the overlapping tiles are blended and the
// windowing undone.
//
// As in the paper the four 16 x 16 matrix products of a tile and the coring between them are fused.
// The paper keeps the blend as a second launch; here the matrix-unit path blends inside the same
// kernel (a workgroup owns a patch of the output and accumulates its tiles in LDS), which saves
// writing and re-reading 1 KB per tile; the vector-ALU twin keeps the two-launch structure with the
// tiles in the workspace.  What the products hand on stays fp32: DCT coefficients reach 16 times the
// pixel range, so fp16 intermediates would cost about 1e-3 of absolute accuracy per rounding.
//
// Every product contracts over the ROW index of what the one before left in its accumulators (lane
// (c, g) holds rows 4g + j of column c), with the accumulators as the A operand: instruction j of the
// next product (K = 4) takes register j as it is, if slot g of its B operand stands for row 4g + j.  The
// result's rows are the old columns, so the next product contracts over the other axis:
//     Q[r][v] = sum_x P[r][x] E[v][x]     Y[v][u] = sum_r Q[r][v] E[u][r]        (E[u][i] = D[u][i] w[i])
//     R[u][x] = sum_v Y[v][u] E[v][x]     rec[x][r] = sum_u R[u][x] E[u][r]
// No transpose and no LDS between the four, and rec ends with four consecutive pixels of a row per lane.
// The windows are part of E.
#include <math.h>

#include "hb_device.hpp"
#include "hb_host.hpp"

namespace hb {

constexpr int kDctWaves = 4;                  // waves per workgroup
constexpr int kDctPitch = 17;                 // floats per row of an LDS tile (conflict-free both ways)

struct DctTables {
    float d[256];                             // D[u][i], orthonormal DCT-II, row-major
    float w[16];                              // sine window
    float e[256];                             // E[u][i] = D[u][i] w[i]
};

struct DctArgs : DctTables {
    const half_t* in;
    float* out;
    float* tiles;                             // workspace: [C][nty][ntx][16][16] windowed reconstructions
    int C, H, W, nty, ntx;
    int64_t in_pitch, in_plane, out_pitch, out_plane;
    float threshold;
};

// acc (lane (c, g): rows 4g + j of column c) -> LDS tile [row][column]
__device__ __forceinline__ void dct_put(float* tile, const floatx4& acc, int c, int g) {
#pragma unroll
    for (int j = 0; j < 4; ++j) tile[(4 * g + j) * kDctPitch + c] = acc[j];
}

__device__ __forceinline__ void dct_tile_origin(const DctArgs& p, int64_t t, int& plane, int& y0, int& x0) {
    const int per_plane = p.nty * p.ntx;
    plane = (int)(t / per_plane);
    const int r = (int)(t - (int64_t)plane * per_plane);
    y0 = 8 * (r / p.ntx);
    x0 = 8 * (r % p.ntx);
}

// ---------------------------------------------------------------------------
// The matrix-unit path in ONE launch: transform, core, transform back AND blend.  A workgroup owns a
// 64 x 64 patch of the output and runs every tile that overlaps it (up to 9 x 9; the tiles on the rim
// are run by the neighbouring patch as well, 1.27x the products), adding the windowed reconstructions
// into an fp32 image of the patch in LDS instead of writing 1 KB per tile to memory and reading it
// back.  Tiles overlap their neighbours at stride 8, tiles at stride 16 do not: the tiles are taken in
// four rounds by the parity of their (row, column) index, within a round the waves add to disjoint
// pixels with plain loads and stores, and the order of the four additions into a pixel is fixed.
//
// What bounds it: the fp32 products, 12 x 32 cycles a tile and SIMD (the first product, whose pixels are
// fp16, is two K = 32 products with E as three fp16 parts, together the fp32 number, instead of four more; two parts
// alone hold 22 of its 24 bits and save 0.2 us), 1.27x for the rim tiles of 64 x 64 patches.  3 x 1024 x 1024: 33.0 ->
// 22.5 us against four fp32 products with an LDS transpose between each two; 61 tiles a SIMD x 416 cycles of products
// are 12.5 us of it.  Error against fp64 0.92 of that kernel's on average over images from 64 x 64 to 4 M pixels and
// thresholds from 0 to 0.5 (1.1 of it above 0.35, where little but the DC bin is left).
constexpr int kDfWaves = 8;
template <int PATCH>
struct DfGeom {
    static constexpr int kPitch = PATCH + 4;              // 16 rows of a tile: 16-byte pieces in different banks
    static constexpr int kRegion = PATCH + 16;            // pixels under the tiles of a patch, per axis
    static constexpr int kPxPitch = kRegion + 8;
};
constexpr float kDfScale = 1024.f;                        // of the first product's E: keeps its low part a normal fp16 number

template <int PATCH>
__global__ void __launch_bounds__(64 * kDfWaves) dct_fused_mfma_kernel(DctArgs p) {
    using G = DfGeom<PATCH>;
    __shared__ __attribute__((aligned(16))) float s_acc[PATCH * G::kPitch];
    __shared__ __attribute__((aligned(16))) half_t s_px[G::kRegion * G::kPxPitch];
    __shared__ float s_w2[16];
    const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int c = lane & 15, g = lane >> 4;
    const int npx = (p.W + PATCH - 1) / PATCH, npy = (p.H + PATCH - 1) / PATCH;
    // every XCD takes one contiguous run of the patches: the 8-pixel rims that neighbouring patches share
    // (whole 128-byte lines in memory) are fetched into one L2 once (measured reads 1.05x the image
    // instead of 2.9x)
    int wg = xcd_contiguous(blockIdx.x, gridDim.x);
    const int pc = wg % npx;
    wg /= npx;
    const int pr = wg % npy, plane = wg / npy;
    const int py0 = PATCH * pr, px0 = PATCH * pc;
    // the pixels under every tile of the patch: rows py0 - 8 .. py0 + PATCH + 7, columns px0 - 8 .. px0 + PATCH + 7
    // (what lies outside the image is under no tile and is never read)
    {
        const half_t* plane_px = p.in + (int64_t)plane * p.in_plane;
        for (int i = threadIdx.x; i < G::kRegion * (G::kRegion / 8); i += 64 * kDfWaves) {
            const int r = i / (G::kRegion / 8), ch = i - r * (G::kRegion / 8);
            const int y = py0 - 8 + r, x = px0 - 8 + 8 * ch;
            if (y >= 0 && y < p.H && x >= 0 && x < p.W)       // W is a multiple of 8: whole chunks
                *reinterpret_cast<half8*>(&s_px[r * G::kPxPitch + 8 * ch]) =
                    *reinterpret_cast<const half8_u*>(plane_px + (int64_t)y * p.in_pitch + x);
        }
    }
    for (int i = threadIdx.x; i < PATCH * G::kPitch / 4; i += 64 * kDfWaves)
        *reinterpret_cast<floatx4*>(&s_acc[4 * i]) = floatx4{0.f, 0.f, 0.f, 0.f};
    if (threadIdx.x < 16) s_w2[threadIdx.x] = p.w[threadIdx.x] * p.w[threadIdx.x];
    half8 e1, e0 = {0, 0, 0, 0, 0, 0, 0, 0};  // E[c][4g + j] as hi (slots 0..3) and lo (4..7), which share a pixel; the rest
    float ef[4], eb[4];                       // E[c][4g + j] (undoing the scale of the first product), E[4g + j][c]
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const float v = kDfScale * p.e[c * 16 + 4 * g + j];
        e1[j] = (half_t)v;
        e1[4 + j] = (half_t)(v - (float)e1[j]);
        e0[j] = (half_t)(v - (float)e1[j] - (float)e1[4 + j]);
        ef[j] = (1.f / kDfScale) * p.e[c * 16 + 4 * g + j];
        eb[j] = p.e[(4 * g + j) * 16 + c];
    }
    const float cut0 = c == 0 && g == 0 ? -1.f : p.threshold;   // the DC bin always stays
    const int lane_px = (c + 8 - py0) * G::kPxPitch + 4 * g + 8 - px0, lane_acc = (c - py0) * G::kPitch + 4 * g - px0;
    // tiles (ty, tx), origin (8 ty, 8 tx), that overlap the patch
    const int ty_lo = max(py0 / 8 - 1, 0), ty_hi = min(py0 / 8 + PATCH / 8 - 1, p.nty - 1);
    const int tx_lo = max(px0 / 8 - 1, 0), tx_hi = min(px0 / 8 + PATCH / 8 - 1, p.ntx - 1);
    __syncthreads();
    for (int round = 0; round < 4; ++round) {
        const int ty0 = ty_lo + ((ty_lo ^ (round >> 1)) & 1), tx0 = tx_lo + ((tx_lo ^ round) & 1);
        const int ny = ty0 <= ty_hi ? (ty_hi - ty0) / 2 + 1 : 0, nx = tx0 <= tx_hi ? (tx_hi - tx0) / 2 + 1 : 0;
        const int inv = nx > 0 ? 65536 / nx + 1 : 0;      // i / nx = i * inv >> 16 for the few tiles of a round
        for (int i = wv; i < ny * nx; i += kDfWaves) {
            const int row = (i * inv) >> 16;
            const int ty = ty0 + 2 * row, tx = tx0 + 2 * (i - row * nx);
            // lane (c = row, g) reads pixels (row, 4g .. 4g + 3)
            const half4 px = *reinterpret_cast<const half4*>(&s_px[lane_px + 8 * (ty * G::kPxPitch + tx)]);
            const floatx4 zero = {0.f, 0.f, 0.f, 0.f};
            const floatx4 q = mfma16x16x32(join(px, px), e1, mfma16x16x32(join(px, px), e0, zero));
            floatx4 y = zero;
#pragma unroll
            for (int j = 0; j < 4; ++j) y = mfma16x16x4f32(q[j], ef[j], y);
            // coring: lane (c = u, g) holds bins (u, v = 4g + j)
#pragma unroll
            for (int j = 0; j < 4; ++j)
                if (fabsf(y[j]) < (j == 0 ? cut0 : p.threshold)) y[j] = 0.f;
            floatx4 r = zero, rec = zero;
#pragma unroll
            for (int j = 3; j >= 0; --j) r = mfma16x16x4f32(y[j], eb[j], r);     // the large low bins last
#pragma unroll
            for (int j = 3; j >= 0; --j) rec = mfma16x16x4f32(r[j], eb[j], rec);
            // lane (c = row, g) holds pixels 4g .. 4g + 3 of its row: add the part inside the patch
            const uint32_t xx = 8 * tx - px0 + 4 * g, yy = 8 * ty - py0 + c;
            if (xx < PATCH && yy < PATCH) {
                floatx4* const dst = reinterpret_cast<floatx4*>(&s_acc[lane_acc + 8 * (ty * G::kPitch + tx)]);
                *dst = *dst + rec;
            }
        }
        __syncthreads();
    }
    // out = sum of the windowed reconstructions / sum of the squared windows of the tiles covering the pixel
    // (the tiles covering a pixel are a product set, so the denominator is a product of two 1-D sums)
    auto covered = [&](int z, int n) {                    // z / 8 - 1 and z / 8: the tiles over pixel z of an axis of n tiles
        const int t = z >> 3, i = z & 7;
        return (t >= 1 ? s_w2[i + 8] : 0.f) + (t < n ? s_w2[i] : 0.f);
    };
    for (int idx = threadIdx.x; idx < PATCH * (PATCH / 4); idx += 64 * kDfWaves) {
        const int r = idx / (PATCH / 4), q4 = idx - r * (PATCH / 4);
        const int y = py0 + r, x = px0 + 4 * q4;
        if (y >= p.H || x >= p.W) continue;
        const float dy = covered(y, p.nty);
        const floatx4 v = *reinterpret_cast<const floatx4*>(&s_acc[r * G::kPitch + 4 * q4]);
        floatx4 o;
#pragma unroll
        for (int q = 0; q < 4; ++q) o[q] = v[q] / (dy * covered(x + q, p.ntx));
        *reinterpret_cast<floatx4_u*>(p.out + (int64_t)plane * p.out_plane + (int64_t)y * p.out_pitch + x) = o;
    }
}

// Vector-ALU twin: the same four products as plain dot products over LDS tiles.
// out[i][j] = sum_k A[i * ai + k * ak] * B[k * bk + j * bj], lane (c, g) computes rows 4g + jj of column c.
__device__ __forceinline__ void dct_mm_valu(const float* A, int ai, int ak, const float* B, int bk, int bj,
                                            floatx4& acc, int c, int g) {
#pragma unroll
    for (int jj = 0; jj < 4; ++jj) {
        float s = 0.f;
        for (int k = 0; k < 16; ++k) s = fmaf(A[(4 * g + jj) * ai + k * ak], B[k * bk + c * bj], s);
        acc[jj] = s;
    }
}

__global__ void __launch_bounds__(64 * kDctWaves) dct_transform_valu_kernel(DctArgs p) {
    __shared__ float s_tile[kDctWaves][2][16 * kDctPitch];
    __shared__ float s_d[16 * kDctPitch];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int c = lane & 15, g = lane >> 4;
    for (int i = threadIdx.x; i < 256; i += 64 * kDctWaves) s_d[(i >> 4) * kDctPitch + (i & 15)] = p.d[i];
    __syncthreads();
    float* ta = s_tile[wv][0];
    float* tb = s_tile[wv][1];
    const int64_t ntiles = (int64_t)p.C * p.nty * p.ntx;
    const int64_t stride = (int64_t)gridDim.x * kDctWaves;
    for (int64_t t = (int64_t)blockIdx.x * kDctWaves + wv; t < ntiles; t += stride) {
        int plane, y0, x0;
        dct_tile_origin(p, t, plane, y0, x0);
        const half_t* src = p.in + (int64_t)plane * p.in_plane + (int64_t)y0 * p.in_pitch + x0;
        floatx4 acc;
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[j] = (float)src[(int64_t)(4 * g + j) * p.in_pitch + c] * p.w[4 * g + j] * p.w[c];
        dct_put(ta, acc, c, g);                                       // T [row][col]
        wave_lds_fence();
        dct_mm_valu(ta, kDctPitch, 1, s_d, 1, kDctPitch, acc, c, g);  // Q[r][v] = sum_col T[r][col] D[v][col]
        dct_put(tb, acc, c, g);
        wave_lds_fence();
        dct_mm_valu(s_d, kDctPitch, 1, tb, kDctPitch, 1, acc, c, g);  // Y[u][v] = sum_r D[u][r] Q[r][v]
#pragma unroll
        for (int j = 0; j < 4; ++j)
            if (fabsf(acc[j]) < p.threshold && !(c == 0 && g == 0 && j == 0)) acc[j] = 0.f;
        dct_put(ta, acc, c, g);
        wave_lds_fence();
        dct_mm_valu(s_d, 1, kDctPitch, ta, kDctPitch, 1, acc, c, g);  // R[r][v] = sum_u D[u][r] Y[u][v]
        dct_put(tb, acc, c, g);
        wave_lds_fence();
        dct_mm_valu(tb, kDctPitch, 1, s_d, kDctPitch, 1, acc, c, g);  // rec[r][col] = sum_v R[r][v] D[v][col]
        float* dst = p.tiles + t * 256;
#pragma unroll
        for (int j = 0; j < 4; ++j) dst[(4 * g + j) * 16 + c] = acc[j] * p.w[4 * g + j] * p.w[c];
        wave_lds_fence();
    }
}

// 2  blend: out = sum over the (up to four) tiles covering a pixel of their windowed
// reconstruction, divided by the sum of their squared windows.  A thread owns four consecutive pixels.
__global__ void __launch_bounds__(256) dct_blend_kernel(DctArgs p) {
    // a workgroup covers 16 rows x 64 columns: the 64-byte rows of a tile it reads share their
    // cache lines with the rows above and below, which the same workgroup reads as well
    const int bx_n = (p.W + 63) / 64, by_n = (p.H + 15) / 16;
    int wg = blockIdx.x;
    const int bx = wg % bx_n;
    wg /= bx_n;
    const int by = wg % by_n, plane = wg / by_n;
    const int y = 16 * by + (threadIdx.x >> 4), x = 64 * bx + 4 * (threadIdx.x & 15);
    if (y >= p.H || x >= p.W) return;
    floatx4 num = {0.f, 0.f, 0.f, 0.f}, den = {0.f, 0.f, 0.f, 0.f};
    for (int ty = y / 8 - 1; ty <= y / 8; ++ty) {
        if (ty < 0 || ty >= p.nty) continue;
        const int r = y - 8 * ty;
        for (int tx = x / 8 - 1; tx <= x / 8; ++tx) {
            if (tx < 0 || tx >= p.ntx) continue;
            const int cc = x - 8 * tx;
            const float* tile = p.tiles + (((int64_t)plane * p.nty + ty) * p.ntx + tx) * 256;
            const floatx4 v = *reinterpret_cast<const floatx4*>(tile + r * 16 + cc);
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const float ww = p.w[r] * p.w[cc + q];
                num[q] += v[q];
                den[q] += ww * ww;
            }
        }
    }
    float* dst = p.out + (int64_t)plane * p.out_plane + (int64_t)y * p.out_pitch + x;
#pragma unroll
    for (int q = 0; q < 4; ++q) dst[q] = num[q] / den[q];
}

static DctTables dct_tables() {
    DctTables a;
    const double pi = 3.14159265358979323846;
    for (int u = 0; u < 16; ++u)
        for (int i = 0; i < 16; ++i)
            a.d[u * 16 + i] = (float)(u == 0 ? 0.25 : sqrt(2.0 / 16.0) * cos(pi * (2.0 * i + 1.0) * u / 32.0));
    for (int i = 0; i < 16; ++i) a.w[i] = (float)sin(pi * (i + 0.5) / 16.0);
    for (int u = 0; u < 16; ++u)
        for (int i = 0; i < 16; ++i)
            a.e[u * 16 + i] = (float)((u == 0 ? 0.25 : sqrt(2.0 / 16.0) * cos(pi * (2.0 * i + 1.0) * u / 32.0)) * sin(pi * (i + 0.5) / 16.0));
    return a;
}

static hb_status dct_run(bool valu, const hb_half* in, float* out, int C, int H, int W,
                         int64_t in_pitch, int64_t in_plane, int64_t out_pitch, int64_t out_plane,
                         float threshold, void* workspace, size_t workspace_bytes, hb_stream stream) {
    if (!in || !out) return HB_ERR_INVALID_ARG;
    if (C < 1 || H < 16 || W < 16 || (H & 7) || (W & 7)) return HB_ERR_INVALID_ARG;
    if (in_pitch < W || out_pitch < W) return HB_ERR_INVALID_ARG;
    if (C > 1 && (in_plane < (int64_t)H * in_pitch || out_plane < (int64_t)H * out_pitch)) return HB_ERR_INVALID_ARG;
    if (!aligned_to(in, 2) || !aligned_to(out, 4)) return HB_ERR_INVALID_ARG;
    if (!(threshold >= 0.f)) return HB_ERR_INVALID_ARG;                // also rejects NaN
    if (C > 65535 || (int64_t)C * H * W > ((int64_t)1 << 40)) return HB_ERR_UNSUPPORTED;
    const size_t need = hb_dct_denoise_workspace_size(C, H, W);
    if (!workspace || workspace_bytes < need || !aligned_to(workspace, 256)) return HB_ERR_WORKSPACE;

    DctArgs a;
    a.in = reinterpret_cast<const half_t*>(in);
    a.out = out;
    a.tiles = reinterpret_cast<float*>(workspace);
    a.C = C;
    a.H = H;
    a.W = W;
    a.nty = H / 8 - 1;
    a.ntx = W / 8 - 1;
    a.in_pitch = in_pitch;
    a.in_plane = in_plane;
    a.out_pitch = out_pitch;
    a.out_plane = out_plane;
    a.threshold = threshold;
    static const DctTables tables = dct_tables();         // computed once: 3 us of the host's 11 per call
    static_cast<DctTables&>(a) = tables;

    hipStream_t st = reinterpret_cast<hipStream_t>(stream);
    const int64_t ntiles = (int64_t)C * a.nty * a.ntx;
    const int64_t wgs = (ntiles + kDctWaves - 1) / kDctWaves;
    const unsigned blocks = (unsigned)(wgs < 4096 ? wgs : 4096);     // waves stride over the tiles
    if (!valu) {
        // one launch: tiles and blend fused, the workspace stays unused
        // 32 x 32 patches (1.56x the products) while there are two of them to a compute unit at most and the larger ones
        // would leave units idle (512 x 512 6.4 us, 10.2 with 64 x 64 patches; 2 x 512 x 512, 512 small ones, 8.8 against 10.3;
        // 720 x 736, 529 small ones, 11.1 against 10.4; 960 x 960 13.7 against 10.7)
        const int64_t patches = (int64_t)C * ceil_div(H, 64) * ceil_div(W, 64);
        const int64_t small = (int64_t)C * ceil_div(H, 32) * ceil_div(W, 32);
        if (patches > 0x7fffffff) return HB_ERR_UNSUPPORTED;
        if (patches < num_cu() && small <= 2 * num_cu())
            hipLaunchKernelGGL(dct_fused_mfma_kernel<32>, dim3((unsigned)small), dim3(64 * kDfWaves), 0, st, a);
        else
            hipLaunchKernelGGL(dct_fused_mfma_kernel<64>, dim3((unsigned)patches), dim3(64 * kDfWaves), 0, st, a);
        return launch_status();
    }
    hipLaunchKernelGGL(dct_transform_valu_kernel, dim3(blocks), dim3(64 * kDctWaves), 0, st, a);
    const int64_t bblocks = (int64_t)C * ((H + 15) / 16) * ((W + 63) / 64);
    if (bblocks > 0x7fffffff) return HB_ERR_UNSUPPORTED;
    hipLaunchKernelGGL(dct_blend_kernel, dim3((unsigned)bblocks), dim3(256), 0, st, a);
    return launch_status();
}

}  // namespace hb

extern "C" size_t hb_dct_denoise_workspace_size(int C, int H, int W) {
    if (C < 1 || H < 16 || W < 16 || (H & 7) || (W & 7)) return 0;
    return (size_t)C * (size_t)(H / 8 - 1) * (size_t)(W / 8 - 1) * 256 * sizeof(float);
}

extern "C" hb_status hb_dct_denoise(const hb_half* in, float* out, int C, int H, int W,
                                    int64_t in_pitch, int64_t in_plane, int64_t out_pitch, int64_t out_plane,
                                    float threshold, void* workspace, size_t workspace_bytes, hb_stream stream) {
    return hb::dct_run(false, in, out, C, H, W, in_pitch, in_plane, out_pitch, out_plane, threshold, workspace,
                       workspace_bytes, stream);
}

extern "C" hb_status hb_dct_denoise_valu(const hb_half* in, float* out, int C, int H, int W,
                                         int64_t in_pitch, int64_t in_plane, int64_t out_pitch, int64_t out_plane,
                                         float threshold, void* workspace, size_t workspace_bytes, hb_stream stream) {
    return hb::dct_run(true, in, out, C, H, W, in_pitch, in_plane, out_pitch, out_plane, threshold, workspace,
                       workspace_bytes, stream);
}
