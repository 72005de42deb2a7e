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
// (c, g) holds rows 4g + j of column c): instruction j of the
// next product (K = 4) takes register j as it is, as A or as B operand, if slot g of the other stands for row 4g + j:
//     Q[r][v] = sum_x P[r][x] E[v][x]     Y[u][v] = sum_r E[u][r] Q[r][v]        (E[u][i] = D[u][i] w[i])
//     R[v][r] = sum_u Y[u][v] E[u][r]     rec[x][r] = sum_v E[v][x] R[v][r]
// No transpose and no LDS between the four, and rec ends with four consecutive pixels of a row per lane.
// The products along the rows are the outer ones, so tiles one above the other share them: Q belongs to a row of pixels and
// columns of a tile, whichever tile asks, and the R of the two tiles over a row are added before the last product.
// The windows are part of E.
#include <math.h>

#include "hb_device.hpp"
#include "hb_host.hpp"

namespace hb {

constexpr int kDctWaves = 4;                  // waves per workgroup
constexpr int kDctPitch = 17;                 // floats per row of an LDS tile (conflict-free both ways)

struct DctArgs {
    const half_t* in;
    float* out;
    float* tiles;                             // workspace: [C][nty][ntx][16][16] windowed reconstructions (the twin's)
    int C, H, W, nty, ntx;
    int64_t in_pitch, in_plane, out_pitch, out_plane;
    float threshold;
};
struct DctTables {
    float d[256];                             // D[u][i], orthonormal DCT-II, row-major
    float w[16];                              // sine window
};
struct DctTwinArgs : DctArgs, DctTables {};

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
// The matrix-unit path in ONE launch: transform, core, transform back AND blend.  A workgroup owns a 64 x 64 patch of the
// output and runs every tile that overlaps it (up to 9 x 9; those on the rim are run by the neighbouring patch as well).  A
// wave walks down a column of tiles; the ninth column, of which the patch has the left half, is dealt out tile by tile, so
// that a workgroup is eight waves, two to a SIMD (with a wave for the ninth column a compute unit held two workgroups
// instead of four, 3 x 1024 x 1024 22.6 us).  The columns meet in LDS: every second one is laid down, the others added.
//
// What bounds it: the fp32 products, 32 cycles each and SIMD.  Per tile Y and R take eight, Q and rec, shared by the tiles
// above each other, half of the two and four they were before (Q: the pixels are fp16, so it is two K = 32 products with E as three
// fp16 parts, together the fp32 number); the waves' 27400 cycles for a patch, six to a SIMD, are 8.6 us of 3 x 1024 x 1024, the
// pixels on their way in 3 us and the way out 3.  Against products of a tile alone, a chain of loads ahead of them and
// cached stores: 3 x 1024 x 1024 22.6 -> 17.7 us, 2048 x 2048 28.8 -> 22.4, 3 x 1080 x 1920 40.3 -> 32.0, 1024 x 1024 10.6 -> 8.6.
// Error against fp64: adding R before the last product costs 1 to 2 %, two short sums instead of one for Y gain 2 to 4: 1080 x
// 1920, thresholds 0 / 0.05 / 0.35 / 0.5 1.218 / 1.191 / 1.055 / 1.063e-7 -> 1.195 / 1.174 / 1.035 / 1.019e-7.
template <int PATCH>
struct DfGeom {
    static constexpr int kWaves = PATCH / 8;              // columns of tiles with a wave of their own
    static constexpr int kBlocks = PATCH / 16;            // of 16 rows
    static constexpr int kPitch = PATCH + 4;              // 16 rows of a tile: 16-byte pieces in different banks
    static constexpr int kRegion = PATCH + 16;            // pixels under the tiles of a patch, per axis
    static constexpr int kPxPitch = kRegion + 8;
    static constexpr int kChunks = kRegion / 8;           // of eight pixels per row of the region
    static constexpr int kPieces = (kRegion * kChunks + 64 * kWaves - 1) / (64 * kWaves);    // of them per thread
};
// E[u][i] = D[u][i] w[i] (D the orthonormal DCT-II), its transpose and the sine window w[i]
static __device__ const float kDctE[256] = {
    0.0245042853f, 0.0725711659f, 0.117849186f, 0.158598319f, 0.193252608f, 0.220480323f, 0.239235088f, 0.24879618f, 0.24879618f, 0.239235088f, 0.220480323f, 0.193252608f, 0.158598319f, 0.117849186f, 0.0725711659f, 0.0245042853f,
    0.0344874226f, 0.0982118696f, 0.146984443f, 0.173379987f, 0.173379987f, 0.146984443f, 0.0982118696f, 0.0344874226f, -0.0344874226f, -0.0982118696f, -0.146984443f, -0.173379987f, -0.173379987f, -0.146984443f, -0.0982118696f, -0.0344874226f,
    0.0339884199f, 0.0853346661f, 0.0925935134f, 0.0437571779f, -0.053318277f, -0.173230276f, -0.281310707f, -0.34509021f, -0.34509021f, -0.281310707f, -0.173230276f, -0.053318277f, 0.0437571779f, 0.0925935134f, 0.0853346661f, 0.0339884199f,
    0.0331620909f, 0.0651085004f, 0.0163359195f, -0.105730467f, -0.241029486f, -0.310304821f, -0.261532247f, -0.102136932f, 0.102136932f, 0.261532247f, 0.310304821f, 0.241029486f, 0.105730467f, -0.0163359195f, -0.0651085004f, -0.0331620909f,
    0.0320163928f, 0.0392752327f, -0.063779518f, -0.207218692f, -0.252496719f, -0.11932309f, 0.12947309f, 0.325067878f, 0.325067878f, 0.12947309f, -0.11932309f, -0.252496719f, -0.207218692f, -0.063779518f, 0.0392752327f, 0.0320163928f,
    0.030562358f, 0.01005961f, -0.128832951f, -0.214633957f, -0.079334937f, 0.197807789f, 0.33670035f, 0.165861383f, -0.165861383f, -0.33670035f, -0.197807789f, 0.079334937f, 0.214633957f, 0.128832951f, -0.01005961f, -0.030562358f,
    0.0288139917f, -0.0200223401f, -0.163461521f, -0.124609903f, 0.151837602f, 0.305814981f, 0.0660048127f, -0.292553365f, -0.292553365f, 0.0660048127f, 0.305814981f, 0.151837602f, -0.124609903f, -0.163461521f, -0.0200223401f, 0.0288139917f,
    0.0267881304f, -0.04837998f, -0.159487426f, 0.0219844505f, 0.271984458f, 0.0905125812f, -0.298379987f, -0.22321187f, 0.22321187f, 0.298379987f, -0.0905125812f, -0.271984458f, -0.0219844505f, 0.159487426f, 0.04837998f, -0.0267881304f,
    0.0245042853f, -0.0725711659f, -0.117849186f, 0.158598319f, 0.193252608f, -0.220480323f, -0.239235088f, 0.24879618f, 0.24879618f, -0.239235088f, -0.220480323f, 0.193252608f, 0.158598319f, -0.117849186f, -0.0725711659f, 0.0245042853f,
    0.0219844505f, -0.0905125812f, -0.04837998f, 0.22321187f, -0.0267881304f, -0.298379987f, 0.159487426f, 0.271984458f, -0.271984458f, -0.159487426f, 0.298379987f, 0.0267881304f, -0.22321187f, 0.04837998f, 0.0905125812f, -0.0219844505f,
    0.0192528926f, -0.100659102f, 0.0325145163f, 0.186491892f, -0.227241039f, -0.0608303808f, 0.331828594f, -0.195477903f, -0.195477903f, 0.331828594f, -0.0608303808f, -0.227241039f, 0.186491892f, 0.0325145163f, -0.100659102f, 0.0192528926f,
    0.0163359195f, -0.102136932f, 0.105730467f, 0.0651085004f, -0.261532247f, 0.241029486f, 0.0331620909f, -0.310304821f, 0.310304821f, -0.0331620909f, -0.241029486f, 0.261532247f, -0.0651085004f, -0.105730467f, 0.102136932f, -0.0163359195f,
    0.0132616237f, -0.0948188007f, 0.153977379f, -0.0858327895f, -0.104587562f, 0.288071424f, -0.312575698f, 0.134647518f, 0.134647518f, -0.312575698f, 0.288071424f, -0.104587562f, -0.0858327895f, 0.153977379f, -0.0948188007f, 0.0132616237f,
    0.01005961f, -0.079334937f, 0.165861383f, -0.197807789f, 0.128832951f, 0.030562358f, -0.214633957f, 0.33670035f, -0.33670035f, 0.214633957f, -0.030562358f, -0.128832951f, 0.197807789f, -0.165861383f, 0.079334937f, -0.01005961f,
    0.0067607169f, -0.0570188016f, 0.138575986f, -0.219982192f, 0.268049061f, -0.259257436f, 0.187965795f, -0.0686427131f, -0.0686427131f, 0.187965795f, -0.259257436f, 0.268049061f, -0.219982192f, 0.138575986f, -0.0570188016f, 0.0067607169f,
    0.00339671457f, -0.0297922455f, 0.0785648227f, -0.142289266f, 0.211264119f, -0.274988562f, 0.323761135f, -0.350156665f, 0.350156665f, -0.323761135f, 0.274988562f, -0.211264119f, 0.142289266f, -0.0785648227f, 0.0297922455f, -0.00339671457f,
};
static __device__ const float kDctEt[256] = {
    0.0245042853f, 0.0344874226f, 0.0339884199f, 0.0331620909f, 0.0320163928f, 0.030562358f, 0.0288139917f, 0.0267881304f, 0.0245042853f, 0.0219844505f, 0.0192528926f, 0.0163359195f, 0.0132616237f, 0.01005961f, 0.0067607169f, 0.00339671457f,
    0.0725711659f, 0.0982118696f, 0.0853346661f, 0.0651085004f, 0.0392752327f, 0.01005961f, -0.0200223401f, -0.04837998f, -0.0725711659f, -0.0905125812f, -0.100659102f, -0.102136932f, -0.0948188007f, -0.079334937f, -0.0570188016f, -0.0297922455f,
    0.117849186f, 0.146984443f, 0.0925935134f, 0.0163359195f, -0.063779518f, -0.128832951f, -0.163461521f, -0.159487426f, -0.117849186f, -0.04837998f, 0.0325145163f, 0.105730467f, 0.153977379f, 0.165861383f, 0.138575986f, 0.0785648227f,
    0.158598319f, 0.173379987f, 0.0437571779f, -0.105730467f, -0.207218692f, -0.214633957f, -0.124609903f, 0.0219844505f, 0.158598319f, 0.22321187f, 0.186491892f, 0.0651085004f, -0.0858327895f, -0.197807789f, -0.219982192f, -0.142289266f,
    0.193252608f, 0.173379987f, -0.053318277f, -0.241029486f, -0.252496719f, -0.079334937f, 0.151837602f, 0.271984458f, 0.193252608f, -0.0267881304f, -0.227241039f, -0.261532247f, -0.104587562f, 0.128832951f, 0.268049061f, 0.211264119f,
    0.220480323f, 0.146984443f, -0.173230276f, -0.310304821f, -0.11932309f, 0.197807789f, 0.305814981f, 0.0905125812f, -0.220480323f, -0.298379987f, -0.0608303808f, 0.241029486f, 0.288071424f, 0.030562358f, -0.259257436f, -0.274988562f,
    0.239235088f, 0.0982118696f, -0.281310707f, -0.261532247f, 0.12947309f, 0.33670035f, 0.0660048127f, -0.298379987f, -0.239235088f, 0.159487426f, 0.331828594f, 0.0331620909f, -0.312575698f, -0.214633957f, 0.187965795f, 0.323761135f,
    0.24879618f, 0.0344874226f, -0.34509021f, -0.102136932f, 0.325067878f, 0.165861383f, -0.292553365f, -0.22321187f, 0.24879618f, 0.271984458f, -0.195477903f, -0.310304821f, 0.134647518f, 0.33670035f, -0.0686427131f, -0.350156665f,
    0.24879618f, -0.0344874226f, -0.34509021f, 0.102136932f, 0.325067878f, -0.165861383f, -0.292553365f, 0.22321187f, 0.24879618f, -0.271984458f, -0.195477903f, 0.310304821f, 0.134647518f, -0.33670035f, -0.0686427131f, 0.350156665f,
    0.239235088f, -0.0982118696f, -0.281310707f, 0.261532247f, 0.12947309f, -0.33670035f, 0.0660048127f, 0.298379987f, -0.239235088f, -0.159487426f, 0.331828594f, -0.0331620909f, -0.312575698f, 0.214633957f, 0.187965795f, -0.323761135f,
    0.220480323f, -0.146984443f, -0.173230276f, 0.310304821f, -0.11932309f, -0.197807789f, 0.305814981f, -0.0905125812f, -0.220480323f, 0.298379987f, -0.0608303808f, -0.241029486f, 0.288071424f, -0.030562358f, -0.259257436f, 0.274988562f,
    0.193252608f, -0.173379987f, -0.053318277f, 0.241029486f, -0.252496719f, 0.079334937f, 0.151837602f, -0.271984458f, 0.193252608f, 0.0267881304f, -0.227241039f, 0.261532247f, -0.104587562f, -0.128832951f, 0.268049061f, -0.211264119f,
    0.158598319f, -0.173379987f, 0.0437571779f, 0.105730467f, -0.207218692f, 0.214633957f, -0.124609903f, -0.0219844505f, 0.158598319f, -0.22321187f, 0.186491892f, -0.0651085004f, -0.0858327895f, 0.197807789f, -0.219982192f, 0.142289266f,
    0.117849186f, -0.146984443f, 0.0925935134f, -0.0163359195f, -0.063779518f, 0.128832951f, -0.163461521f, 0.159487426f, -0.117849186f, 0.04837998f, 0.0325145163f, -0.105730467f, 0.153977379f, -0.165861383f, 0.138575986f, -0.0785648227f,
    0.0725711659f, -0.0982118696f, 0.0853346661f, -0.0651085004f, 0.0392752327f, -0.01005961f, -0.0200223401f, 0.04837998f, -0.0725711659f, 0.0905125812f, -0.100659102f, 0.102136932f, -0.0948188007f, 0.079334937f, -0.0570188016f, 0.0297922455f,
    0.0245042853f, -0.0344874226f, 0.0339884199f, -0.0331620909f, 0.0320163928f, -0.030562358f, 0.0288139917f, -0.0267881304f, 0.0245042853f, -0.0219844505f, 0.0192528926f, -0.0163359195f, 0.0132616237f, -0.01005961f, 0.0067607169f, -0.00339671457f,
};
static __device__ const float kDctW[16] = {
    0.0980171412f, 0.290284663f, 0.471396744f, 0.634393275f, 0.773010433f, 0.881921291f, 0.956940353f, 0.99518472f, 0.99518472f, 0.956940353f, 0.881921291f, 0.773010433f, 0.634393275f, 0.471396744f, 0.290284663f, 0.0980171412f,
};
constexpr float kDfScale = 1024.f;                        // of the first product's E: keeps its low part a normal fp16 number

template <int PATCH>
__global__ void __launch_bounds__(64 * DfGeom<PATCH>::kWaves, 8) dct_fused_mfma_kernel(DctArgs p) {
    using G = DfGeom<PATCH>;
    __shared__ __attribute__((aligned(16))) float s_acc[PATCH * G::kPitch];
    __shared__ __attribute__((aligned(16))) half_t s_px[G::kRegion * G::kPxPitch];
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
    // (what lies outside the image is under no tile, and no sum takes it in: some pixel of the image stands there).
    // Everything the workgroup needs is requested here, at once.
    half8 px[G::kPieces];
#pragma unroll
    for (int k = 0; k < G::kPieces; ++k) {
        const int i = min((int)threadIdx.x + 64 * G::kWaves * k, G::kRegion * G::kChunks - 1), r = i / G::kChunks;
        const int y = clampi(py0 - 8 + r, 0, p.H - 1), x = clampi(px0 - 8 + 8 * (i - r * G::kChunks), 0, p.W - 8);
        px[k] = *reinterpret_cast<const half8_u*>(p.in + (int64_t)plane * p.in_plane + (int64_t)y * p.in_pitch + x);
    }
    floatx4 ef[2], eb[2];                     // E[c][4g + j], E[4g + j][c]; [1]: rows 8 further
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        ef[h] = *reinterpret_cast<const floatx4*>(kDctE + c * 16 + ((4 * g + 8 * h) & 15));
        eb[h] = *reinterpret_cast<const floatx4*>(kDctEt + ((c + 8 * h) & 15) * 16 + 4 * g);
    }
#pragma unroll
    for (int k = 0; k < G::kPieces; ++k) {
        const int i = min((int)threadIdx.x + 64 * G::kWaves * k, G::kRegion * G::kChunks - 1), r = i / G::kChunks;
        *reinterpret_cast<half8*>(&s_px[r * G::kPxPitch + 8 * (i - r * G::kChunks)]) = px[k];
    }
    half8 e1, e0 = {0, 0, 0, 0, 0, 0, 0, 0};  // scaled E[c][4g + j] as hi (slots 0..3) and lo (4..7), which share a pixel; the rest
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const float v = kDfScale * ef[0][j];
        e1[j] = (half_t)v;
        e1[4 + j] = (half_t)(v - (float)e1[j]);
        e0[j] = (half_t)(v - (float)e1[j] - (float)e1[4 + j]);
    }
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        ef[h] *= 1.f / kDfScale;              // the first product's scale undone
        asm volatile("" : "+v"(ef[h]), "+v"(eb[h]));      // loaded here, not where they are used
    }
    const float cut0 = c == 0 && g == 0 ? -1.f : p.threshold;   // the DC bin always stays
    const int ty0 = py0 / 8, tx0 = px0 / 8 - 1;           // tile (ty, tx): origin (8 ty, 8 tx)
    const floatx4 zero = {0.f, 0.f, 0.f, 0.f};
    __syncthreads();
    // Q of rows py0 + row0 .. + 15 of column `col` of tiles: lane (c = v, g) holds rows 4g + j (rows beyond the region: another one's)
    auto along_rows = [&](int row0, int col) {
        const int row = clampi(row0 + c + 8, 0, G::kRegion - 1);
        const half4 px = *reinterpret_cast<const half4*>(&s_px[row * G::kPxPitch + 8 * col + 4 * g]);
        return mfma16x16x32(join(px, px), e1, mfma16x16x32(join(px, px), e0, zero));
    };
    // a tile from Q of its rows (in slots 8 rows further if h = 1) to R: lane (c = row, 8 further if h = 1; g) holds v = 4g + j
    auto tile = [&](const floatx4& q, int h) {
        floatx4 y = mfma16x16x4f32(ef[h][1], q[1], mfma16x16x4f32(ef[h][0], q[0], zero));      // two short sums: see the error above
        y += mfma16x16x4f32(ef[h][3], q[3], mfma16x16x4f32(ef[h][2], q[2], zero));
        // coring: lane (c = v, g) holds bins (u = 4g + j, v)
#pragma unroll
        for (int j = 0; j < 4; ++j)
            if (fabsf(y[j]) < (j == 0 ? cut0 : p.threshold)) y[j] = 0.f;
        floatx4 r = zero;
#pragma unroll
        for (int j = 3; j >= 0; --j) r = mfma16x16x4f32(y[j], eb[h][j], r);         // the large low bins last
        return r;
    };
    // back along the rows: lane (c = row, g) holds pixels 4g .. 4g + 3
    auto back = [&](const floatx4& r) {
        floatx4 rec = zero;
#pragma unroll
        for (int j = 3; j >= 0; --j) rec = mfma16x16x4f32(eb[0][j], r[j], rec);
        return rec;
    };
    auto pick = [](bool second, const floatx4& a, const floatx4& b) {
        return floatx4{second ? b[0] : a[0], second ? b[1] : a[1], second ? b[2] : a[2], second ? b[3] : a[3]};
    };
    // The wave's column, tiles ty0 - 1 .. ty0 + PATCH / 8 - 1
    const bool live = tx0 + wv >= 0 && tx0 + wv < p.ntx;  // uniform
    floatx4 rec[G::kBlocks];
#pragma unroll
    for (int b = 0; b < G::kBlocks; ++b) rec[b] = zero;
    if (live) {
        floatx4 q = along_rows(0, wv), before = zero;
        if (ty0 >= 1) before = tile(pick(g >= 2, q, along_rows(-16, wv)), 1);
#pragma unroll
        for (int b = 0; b < G::kBlocks; ++b) {
            floatx4 r = zero, after = zero;
            if (ty0 + 2 * b < p.nty) r = tile(q, 0);
            const floatx4 next = along_rows(16 * b + 16, wv);
            if (ty0 + 2 * b + 1 < p.nty) after = tile(pick(g >= 2, next, q), 1);
            r += pick(c >= 8, before, after);
            rec[b] = back(r);
            before = after;
            q = next;
        }
    }
    // The last column, of which the patch has the left half: a tile a wave, the even ones (from ty0 on) and then the odd ones.
    const bool live_last = tx0 + G::kWaves < p.ntx;
    const int k = wv < G::kBlocks ? 2 * wv : 2 * (wv - G::kBlocks) + 1;
    floatx4 last = zero;
    if (live_last && ty0 + k < p.nty) last = back(tile(along_rows(8 * k, G::kWaves), 0));
    floatx4 first = zero;                                 // the last wave also has the tile above
    if (wv == G::kWaves - 1 && live_last && ty0 >= 1) first = back(tile(along_rows(-8, G::kWaves), 0));
    // Blend.  Every second column covers the patch once, and so do the even tiles of the last one: they are laid down, then
    // the other columns added, then the last one's odd tiles.
    float* const acc = &s_acc[c * G::kPitch + 4 * g];
    float* const acc_last = acc + 8 * k * G::kPitch + PATCH - 8;
    auto add = [](float* at, const floatx4& v) { *reinterpret_cast<floatx4*>(at) = *reinterpret_cast<const floatx4*>(at) + v; };
    if (!(wv & 1) && 8 * wv - 8 + 4 * g >= 0) {
#pragma unroll
        for (int b = 0; b < G::kBlocks; ++b) *reinterpret_cast<floatx4*>(acc + 16 * b * G::kPitch + 8 * wv - 8) = rec[b];
    }
    if (wv < G::kBlocks && g < 2) *reinterpret_cast<floatx4*>(acc_last) = last;
    __syncthreads();
    if ((wv & 1) && live) {
#pragma unroll
        for (int b = 0; b < G::kBlocks; ++b) add(acc + 16 * b * G::kPitch + 8 * wv - 8, rec[b]);
    }
    __syncthreads();
    if (wv >= G::kBlocks && live_last && g < 2) {
        if (8 * k + c < PATCH && ty0 + k < p.nty) add(acc_last, last);
        if (wv == G::kWaves - 1 && ty0 >= 1 && c >= 8) add(acc - 8 * G::kPitch + PATCH - 8, first);
    }
    __syncthreads();
    // out = sum of the windowed reconstructions / sum of the squared windows of the tiles covering the pixel
    // (the tiles covering a pixel are a product set, so the denominator is a product of two 1-D sums)
    auto covered = [&](int z, int n) {                    // z / 8 - 1 and z / 8: the tiles over pixel z of an axis of n tiles
        const int t = z >> 3, i = z & 7;
        const float a = kDctW[i + 8] * kDctW[i + 8], b = kDctW[i] * kDctW[i];
        return (t >= 1 ? a : 0.f) + (t < n ? b : 0.f);
    };
    for (int idx = threadIdx.x; idx < PATCH * (PATCH / 4); idx += 64 * G::kWaves) {
        const int r = idx / (PATCH / 4), q4 = idx - r * (PATCH / 4);
        const int y = py0 + r, x = px0 + 4 * q4;
        if (y >= p.H || x >= p.W) continue;
        const float dy = covered(y, p.nty);
        const floatx4 v = *reinterpret_cast<const floatx4*>(&s_acc[r * G::kPitch + 4 * q4]);
        floatx4 o;
#pragma unroll
        for (int q = 0; q < 4; ++q) o[q] = v[q] / (dy * covered(x + q, p.ntx));
        // streamed whatever the rows' alignment: a patch's rows are 256 bytes long, and nothing reads them here (3 x 2000 x 2040 with rows of 2040 / 2041 / 2043
        // 64.1 / 62.2 / 62.3 us, cached 67.9 / 66.5 / 65.9; 1 x 2048 x 2048 in rows of 2049 23.0, 24.7; 1000 x 1000 8.9 either way)
        __builtin_nontemporal_store(o, reinterpret_cast<floatx4_u*>(p.out + (int64_t)plane * p.out_plane + (int64_t)y * p.out_pitch + x));
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

__global__ void __launch_bounds__(64 * kDctWaves) dct_transform_valu_kernel(DctTwinArgs p) {
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
__global__ void __launch_bounds__(256) dct_blend_kernel(DctTwinArgs p) {
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

    hipStream_t st = reinterpret_cast<hipStream_t>(stream);
    const int64_t ntiles = (int64_t)C * a.nty * a.ntx;
    const int64_t wgs = (ntiles + kDctWaves - 1) / kDctWaves;
    const unsigned blocks = (unsigned)(wgs < 4096 ? wgs : 4096);     // waves stride over the tiles
    if (!valu) {
        // one launch: tiles and blend fused, the workspace stays unused
        // 32 x 32 patches (1.4x the products) where one takes no more than a third of the rounds that the larger ones take, up to two
        // of these: a round of 64 x 64 patches on all compute units is 4.5 us, one of the small ones 1.5 (512 x 512 6.4 us, 8.3 with
        // the larger ones; 3 x 512 x 512, three small rounds, 7.9 and 8.5; 880 x 880, four, 9.2 and 8.5; 3 x 640 x 640, five, 10.8 and
        // 12.9 in two large rounds; 1536 x 1536, nine against three, 18.1 and 17.6).
        const int64_t patches = (int64_t)C * ceil_div(H, 64) * ceil_div(W, 64);
        const int64_t small = (int64_t)C * ceil_div(H, 32) * ceil_div(W, 32);
        if (patches > 0x7fffffff) return HB_ERR_UNSUPPORTED;
        const int64_t rounds = (patches + num_cu() - 1) / num_cu(), small_rounds = (small + num_cu() - 1) / num_cu();
        if (rounds <= 2 && small_rounds <= 3 * rounds)
            hipLaunchKernelGGL(dct_fused_mfma_kernel<32>, dim3((unsigned)small), dim3(64 * DfGeom<32>::kWaves), 0, st, a);
        else
            hipLaunchKernelGGL(dct_fused_mfma_kernel<64>, dim3((unsigned)patches), dim3(64 * DfGeom<64>::kWaves), 0, st, a);
        return launch_status();
    }
    static const DctTables tables = dct_tables();         // computed once: 3 us of the host's 11 per call
    DctTwinArgs b;
    static_cast<DctArgs&>(b) = a;
    static_cast<DctTables&>(b) = tables;
    hipLaunchKernelGGL(dct_transform_valu_kernel, dim3(blocks), dim3(64 * kDctWaves), 0, st, b);
    const int64_t bblocks = (int64_t)C * ((H + 15) / 16) * ((W + 63) / 64);
    if (bblocks > 0x7fffffff) return HB_ERR_UNSUPPORTED;
    hipLaunchKernelGGL(dct_blend_kernel, dim3((unsigned)bblocks), dim3(256), 0, st, b);
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
