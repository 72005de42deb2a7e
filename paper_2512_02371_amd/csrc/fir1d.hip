// hb_fir1d: row-wise FIR as a product with a Toeplitz matrix held in registers
// (Sec. V-A: O(x..x+k-1) = I(x..x+k+l-1) * A_K, A_K(x, y) = K(y - x)), and its
// vector-ALU twin.
//
// MFMA formulation.  The paper lifts the vector-matrix product to a matrix-matrix
// product by stacking overlapped segments of ONE row (Eq. 1).  An image already
// has the second dimension: 16 image rows are the 16 independent vectors, so the
// image operand is read straight from memory in its natural layout (each lane: 8
// consecutive pixels of one row, one 16-byte load at any pixel offset) and no
// overlapped view has to be staged.  For a 16-column output tile starting at x0 the
// window is the 32*NK pixels from x0 - anchor - e on (e = anchor & 1 keeps the window
// on an even pixel, i.e. dword aligned: 16-byte loads at odd pixel offsets run at a
// fraction of the rate), and we compute the transposed tile
//     D'[m][n] = sum_k A[m][k] * P[k][n],   m = output column in the tile,
//                                            n = image row in a 16-row group,
//                                            k = pixel in the window,
// with A[m][k] = taps[k - m - e] (zero outside the taps): A_K itself, built once per
// wave from a zero-padded tap table.  In D' a lane owns four consecutive output
// columns of one row, so the result leaves with one 16-byte store per lane.
#include <utility>

#include "fir1d_plan.hpp"
#include "hb_device.hpp"
#include "hb_host.hpp"

namespace hb {

// f(integral_constant<int, 0>) ... f(integral_constant<int, N-1>): a loop that is unrolled by construction,
// so that register arrays indexed by the step stay in registers.
template <class F, int... I>
__device__ __forceinline__ void unrolled_steps_impl(F& f, std::integer_sequence<int, I...>) {
    (f(std::integral_constant<int, I>{}), ...);
}
template <int N, class F>
__device__ __forceinline__ void unrolled_steps(F& f) {
    unrolled_steps_impl(f, std::make_integer_sequence<int, N>{});
}

struct FirArgs {
    const half_t* in;
    float* out;
    int H, W;
    int64_t in_pitch, out_pitch;
    int T, anchor;
    int nct;             // strips per row group
    int ntasks;          // strips x row groups
    int lines;           // every row of the output starts a 128-byte line
    int ntiles, run_tiles, nruns, wtasks;   // the walk of long filters: tiles per row, per run, runs per row group, tasks
    TapsT<HB_MAX_TAPS_FIR1D> taps;
    int step;            // rows of a group are this far apart: see FirRows
};

// Eight pixels from column xs on of the row at byte offset rowoff, requested from an address inside the row
// (W >= 8); fir_clamped() shifts what reaches over the row's ends into place, which is the column clamp.
__device__ __forceinline__ half8 fir_request(const FirArgs& p, uint32_t rowoff, int xs) {
    return ldg8(p.in, rowoff + 2u * (uint32_t)clampi(xs, 0, p.W - 8));
}
__device__ __forceinline__ half8 fir_clamped(const FirArgs& p, half8 v, int xs) {
    return shift_in_from_left(shift_in_from_right(v, max(xs - (p.W - 8), 0)), max(-xs, 0));
}

// A group of 16 rows.  Where rows start on odd pixels (LEAN), a window that starts on an even one is no run of whole dwords, and
// every lane's 16 bytes are several cache accesses.  There the windows of a group start on the pixel that makes their address
// even, one further left or not, with the coefficients moved by as much; of an odd pitch that is another one in every second row, and a
// group has every second row (p.step = 2): the even ones of 32, then the odd ones.  4095 x 4095, 8 / 40 / 256 taps 33.7 / 25.9 / 31.0 -> 23.3 /
// 24.0 / 28.1 us, 2047 x 2047 10.8 / 11.2 / 17.0 -> 8.0 / 8.9 / 14.7, 300 x 8191, 8 taps 8.7 -> 5.9, 17 x 3001, 100 taps 6.9 -> 6.2.
struct FirRows {
    int y0, e;                                // first row; pixels that its windows start left of the anchor's
};
template <bool LEAN>
__device__ __forceinline__ FirRows fir_rows(const FirArgs& p, int rg) {
    if constexpr (!LEAN) return {16 * rg, p.anchor & 1};
    const int y0 = p.step == 2 ? 32 * (rg >> 1) + (rg & 1) : 16 * rg;
    return {y0, (int)((reinterpret_cast<uintptr_t>(p.in) >> 1) + (uintptr_t)y0 * (uintptr_t)p.in_pitch + (uintptr_t)p.anchor) & 1};
}

// One window per tile (up to 17 taps): nothing to share between tiles or steps.  A wave takes HB_FIR_TILES tiles of one
// 16-row group, all requested up front, and leaves.  A strip at the image's border shifts its pixels into place in
// registers (with the clamp folded into per-tile coefficients from tables in the kernel arguments the 256 x 256 launch
// took 5.0 us, now 3.8; 4096 x 4096 20.7 -> 19.0, a copy 18.3).
template <bool LEAN>
__global__ void __launch_bounds__(256) fir1d_mfma_kernel(FirArgs p) {
    constexpr int NW = HB_FIR_TILES;
    __shared__ __attribute__((aligned(16))) float s_patch[4][RowPatch<NW>::kFloats];
    const int lane = threadIdx.x & 63;
    const int c = lane & 15, g = lane >> 4;
    int e = p.anchor & 1, aw = p.anchor + e;              // window start, left of the tile
    // (tasks in plain launch order: with one contiguous eighth of the tasks per XCD this kernel measured
    // 10 % slower on tall images, 100 against 89 us on 262144 x 256; groups of 2 to 8 neighbours per XCD
    // measured within 2 % of the plain order there)
    const int task = __builtin_amdgcn_readfirstlane(blockIdx.x * 4 + (threadIdx.x >> 6));
    if (task >= p.ntasks) return;
    const int rg = task / p.nct, ct = task - rg * p.nct;
    const FirRows rows = fir_rows<LEAN>(p, rg);
    const int apart = LEAN ? p.step : 1;
    if constexpr (LEAN) {
        e = rows.e;
        aw = p.anchor + e;
    }
    const int x0 = 16 * NW * ct, y0 = rows.y0;
    const bool inside = x0 >= aw && x0 + 16 * (NW - 1) - aw + 32 <= p.W && x0 + 16 * NW <= p.W;   // uniform
    const uint32_t rowoff = (uint32_t)min(y0 + apart * c, p.H - 1) * (uint32_t)p.in_pitch * 2u;
    half8 px[NW];
#pragma unroll
    for (int w = 0; w < NW; ++w) px[w] = fir_request(p, rowoff, x0 - aw + 16 * w + 8 * g);
    // The Toeplitz fragment, A-operand layout: lane (c, g) holds A[c][8g + i] = taps[8g + i - c - e], read from the tap
    // table in the kernel arguments only now: a wave that waited for the table first would put a memory round
    // trip in front of its pixel requests.
    __builtin_amdgcn_sched_barrier(0);
    const half8 coef = tap_run(p.taps.tab, 8 * g - c - e);
    if (!inside) {
#pragma unroll
        for (int w = 0; w < NW; ++w) px[w] = fir_clamped(p, px[w], x0 - aw + 16 * w + 8 * g);
    }
    floatx4 acc[NW];
#pragma unroll
    for (int w = 0; w < NW; ++w) {
        const floatx4 zero = {0.f, 0.f, 0.f, 0.f};
        acc[w] = mfma16x16x32(coef, px[w], zero);
    }
    float* const dst = p.out + (int64_t)y0 * p.out_pitch + x0;
    float* const patch = s_patch[threadIdx.x >> 6];
    const int64_t pitch = apart * p.out_pitch;
    if (inside && y0 + 15 * apart + 1 <= p.H) store_rows_via_lds<NW, true>(patch, dst, (uint32_t)pitch, acc, lane);
    else store_rows_via_lds_masked<NW, true>(patch, dst, pitch, acc, lane, (p.H - y0 + apart - 1) / apart, p.W - x0);
}

// ---------------------------------------------------------------------------
// Long filters (two or more windows per tile): the walk along the row.
//
// In the kernel above every product loads its own window, NK loads of 16 rows x 64 bytes per
// 16 x 16 outputs, and with long filters those loads are all the kernel does (256 taps: 9 KB requested
// per 1 KB of outputs; the matrix units idle).  Here a wave walks along a run of tiles of one
// 16-row group and loads every pixel of it once, in windows of 32 side by side.  Tiles go in PAIRS: window v (the 32 pixels from
// 32 v - aw on) is the kk-th window of the even tile of pair v - kk for every kk < NK, and of the odd one, 16 pixels further, for
// every kk < NKO, with Toeplitz fragments that are shifted by 16; NKO is NK or NK + 1.  So a window feeds up to 2 NKO products, each
// into the accumulator of its own tile.  NKO pairs are open at any time (a ring
// of accumulators, indexed at compile time: the walk is unrolled over one turn of the ring); a pair is
// complete NKO - 1 steps after its first window and leaves through the LDS
// patch as 128-byte runs.  Windows that reach over the row ends are shifted into place when they are used:
// the Toeplitz matrix is indexed by window position, so the border rule needs nothing else.
// A run of n pairs walks n + NKO - 1 windows, the last NKO - 1 of them the next run's too (what they and the first windows
// add to pairs outside the run is dropped): the price of cutting a row into several tasks.
// What it gains: with windows of 32 pixels at a stride of 16, one step a
// tile, every pixel was requested twice: 4096 x 4096, 40 / 64 / 256 taps 18.6 / 18.8 / 25.2
// -> 17.3 / 17.6 / 22.3 us, 8192 x 8192, 30 taps 124 -> 101, 4095 x 4095, 100 taps 37.8 -> 25.9.  What bounds it is not the bytes in flight
// alone (NKO KB a wave; with twice as many windows ahead 256 taps took 24.6 us): from four windows on half the waves, each
// walking fewer windows for its neighbour (with 256 taps one in five, one in three with two waves per SIMD), are mostly the faster.
template <int NK, int NKO, bool LEAN>
__global__ void __launch_bounds__(64 * fir_walk_waves(NK)) fir1d_walk_kernel(FirArgs p) {
    constexpr int WV = fir_walk_waves(NK);
    __shared__ __attribute__((aligned(16))) float s_patch[WV][RowPatch<4>::kFloats];
    const int lane = threadIdx.x & 63;
    const int c = lane & 15, g = lane >> 4;
    half8 even[NK], odd[NKO];
    // written out twice: in a function of e they cost the plain kernel address arithmetic and a later first load, 0.2 us of a small call (654 x 42,
    // 20 taps 5.0, 5.2)
    int e = p.anchor & 1;
    if constexpr (!LEAN) {
#pragma unroll
        for (int kk = 0; kk < NK; ++kk) even[kk] = tap_run(p.taps.tab, 32 * kk + 8 * g - c - e);
#pragma unroll
        for (int kk = 0; kk < NKO; ++kk) odd[kk] = tap_run(p.taps.tab, 32 * kk - 16 + 8 * g - c - e);
    }

    const int wgpos = xcd_contiguous(blockIdx.x, gridDim.x);
    const int task = __builtin_amdgcn_readfirstlane(wgpos * WV + (threadIdx.x >> 6));
    if (task >= p.wtasks) return;
    const int rg = task / p.nruns, run = task - rg * p.nruns;
    const FirRows rows = fir_rows<LEAN>(p, rg);
    const int y0 = rows.y0, apart = LEAN ? p.step : 1;
    if constexpr (LEAN) e = rows.e;
    const int aw = p.anchor + e;
    if constexpr (LEAN) {
#pragma unroll
        for (int kk = 0; kk < NK; ++kk) even[kk] = tap_run(p.taps.tab, 32 * kk + 8 * g - c - e);
#pragma unroll
        for (int kk = 0; kk < NKO; ++kk) odd[kk] = tap_run(p.taps.tab, 32 * kk - 16 + 8 * g - c - e);
    }
    const int t0 = run * p.run_tiles;                     // first tile of the run
    const int L = min(p.run_tiles, p.ntiles - t0);        // its tiles
    const int npairs = (L + 1) / 2, nsteps = npairs + NKO - 1;        // pairs of tiles, windows
    const uint32_t rowoff = (uint32_t)min(y0 + apart * c, p.H - 1) * (uint32_t)p.in_pitch * 2u;
    float* patch = s_patch[threadIdx.x >> 6];
    const bool rows16 = y0 + 15 * apart + 1 <= p.H;

    auto load_window = [&](int v) { return fir_request(p, rowoff, 16 * t0 + 32 * v - aw + 8 * g); };
    auto window_inside = [&](int v) {                     // uniform
        const int xs = 16 * t0 + 32 * v - aw;
        return xs >= 0 && xs + 32 <= p.W;
    };
    // Rows that start inside a 128-byte line: columns 32 k + o .. 32 k + o + 31 of the run are a line of the row, o its
    // first column's distance to the next line.  The patch keeps the last two pairs, and with pair k the line that ends in
    // it leaves, whole: pairs stored as they are would write two parts of a line (100 taps, 4095 x 4095 63 us
    // so, 38 by lines; 4096 x 4100 46, 23.6).
    const int limit = min(16 * L, p.W - 16 * t0);         // columns of the run
    int o[2];
#pragma unroll
    for (int s = 0; s < 2; ++s) {
        const int64_t at = (int64_t)(reinterpret_cast<uintptr_t>(p.out) / 4) + (int64_t)(y0 + apart * (8 * s + (lane >> 3))) * p.out_pitch + 16 * t0;
        o[s] = (int)(-at & 31);
    }
    auto store_line = [&](int k) {                        // the one that ends in pair k
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            const int row = 8 * s + (lane >> 3), col = 32 * (k - 1) + o[s] + 4 * (lane & 7);
            floatx4 v;
#pragma unroll
            for (int i = 0; i < 4; ++i) v[i] = patch[row * RowPatch<4>::kPitch + ((col + i) & 63)];
            if (y0 + apart * row >= p.H) continue;
            float* const q = p.out + (int64_t)(y0 + apart * row) * p.out_pitch + 16 * t0 + col;
            if (col >= 0 && col + 4 <= limit) {
                __builtin_nontemporal_store(v, reinterpret_cast<floatx4_u*>(q));
            } else {
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    if (col + i >= 0 && col + i < limit) q[i] = v[i];
            }
        }
        wave_lds_fence();
    };
    // pair j of the run, completed in the step before
    auto store_pair = [&](int j, const floatx4 (&done)[2]) {
        if (j < 0 || j >= npairs) return;
        const int tb = 2 * j, x = 16 * (t0 + tb);
        if (!p.lines) {                                   // uniform
#pragma unroll
            for (int w = 0; w < 2; ++w)
                *reinterpret_cast<floatx4*>(patch + c * RowPatch<4>::kPitch + ((16 * (tb + w)) & 63) + 4 * g) = done[w];
            wave_lds_fence();
            store_line(j);
        } else if (rows16 && x + 32 <= p.W) {
            store_rows_via_lds<2, true>(patch, p.out + (int64_t)y0 * p.out_pitch + x, (uint32_t)(apart * p.out_pitch), done, lane);
        } else if (y0 + apart * c < p.H) {
            float* row = p.out + (int64_t)(y0 + apart * c) * p.out_pitch;
            store4_mask(row, x + 4 * g, p.W, done[0]);
            if (tb + 1 < L) store4_mask(row, x + 16 + 4 * g, p.W, done[1]);
        }
    };

    floatx4 acc[NKO][2];
    // as many windows in flight as a tile needs: the longer the filter, the more products a window feeds and the further
    // ahead the loads have to run to cover their latency
    half8 win[NKO];
#pragma unroll
    for (int i = 0; i < NKO; ++i) win[i] = load_window(i);              // nsteps >= NKO
    int ub = 0;
    // one step: window v = ub + S against every fragment, pair v - kk in slot (v - kk) % NKO; the pair before it in slot S is complete
    auto step = [&](auto sc) {
        constexpr int S = decltype(sc)::value;
        const int v = ub + S;
        store_pair(v - NKO, acc[S]);                      // before the loads: loads and stores share one counter
        if (v < nsteps) {
            if (!window_inside(v)) win[S] = fir_clamped(p, win[S], 16 * t0 + 32 * v - aw + 8 * g);
            auto product = [&](auto kc) {
                constexpr int KK = decltype(kc)::value, slot = (S - KK + NKO) % NKO;
                const floatx4 zero = {0.f, 0.f, 0.f, 0.f};
                if constexpr (KK < NK) acc[slot][0] = mfma16x16x32(even[KK], win[S], KK == 0 ? zero : acc[slot][0]);
                acc[slot][1] = mfma16x16x32(odd[KK], win[S], KK == 0 ? zero : acc[slot][1]);
            };
            unrolled_steps<NKO>(product);
            if (v + NKO < nsteps) win[S] = load_window(v + NKO);
        }
    };
#pragma unroll
    for (int i = 0; i < NKO; ++i) acc[i][0] = acc[i][1] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
    for (ub = 0; ub < nsteps; ub += NKO) unrolled_steps<NKO>(step);
    store_pair(ub - NKO, acc[0]);
    if (!p.lines) store_line((L + 1) / 2);                // what is left of the last line
}

// Vector-ALU twin: a 16 x 128 tile is staged in LDS as fp32 with its halo, the column index clamped
// (the definition's border rule verbatim).  A thread owns 8 consecutive outputs of one row and slides
// the taps over them eight at a time: 8 taps and 8 new pixels are read (16-byte LDS reads), 64 FMAs use
// them.  Taps are padded with zeros to a multiple of 8.
constexpr int kValuTileW = 128;
constexpr int kValuPitch = kValuTileW + HB_MAX_TAPS_FIR1D + 8;   // floats per staged row

__global__ void __launch_bounds__(256) fir1d_valu_kernel(FirArgs p) {
    __shared__ __attribute__((aligned(16))) float s_px[16 * kValuPitch];
    __shared__ __attribute__((aligned(16))) float s_k[HB_MAX_TAPS_FIR1D];
    static_assert(HB_MAX_TAPS_FIR1D <= 256, "one tap per thread");
    const int tp = (p.T + 7) & ~7;
    if ((int)threadIdx.x < tp) s_k[threadIdx.x] = (int)threadIdx.x < p.T ? (float)tap_at(p.taps.tab, threadIdx.x) : 0.f;

    const int nctv = (p.W + kValuTileW - 1) / kValuTileW;
    const int rg = blockIdx.x / nctv, ct = blockIdx.x - rg * nctv;
    const int x0 = ct * kValuTileW;
    // staged column j holds pixel clampW(x0 - anchor + j); j < 128 + tp covers every window
    const int nch = (kValuTileW + tp) / 8;
    for (int idx = threadIdx.x; idx < 16 * nch; idx += 256) {
        const int r = idx / nch, ch = idx - r * nch;
        const half_t* row = p.in + (int64_t)min(16 * rg + r, p.H - 1) * p.in_pitch;
        const half8 v = load8_clamp(row, x0 - p.anchor + 8 * ch, p.W);
        floatx4* dst = reinterpret_cast<floatx4*>(&s_px[r * kValuPitch + 8 * ch]);
        dst[0] = floatx4{(float)v[0], (float)v[1], (float)v[2], (float)v[3]};
        dst[1] = floatx4{(float)v[4], (float)v[5], (float)v[6], (float)v[7]};
    }
    __syncthreads();

    const int r = threadIdx.x >> 4, xl = 8 * (threadIdx.x & 15);
    const int y = 16 * rg + r;
    if (y >= p.H || x0 + xl >= p.W) return;
    const floatx4* src = reinterpret_cast<const floatx4*>(&s_px[r * kValuPitch + xl]);
    float acc[8], w[16];
#pragma unroll
    for (int q = 0; q < 8; ++q) acc[q] = 0.f;
    {
        const floatx4 a = src[0], b = src[1];
#pragma unroll
        for (int i = 0; i < 4; ++i) w[i] = a[i], w[4 + i] = b[i];
    }
    for (int tb = 0; tb < tp; tb += 8) {
        const floatx4 a = src[tb / 4 + 2], b = src[tb / 4 + 3];      // pixels xl + tb + 8 .. + 15
        const floatx4 ka = *reinterpret_cast<const floatx4*>(&s_k[tb]), kb = *reinterpret_cast<const floatx4*>(&s_k[tb + 4]);
#pragma unroll
        for (int i = 0; i < 4; ++i) w[8 + i] = a[i], w[12 + i] = b[i];
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const float kv = i < 4 ? ka[i] : kb[i - 4];
#pragma unroll
            for (int q = 0; q < 8; ++q) acc[q] = fmaf(kv, w[q + i], acc[q]);
        }
#pragma unroll
        for (int i = 0; i < 8; ++i) w[i] = w[8 + i];
    }
    float* orow = p.out + (int64_t)y * p.out_pitch;
    store4_mask(orow, x0 + xl, p.W, floatx4{acc[0], acc[1], acc[2], acc[3]});
    store4_mask(orow, x0 + xl + 4, p.W, floatx4{acc[4], acc[5], acc[6], acc[7]});
}

static hb_status fir1d_prepare(FirArgs& a, FirPlan& plan, const hb_half* in, float* out, int H, int W,
                               int64_t in_pitch, int64_t out_pitch,
                               const hb_half* taps_host, int ntaps, int anchor) {
    hb_status s = check_image(in, out, H, W, in_pitch, out_pitch);
    if (s != HB_OK) return s;
    // lanes address rows with 32-bit byte offsets from the image base
    if ((int64_t)H * in_pitch >= ((int64_t)1 << 31) || (int64_t)H * out_pitch >= ((int64_t)1 << 30)) return HB_ERR_UNSUPPORTED;
    s = check_taps(taps_host, ntaps, anchor, HB_MAX_TAPS_FIR1D);
    if (s != HB_OK) return s;
    a.in = reinterpret_cast<const half_t*>(in);
    a.out = out;
    a.H = H;
    a.W = W;
    a.in_pitch = in_pitch;
    a.out_pitch = out_pitch;
    a.lines = out_pitch % 32 == 0 && aligned_to(out, 128);
    a.T = ntaps;
    a.anchor = anchor;
    plan = fir_plan({H, W, in_pitch, out_pitch, in_pitch % 2 == 0 && aligned_to(in, 4), a.lines != 0, ntaps, anchor, num_cu()});
    a.step = plan.step;
    a.nct = ceil_div(W, 16 * HB_FIR_TILES);
    if ((int64_t)plan.rowsteps * a.nct > 0x7fffffff / 2) return HB_ERR_UNSUPPORTED;
    a.ntasks = plan.rowsteps * a.nct;
    a.ntiles = plan.ntiles;
    a.run_tiles = plan.run_tiles;
    a.nruns = plan.nruns;
    const int64_t wtasks = (int64_t)plan.rowsteps * a.nruns;
    if (wtasks > 0x7fffffff / 4) return HB_ERR_UNSUPPORTED;
    a.wtasks = (int)wtasks;
    a.taps = pack_taps<HB_MAX_TAPS_FIR1D>(taps_host, ntaps);
    return HB_OK;
}

template <bool LEAN>
static hb_status fir1d_launch(const FirArgs& a, const FirPlan& plan, hipStream_t st) {
#define HB_FIR_WALK_AS(N, NO)                                                                     \
    hipLaunchKernelGGL((fir1d_walk_kernel<N, NO, LEAN>), dim3(ceil_div(a.wtasks, fir_walk_waves(N))), dim3(64 * fir_walk_waves(N)), 0, st, a)
#define HB_FIR_WALK(N)                                                                            \
    case N:                                                                                       \
        if (plan.nko > N) HB_FIR_WALK_AS(N, N + 1);                                                  \
        else HB_FIR_WALK_AS(N, N);                                                                \
        break;
    switch (plan.nk) {
        // one window per tile: nothing to share between tiles, every wave takes one strip of tiles
        case 1: hipLaunchKernelGGL(fir1d_mfma_kernel<LEAN>, dim3(ceil_div(a.ntasks, 4)), dim3(256), 0, st, a); break;
        // long filters: the walk along the row, every window loaded once
        HB_FIR_WALK(2) HB_FIR_WALK(3) HB_FIR_WALK(4) HB_FIR_WALK(5) HB_FIR_WALK(6) HB_FIR_WALK(7) HB_FIR_WALK(8)
        case 9: HB_FIR_WALK_AS(9, 9); break;
        default: break;
    }
#undef HB_FIR_WALK
#undef HB_FIR_WALK_AS
    return launch_status();
}

}  // namespace hb

extern "C" hb_status hb_fir1d_valu(const hb_half* in, float* out, int H, int W,
                                   int64_t in_pitch, int64_t out_pitch,
                                   const hb_half* taps_host, int ntaps, int anchor, hb_stream stream);

extern "C" hb_status hb_fir1d(const hb_half* in, float* out, int H, int W,
                              int64_t in_pitch, int64_t out_pitch,
                              const hb_half* taps_host, int ntaps, int anchor, hb_stream stream) {
    using namespace hb;
    FirArgs a;
    FirPlan plan;
    hb_status s = fir1d_prepare(a, plan, in, out, H, W, in_pitch, out_pitch, taps_host, ntaps, anchor);
    if (s != HB_OK) return s;
    // a 16-column tile reads the 16 + ntaps - 1 pixels from x0 - anchor on (one more when the
    // window is moved to an even pixel): NK windows of 32
    const int nk = plan.nk;
    // narrow images are one short run per row group, whose windows all reach over the row's ends: with rows inside lines
    // the vector ALU is the faster one (1000 x 100, 100 / 159 taps 5.4 / 6.7 us, walked 7.4 / 8.3, but 200 taps 8.3 and 7.8; 8192 x 65, 200 taps 8.7
    // and 9.3), with whole lines (1000 x 128, 100 / 200 taps 5.4 / 8.3, 4.9 / 5.3) and in tall images (20000 x 100, 159 taps 15, 11;
    // 50000 x 83 31, 21) it is not, nor below 33 columns (3600 x 16, 100 taps 10.5, 5.6)
    if (W < kFirMinWidth || (nk >= 4 && W > 32 && W <= 128 && !a.lines && H <= 32 * num_cu()))
        return hb_fir1d_valu(in, out, H, W, in_pitch, out_pitch, taps_host, ntaps, anchor, stream);
    hipStream_t st = reinterpret_cast<hipStream_t>(stream);
    return plan.lean ? fir1d_launch<true>(a, plan, st) : fir1d_launch<false>(a, plan, st);
}

extern "C" hb_status hb_fir1d_valu(const hb_half* in, float* out, int H, int W,
                                   int64_t in_pitch, int64_t out_pitch,
                                   const hb_half* taps_host, int ntaps, int anchor, hb_stream stream) {
    using namespace hb;
    FirArgs a;
    FirPlan plan;
    hb_status s = fir1d_prepare(a, plan, in, out, H, W, in_pitch, out_pitch, taps_host, ntaps, anchor);
    if (s != HB_OK) return s;
    const int64_t blocks = (int64_t)ceil_div(H, 16) * ceil_div(W, kValuTileW);
    if (blocks > 0x7fffffff) return HB_ERR_UNSUPPORTED;
    hipLaunchKernelGGL(fir1d_valu_kernel, dim3((unsigned)blocks), dim3(256), 0,
                       reinterpret_cast<hipStream_t>(stream), a);
    return launch_status();
}
