// hb_down2 / hb_up2: resampling by a factor of two with an arbitrary 2-D kernel, and their
// vector-ALU twins (Sec. V-B).
//
// Downsampling is a strided convolution, O(x, y) = sum I(2x + rx, 2y + ry) K(rx, ry).  Along x it
// is a product with the strided Toeplitz matrix A^down_K(x, y) = K(y - 2x): a tile of 16 outputs
// reads a window of 30 + kw pixels.
//
// Upsampling is the multiphase filter O(2x + dx, 2y + dy) = sum I(x + rx, y + ry) K(2rx + dx, 2ry + dy).
// Along x the two column phases interleave inside one coefficient matrix (row 2i + dx of the
// matrix holds K(2(k - i) + dx, .)), so a tile of 16 outputs comes from a window of 8 + kw/2 - 1
// input pixels and is stored as it is.
//
// Both run as a serial loop over the kernel rows; see toeplitz2d.hpp.
#include "hb_device.hpp"
#include "hb_host.hpp"
#include "toeplitz2d.hpp"

namespace hb {

// ---------------------------------------------------------------------------
// Vector-ALU kernels.  The input pixels an output tile needs are staged in LDS as fp32 with both
// indices clamped (the definition's border rule verbatim).  A thread owns 8 consecutive outputs of
// one row: for every kernel row it reads the pixels under them once (16-byte LDS reads) and slides
// the taps over them in registers, 8 FMAs per tap read.  KWP = kernel width rounded up to 8, 16 or
// 32; the taps beyond kw are zeros, and so are the staged columns only they can reach.
constexpr int kRsTaps = HB_MAX_TAPS_CONV2D;
constexpr int kRsDownRows = 2 * 15 + kRsTaps;                          // 62
constexpr int kRsDownPitch = 2 * 64 + kRsTaps;                         // 160 floats
constexpr int kRsUpRows = 8 + kRsTaps / 2 - 1;                         // 23
constexpr int kRsUpPitch = 64 + kRsTaps / 2;                           // 80 floats

template <int KWP>
__device__ __forceinline__ void rs2_stage_taps(const T2Args& p, float* s_k, int nthreads) {
    for (int i = threadIdx.x; i < p.kh * KWP; i += nthreads) {
        const int ry = i / KWP, t = i - ry * KWP;
        s_k[i] = t < p.kw ? (float)__builtin_bit_cast(half_t, p.taps[ry * p.kw + t]) : 0.f;
    }
}

// 16 x 64 outputs per workgroup of 128 threads
template <int KWP>
__global__ void __launch_bounds__(128) down2_valu_kernel(T2Args p) {
    __shared__ __attribute__((aligned(16))) float s_px[kRsDownRows * kRsDownPitch];
    __shared__ float s_k[kRsTaps * KWP];
    rs2_stage_taps<KWP>(p, s_k, 128);
    const int nt = (p.Wo + 63) / 64;
    const int rg = blockIdx.x / nt, tc = blockIdx.x - rg * nt;
    const int x0 = 64 * tc, y0 = 16 * rg;
    const int nrows = 30 + p.kh;
    for (int idx = threadIdx.x; idx < nrows * kRsDownPitch; idx += 128) {
        const int r = idx / kRsDownPitch, cc = idx - r * kRsDownPitch;
        float v = 0.f;
        if (cc < 126 + p.kw) {
            const int y = clampi(2 * y0 + r - p.ay, 0, p.H - 1), x = clampi(2 * x0 + cc - p.ax, 0, p.W - 1);
            v = (float)p.in[(int64_t)y * p.in_pitch + x];
        }
        s_px[idx] = v;
    }
    __syncthreads();
    const int r = threadIdx.x >> 3, xl = 8 * (threadIdx.x & 7);
    const int y = y0 + r;
    if (y >= p.Ho || x0 + xl >= p.Wo) return;
    float acc[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) acc[q] = 0.f;
    for (int ry = 0; ry < p.kh; ++ry) {
        float w[KWP + 16];                                 // inputs 2 xl .. 2 xl + KWP + 15 of row 2 r + ry
        const floatx4* src = reinterpret_cast<const floatx4*>(&s_px[(2 * r + ry) * kRsDownPitch + 2 * xl]);
#pragma unroll
        for (int i = 0; i < (KWP + 16) / 4; ++i) {
            const floatx4 v = src[i];
            w[4 * i] = v[0];
            w[4 * i + 1] = v[1];
            w[4 * i + 2] = v[2];
            w[4 * i + 3] = v[3];
        }
        const float* k = &s_k[ry * KWP];
#pragma unroll
        for (int t = 0; t < KWP; ++t) {
            const float kv = k[t];
#pragma unroll
            for (int q = 0; q < 8; ++q) acc[q] = fmaf(kv, w[2 * q + t], acc[q]);
        }
    }
    float* row = p.out + (int64_t)y * p.out_pitch;
    store4_mask(row, x0 + xl, p.Wo, floatx4{acc[0], acc[1], acc[2], acc[3]});
    store4_mask(row, x0 + xl + 4, p.Wo, floatx4{acc[4], acc[5], acc[6], acc[7]});
}

// 16 x 128 outputs per workgroup of 256 threads = 8 x 64 input positions plus halo
template <int KWP>
__global__ void __launch_bounds__(256) up2_valu_kernel(T2Args p) {
    constexpr int RXP = KWP / 2;
    __shared__ __attribute__((aligned(16))) float s_px[kRsUpRows * kRsUpPitch];
    __shared__ float s_k[kRsTaps * KWP];
    rs2_stage_taps<KWP>(p, s_k, 256);
    const int nt = (p.Wo + 127) / 128;
    const int rg = blockIdx.x / nt, tc = blockIdx.x - rg * nt;
    const int x0 = 128 * tc, y0 = 16 * rg;    // output tile; input tile starts at (y0 / 2, x0 / 2)
    const int nrows = 8 + p.kh / 2 - 1;
    for (int idx = threadIdx.x; idx < nrows * kRsUpPitch; idx += 256) {
        const int r = idx / kRsUpPitch, cc = idx - r * kRsUpPitch;
        float v = 0.f;
        if (cc < 64 + p.kw / 2 - 1) {
            const int y = clampi(y0 / 2 + r - p.ay, 0, p.H - 1), x = clampi(x0 / 2 + cc - p.ax, 0, p.W - 1);
            v = (float)p.in[(int64_t)y * p.in_pitch + x];
        }
        s_px[idx] = v;
    }
    __syncthreads();
    const int r = threadIdx.x >> 4, xl = 8 * (threadIdx.x & 15);
    const int y = y0 + r;
    if (y >= p.Ho || x0 + xl >= p.Wo) return;
    const int dy = y & 1;
    float acc[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) acc[q] = 0.f;
    for (int ry = 0; ry < p.kh / 2; ++ry) {
        float w[RXP + 4];                                  // inputs xl / 2 .. xl / 2 + RXP + 3 of row r / 2 + ry
        const floatx4* src = reinterpret_cast<const floatx4*>(&s_px[(r / 2 + ry) * kRsUpPitch + xl / 2]);
#pragma unroll
        for (int i = 0; i < (RXP + 4) / 4; ++i) {
            const floatx4 v = src[i];
            w[4 * i] = v[0];
            w[4 * i + 1] = v[1];
            w[4 * i + 2] = v[2];
            w[4 * i + 3] = v[3];
        }
        const float* k = &s_k[(2 * ry + dy) * KWP];
#pragma unroll
        for (int rx = 0; rx < RXP; ++rx) {
            const float k0 = k[2 * rx], k1 = k[2 * rx + 1];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                acc[2 * i] = fmaf(k0, w[i + rx], acc[2 * i]);
                acc[2 * i + 1] = fmaf(k1, w[i + rx], acc[2 * i + 1]);
            }
        }
    }
    float* row = p.out + (int64_t)y * p.out_pitch;
    store4_mask(row, x0 + xl, p.Wo, floatx4{acc[0], acc[1], acc[2], acc[3]});
    store4_mask(row, x0 + xl + 4, p.Wo, floatx4{acc[4], acc[5], acc[6], acc[7]});
}

// ---------------------------------------------------------------------------
static hb_status rs2_prepare(T2Args& a, bool up, const hb_half* in, float* out, int H, int W,
                             int64_t in_pitch, int64_t out_pitch,
                             const hb_half* taps_host, int kh, int kw, int ay, int ax) {
    if (H <= 0 || W <= 0 || H > (1 << 29) || W > (1 << 29)) return HB_ERR_INVALID_ARG;
    const int Ho = up ? 2 * H : (H + 1) / 2, Wo = up ? 2 * W : (W + 1) / 2;
    // check_image wants one shape for both sides: validate each side against its own width
    hb_status s = check_image(in, out, H, W, in_pitch, in_pitch);
    if (s != HB_OK) return s;
    s = check_image(in, out, Ho, Wo, Wo, out_pitch);
    if (s != HB_OK) return s;
    // lanes address rows with 32-bit byte offsets from the image base
    if ((int64_t)H * in_pitch >= ((int64_t)1 << 31) || (int64_t)Ho * out_pitch >= ((int64_t)1 << 30)) return HB_ERR_UNSUPPORTED;
    if (!taps_host) return HB_ERR_INVALID_ARG;
    if (kh < 1 || kh > HB_MAX_TAPS_CONV2D || kw < 1 || kw > HB_MAX_TAPS_CONV2D) return HB_ERR_INVALID_ARG;
    if (up) {
        if ((kh & 1) || (kw & 1)) return HB_ERR_INVALID_ARG;
        if (ay < 0 || ay >= kh / 2 || ax < 0 || ax >= kw / 2) return HB_ERR_INVALID_ARG;
    } else {
        if (ay < 0 || ay >= kh || ax < 0 || ax >= kw) return HB_ERR_INVALID_ARG;
    }
    a.in = reinterpret_cast<const half_t*>(in);
    a.out = out;
    a.H = H;
    a.W = W;
    a.Ho = Ho;
    a.Wo = Wo;
    a.in_pitch = in_pitch;
    a.out_pitch = out_pitch;
    a.kh = kh;
    a.kw = kw;
    a.ay = ay;
    a.ax = ax;
    memset(a.taps, 0, sizeof(a.taps));
    memcpy(a.taps, taps_host, sizeof(uint16_t) * (size_t)kh * (size_t)kw);
    a.ncol = a.nrow = a.ntiles = a.stream = a.alias = a.steps = a.srows = a.rows = 0;
    return HB_OK;
}

template <int MODE, int NK, int NW>
static hb_status rs2_launch(T2Args& a, hipStream_t st) {
    const T2Shape shape = t2_resample_tile((T2Mode)MODE, NK, a.kh, a.Ho, a.Wo, num_cu());
    if constexpr (MODE == kT2Down) {
        if (shape == kT2Stack) return t2_launch<MODE, NK, NW, kT2Stack>(a, st);
        if (shape == kT2FlatPair) return t2_launch<MODE, NK, NW, kT2FlatPair>(a, st);
    }
    if (shape == kT2Block) return t2_launch<MODE, NK, NW, kT2Block>(a, st);
    if (shape == kT2Flat) return t2_launch<MODE, NK, NW, kT2Flat>(a, st);
    return t2_launch<MODE, NK, NW, kT2Row>(a, st);
}

template <class K>
static hb_status rs2_launch_valu(K kernel, const T2Args& a, int tile_w, int threads, hipStream_t st) {
    const int64_t blocks = (int64_t)ceil_div(a.Ho, 16) * ceil_div(a.Wo, tile_w);
    if (blocks > 0x7fffffff) return HB_ERR_UNSUPPORTED;
    hipLaunchKernelGGL(kernel, dim3((unsigned)blocks), dim3(threads), 0, st, a);
    return launch_status();
}

}  // namespace hb

extern "C" hb_status hb_down2(const hb_half* in, float* out, int H, int W, int64_t in_pitch, int64_t out_pitch,
                              const hb_half* taps_host, int kh, int kw, int anchor_y, int anchor_x, hb_stream stream) {
    using namespace hb;
    T2Args a;
    hb_status s = rs2_prepare(a, false, in, out, H, W, in_pitch, out_pitch, taps_host, kh, kw, anchor_y, anchor_x);
    if (s != HB_OK) return s;
    if (W < kT2MinWidth)
        return hb_down2_valu(in, out, H, W, in_pitch, out_pitch, taps_host, kh, kw, anchor_y, anchor_x, stream);
    hipStream_t st = reinterpret_cast<hipStream_t>(stream);
    switch (ceil_div(30 + kw, 16)) {
        case 2: return rs2_launch<kT2Down, 2, 1>(a, st);
        case 3: return rs2_launch<kT2Down, 3, 1>(a, st);
        default: return rs2_launch<kT2Down, 4, 1>(a, st);
    }
}

extern "C" hb_status hb_down2_valu(const hb_half* in, float* out, int H, int W, int64_t in_pitch, int64_t out_pitch,
                                   const hb_half* taps_host, int kh, int kw, int anchor_y, int anchor_x, hb_stream stream) {
    using namespace hb;
    T2Args a;
    hb_status s = rs2_prepare(a, false, in, out, H, W, in_pitch, out_pitch, taps_host, kh, kw, anchor_y, anchor_x);
    if (s != HB_OK) return s;
    hipStream_t st = reinterpret_cast<hipStream_t>(stream);
    if (kw <= 8) return rs2_launch_valu(down2_valu_kernel<8>, a, 64, 128, st);
    if (kw <= 16) return rs2_launch_valu(down2_valu_kernel<16>, a, 64, 128, st);
    return rs2_launch_valu(down2_valu_kernel<32>, a, 64, 128, st);
}

extern "C" hb_status hb_up2(const hb_half* in, float* out, int H, int W, int64_t in_pitch, int64_t out_pitch,
                            const hb_half* taps_host, int kh, int kw, int anchor_y, int anchor_x, hb_stream stream) {
    using namespace hb;
    T2Args a;
    hb_status s = rs2_prepare(a, true, in, out, H, W, in_pitch, out_pitch, taps_host, kh, kw, anchor_y, anchor_x);
    if (s != HB_OK) return s;
    if (W < kT2MinWidth)
        return hb_up2_valu(in, out, H, W, in_pitch, out_pitch, taps_host, kh, kw, anchor_y, anchor_x, stream);
    hipStream_t st = reinterpret_cast<hipStream_t>(stream);
    if (7 + kw / 2 <= 16) return rs2_launch<kT2Up, 1, 2>(a, st);
    return rs2_launch<kT2Up, 2, 2>(a, st);
}

extern "C" hb_status hb_up2_valu(const hb_half* in, float* out, int H, int W, int64_t in_pitch, int64_t out_pitch,
                                 const hb_half* taps_host, int kh, int kw, int anchor_y, int anchor_x, hb_stream stream) {
    using namespace hb;
    T2Args a;
    hb_status s = rs2_prepare(a, true, in, out, H, W, in_pitch, out_pitch, taps_host, kh, kw, anchor_y, anchor_x);
    if (s != HB_OK) return s;
    hipStream_t st = reinterpret_cast<hipStream_t>(stream);
    if (kw <= 8) return rs2_launch_valu(up2_valu_kernel<8>, a, 128, 256, st);
    if (kw <= 16) return rs2_launch_valu(up2_valu_kernel<16>, a, 128, 256, st);
    return rs2_launch_valu(up2_valu_kernel<32>, a, 128, 256, st);
}
