// hb_conv2d: single-channel 2-D convolution with an arbitrary (non-separable) kernel, and its
// vector-ALU twin (Sec. V-A, 2-D form: O(x, y) = sum_{rx, ry} I(x + rx, y + ry) K(rx, ry)).
//
// MFMA formulation: the serial loop over the kernel rows r_y of Sec. V-A, one Toeplitz product per row into the
// same accumulator; see toeplitz2d.hpp.
#include "hb_device.hpp"
#include "hb_host.hpp"
#include "toeplitz2d.hpp"

namespace hb {

// ---------------------------------------------------------------------------
// Vector-ALU kernel: a 16 x 128 output tile per workgroup.  The tile and its halo are staged in LDS
// as fp32 with both indices clamped (the definition's border rule verbatim).  A thread owns 8
// consecutive outputs of one row: for every kernel row it reads the 8 + KWP - 1 pixels under them
// once (16-byte LDS reads) and slides the taps over them in registers, 8 FMAs per tap read.
// KWP = kernel width rounded up to 8, 16 or 32; the taps beyond kw are zeros.
constexpr int kC2vW = 128;
constexpr int kC2vRows = 16 + HB_MAX_TAPS_CONV2D - 1;                 // 47
constexpr int kC2vPitch = kC2vW + HB_MAX_TAPS_CONV2D;                  // 160 floats

template <int KWP>
__global__ void __launch_bounds__(256) conv2d_valu_kernel(T2Args p) {
    __shared__ __attribute__((aligned(16))) float s_px[kC2vRows * kC2vPitch];
    __shared__ float s_k[HB_MAX_TAPS_CONV2D * KWP];
    for (int i = threadIdx.x; i < p.kh * KWP; i += 256) {
        const int ry = i / KWP, t = i - ry * KWP;
        s_k[i] = t < p.kw ? (float)__builtin_bit_cast(half_t, p.taps[ry * p.kw + t]) : 0.f;
    }
    const int nt = (p.W + kC2vW - 1) / kC2vW;
    const int rg = blockIdx.x / nt, tc = blockIdx.x - rg * nt;
    const int x0 = kC2vW * tc, y0 = 16 * rg;
    const int nrows = 16 + p.kh - 1;
    for (int idx = threadIdx.x; idx < nrows * kC2vPitch; idx += 256) {
        const int r = idx / kC2vPitch, cc = idx - r * kC2vPitch;
        float v = 0.f;                                    // columns only zero taps can reach stay zero
        if (cc < kC2vW + p.kw - 1) {
            const int y = clampi(y0 + r - p.ay, 0, p.H - 1), x = clampi(x0 + cc - p.ax, 0, p.W - 1);
            v = (float)p.in[(int64_t)y * p.in_pitch + x];
        }
        s_px[idx] = v;
    }
    __syncthreads();

    const int r = threadIdx.x >> 4, xl = 8 * (threadIdx.x & 15);
    const int y = y0 + r;
    if (y >= p.H || x0 + xl >= p.W) return;
    float acc[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) acc[q] = 0.f;
    for (int ry = 0; ry < p.kh; ++ry) {
        float w[KWP + 8];
        const floatx4* src = reinterpret_cast<const floatx4*>(&s_px[(r + ry) * kC2vPitch + xl]);
#pragma unroll
        for (int i = 0; i < (KWP + 8) / 4; ++i) {
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
            for (int q = 0; q < 8; ++q) acc[q] = fmaf(kv, w[t + q], acc[q]);
        }
    }
    float* row = p.out + (int64_t)y * p.out_pitch;
    store4_mask(row, x0 + xl, p.W, floatx4{acc[0], acc[1], acc[2], acc[3]});
    store4_mask(row, x0 + xl + 4, p.W, floatx4{acc[4], acc[5], acc[6], acc[7]});
}

static hb_status conv2d_prepare(T2Args& a, const hb_half* in, float* out, int H, int W,
                                int64_t in_pitch, int64_t out_pitch,
                                const hb_half* taps_host, int kh, int kw, int ay, int ax) {
    hb_status s = check_image(in, out, H, W, in_pitch, out_pitch);
    if (s != HB_OK) return s;
    // lanes address rows with 32-bit byte offsets from the image base
    if ((int64_t)H * in_pitch >= ((int64_t)1 << 31) || (int64_t)H * out_pitch >= ((int64_t)1 << 30)) return HB_ERR_UNSUPPORTED;
    if (!taps_host) return HB_ERR_INVALID_ARG;
    if (kh < 1 || kh > HB_MAX_TAPS_CONV2D || kw < 1 || kw > HB_MAX_TAPS_CONV2D) return HB_ERR_INVALID_ARG;
    if (ay < 0 || ay >= kh || ax < 0 || ax >= kw) return HB_ERR_INVALID_ARG;
    a.in = reinterpret_cast<const half_t*>(in);
    a.out = out;
    a.H = H;
    a.W = W;
    a.in_pitch = in_pitch;
    a.out_pitch = out_pitch;
    a.kh = kh;
    a.kw = kw;
    a.ay = ay;
    a.ax = ax;
    memset(a.taps, 0, sizeof(a.taps));
    memcpy(a.taps, taps_host, sizeof(uint16_t) * (size_t)kh * (size_t)kw);
    a.Ho = H;
    a.Wo = W;
    a.ncol = a.nrow = a.ntiles = a.stream = a.alias = a.steps = a.srows = a.rows = 0;
    return HB_OK;
}

static hb_status conv2d_launch_valu(const T2Args& a, hipStream_t st) {
    const int64_t blocks = (int64_t)ceil_div(a.H, 16) * ceil_div(a.W, kC2vW);
    if (blocks > 0x7fffffff) return HB_ERR_UNSUPPORTED;
    if (a.kw <= 8) hipLaunchKernelGGL(conv2d_valu_kernel<8>, dim3((unsigned)blocks), dim3(256), 0, st, a);
    else if (a.kw <= 16) hipLaunchKernelGGL(conv2d_valu_kernel<16>, dim3((unsigned)blocks), dim3(256), 0, st, a);
    else hipLaunchKernelGGL(conv2d_valu_kernel<32>, dim3((unsigned)blocks), dim3(256), 0, st, a);
    return launch_status();
}

template <int NK>
static hb_status conv2d_launch(T2Args& a, hipStream_t st) {
    const T2Tile t = t2_conv_tile(a.H, a.W, a.kh, NK, a.out_pitch % 16 != 0 || !aligned_to(a.out, 64), num_cu());
    if (t.shape == kT2Block) return t.nw == 2 ? t2_launch<kT2Conv, NK, 2, kT2Block>(a, st) : t2_launch<kT2Conv, NK, 1, kT2Block>(a, st);
    if (t.shape == kT2Flat) return t2_launch<kT2Conv, NK, 2, kT2Flat>(a, st);
    switch (t.nw) {
        case 4: return t2_launch<kT2Conv, NK, 4, kT2Row>(a, st);
        case 2: return t2_launch<kT2Conv, NK, 2, kT2Row>(a, st);
        default: return t2_launch<kT2Conv, NK, 1, kT2Row>(a, st);
    }
}

}  // namespace hb

extern "C" hb_status hb_conv2d(const hb_half* in, float* out, int H, int W,
                               int64_t in_pitch, int64_t out_pitch,
                               const hb_half* taps_host, int kh, int kw, int anchor_y, int anchor_x,
                               hb_stream stream) {
    using namespace hb;
    T2Args a;
    hb_status s = conv2d_prepare(a, in, out, H, W, in_pitch, out_pitch, taps_host, kh, kw, anchor_y, anchor_x);
    if (s != HB_OK) return s;
    hipStream_t st = reinterpret_cast<hipStream_t>(stream);
    if (W < kT2MinWidth) return conv2d_launch_valu(a, st);
    switch (ceil_div(15 + kw, 16)) {
        case 1: return conv2d_launch<1>(a, st);
        case 2: return conv2d_launch<2>(a, st);
        default: return conv2d_launch<3>(a, st);
    }
}

extern "C" hb_status hb_conv2d_valu(const hb_half* in, float* out, int H, int W,
                                    int64_t in_pitch, int64_t out_pitch,
                                    const hb_half* taps_host, int kh, int kw, int anchor_y, int anchor_x,
                                    hb_stream stream) {
    using namespace hb;
    T2Args a;
    hb_status s = conv2d_prepare(a, in, out, H, W, in_pitch, out_pitch, taps_host, kh, kw, anchor_y, anchor_x);
    if (s != HB_OK) return s;
    return conv2d_launch_valu(a, reinterpret_cast<hipStream_t>(stream));
}
