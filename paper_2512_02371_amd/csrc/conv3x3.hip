// hb_conv3x3: 64 -> 64 channel 3x3 convolution (stride 1, zero padding 1, NHWC) as an implicit
// GEMM on the matrix units (Sec. V-A 2-D form summed over channels; the conv layer of Sec. IV
// without bias and activation), and its vector-ALU twin.
//
// MFMA formulation, transposed so that a lane ends with consecutive output channels of one pixel:
//   O'[m][n] = sum_k Wt[m][k] * X[k][n]     m = output channel, n = pixel, k = (tap, input channel)
// with v_mfma_f32_16x16x32_f16: 16 channels x 16 pixels per product, K = 32 input channels.
//   A wave walks DOWN a strip of 32 pixels on its own, one to a SIMD: it holds the 9 x 64 x 64 weights in 288 registers (256 of
//     them accumulation registers, from which the products read them), the twelve pixel fragments of ONE image row in
//     48 and the sums of two output rows in 64.  Row r belongs to output row r - 1 with kernel row 2, to r with 1 and to
//     r + 1 with 0: 48 products each, after which a finished row is rounded to fp16 (RNE) and leaves.  So a pixel is
//     read from LDS once per horizontal tap, and no wave ever waits for another one.
//   Image rows (34 pixels x 64 channels each, with the one-pixel halo) stream through a ring of eight rows in LDS that belongs
//     to the wave: one is in use, up to seven are on their way (three to four beside the stores of finished rows, which the counted
//     waits cannot tell from loads).  They arrive by buffer loads that write LDS directly, in the image's
//     own order (pixel-major, 128 bytes per pixel) with the eight 16-byte channel pieces of a pixel permuted
//     by an XOR with bits 1..3 of the pixel index: a row is a few contiguous 1 KB copies, and the
//     16-byte reads of 16 consecutive pixels at one channel piece still fall into 64 different
//     banks for every tap shift (the overlapped view of Eq. 1: the three horizontal taps read the
//     same LDS row at pixel offsets 0, 1, 2).  Pixels outside the image arrive as zeros (requested
//     beyond the end of the buffer descriptor), which is the zero padding.
//   Everything but the products (fragments of the next row, its requests, the way out of the last one through an LDS stage of the
//     wave, whole 128-byte pixels, 1 KB per store instruction) stands between two products, one or two instructions at a time: an instruction
//     costs a wave that is alone on its SIMD issue time, and least there.
//
// What bounds it: power, then memory.  1 x 1024 x 1024: 65 us (58.5 while the input is in the memory-side cache) against 80 (76) for
// eight waves that shared 8 x 32 tiles with v_mfma_f32_32x32x16_f16 and met twice a tile; zeros instead of pixels 44 against 55.
// A loop of nothing but products with operands like these sustains 1.85 PFLOP/s in 16 x 16 x 32 and 1.65 in 32 x 32 x 16 (clock
// 1.5 to 1.8 GHz; zeros 2.3 in both), a library product of 8192^3 1.25.  Non-temporal stores: 58.5 us, cached ones 66.4 (4 x 300 x 200 17.8, 22.7).
// The weights come straight to LDS and leave it by transposing reads: with a pass through registers and 64-bit task arithmetic the start
// of a workgroup took 2 us more (8 x 56 x 56 8.0 us, 5.7 now, 8.1 before; 3 x 100 x 100 9.5, 7.0, 8.6).
#include <algorithm>
#include <utility>

#include "hb_device.hpp"
#include "hb_host.hpp"

namespace hb {

constexpr int kCvC = 64;                 // channels in and out
constexpr int kCvTY = 8, kCvTX = 32;     // output tile (rows x pixels) per workgroup step
constexpr int kCvRows = kCvTY + 2, kCvPx = kCvTX + 2;
constexpr int kCvLdsHalves = kCvRows * 4 * kCvPx * 16;    // tile of the vector-ALU twin

struct ConvArgs {
    const half_t* in;
    const half_t* w;
    half_t* out;
    int N, H, W;
    int tiles_x, tiles_y;      // per image
    int ntiles;                // N * tiles_y * tiles_x
    int seg_len, nseg;         // MFMA kernel: rows per column segment, segments per column
    uint32_t ntasks;           // strips of 32 pixels x segments
};

// LDS layout of the vector-ALU twin: [row][16-channel chunk][8-channel half][pixel][8 channels].
__device__ __forceinline__ int cv_lds_index(int r, int kc, int half, int px) {
    return (((r * 4 + kc) * 2 + half) * kCvPx + px) * 8;
}

// A strip's rows in LDS, a ring per wave: kCvRing rows of 34 pixels x 128 bytes; channel piece cp (16 bytes) of
// pixel px sits in slot cp ^ ((px >> 1) & 7) of the pixel's eight.
constexpr int kCvWaves = 4;
constexpr int kCvRing = 8;                                // one in use, up to seven on their way
constexpr int kCvRowBytes = kCvPx * 128;                  // 4352
constexpr int kCvRowLoads = 5;                            // of 64 x 16 bytes per row, the last one of 16 lanes
constexpr int kCvRingBytes = kCvRing * kCvRowBytes;       // 34816 per wave
constexpr int kCvStream = 2;                               // stores: non-temporal
constexpr uint32_t kCvOutside = 0x80000000u;              // offset beyond any descriptor used here
// Output stage of a wave: 32 pixels x 64 channels of fp16, 144-byte pixel pitch (conflict-free both ways).
constexpr int kCvStagePitch = 144;
constexpr int kCvStageBytes = kCvTX * kCvStagePitch;      // 4608
// The weights pass through LDS on their way to the registers: taps 2w, 2w + 1 in wave w's ring behind the rows that are requested
// ahead of them, tap 8 in the stages.
constexpr int kCvTapBytes = kCvC * kCvC * 2;              // 8192
constexpr int kCvEarly = 3;                               // rows requested ahead of the weights' arrival
static_assert(kCvEarly * kCvRowBytes + 2 * kCvTapBytes <= kCvRingBytes && kCvTapBytes <= kCvWaves * kCvStageBytes, "room for the weights");

__device__ __forceinline__ uint32_t cv_lds_addr(const void* p) {
    return (uint32_t)(size_t)(__attribute__((address_space(3))) const void*)p;
}
template <int I>
struct CvInt {
    static constexpr int value = I;
};
template <class F, int... J>
__device__ __forceinline__ void cv_each(F f, std::integer_sequence<int, J...>) {
    (f(CvInt<J>{}), ...);
}
// LDS-direct loads: the active lanes copy 16 bytes each from the descriptor's base + voff (per lane) + OFFSET to LDS at M0 + OFFSET + 16 * lane.
// Written as assembly so that the compiler keeps no book on them: it would make LDS reads of other ring rows
// wait for these loads, which are meant to stay in flight for rows.  The waits that order them are explicit.
// No other instruction of this kernel uses M0.
__device__ __forceinline__ void cv_lds_base(uint32_t lds_addr) { asm volatile("s_mov_b32 m0, %0\n\ts_nop 0" ::"s"(lds_addr) : "memory"); }
template <int OFFSET>
__device__ __forceinline__ void cv_dma16(u32x4 rsrc, uint32_t voff) {
    asm volatile("buffer_load_dwordx4 %0, %1, 0 offen offset:%2 lds" ::"v"(voff), "s"(rsrc), "n"(OFFSET) : "memory");
}
template <int LANES>                                      // the first LANES < 32 lanes only (all are active outside)
__device__ __forceinline__ void cv_dma16_part(u32x4 rsrc, uint32_t voff) {
    asm volatile("s_mov_b64 exec, %2\n\tbuffer_load_dwordx4 %0, %1, 0 offen lds\n\ts_mov_b64 exec, -1" ::"v"(voff), "s"(rsrc), "n"((1 << LANES) - 1) : "memory");
}
// At most N memory instructions of this wave are outstanding afterwards, loads and stores together.  Loads are done in their order, so those
// outstanding are at most the newest N loads, in whatever order the stores are done among them.
template <int N>
__device__ __forceinline__ void cv_wait_loads() {
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}
__device__ __forceinline__ void cv_pin() { __builtin_amdgcn_sched_barrier(0); }

__global__ void __launch_bounds__(64 * kCvWaves, 1) conv3x3_mfma_kernel(ConvArgs p) {
    __shared__ __attribute__((aligned(128))) char s_ring[kCvWaves * kCvRingBytes];
    __shared__ __attribute__((aligned(128))) char s_stage[kCvWaves * kCvStageBytes];
    const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int c = lane & 15, g = lane >> 4;
    char* const ring = s_ring + wv * kCvRingBytes;
    char* const stage = s_stage + wv * kCvStageBytes;
    const uint32_t ring0 = cv_lds_addr(ring);

    // weights, as they are in memory (rows of 64 output channels per input channel) but for the 32-byte pairs of a row, which
    // change places with bits 1 and 3 of the input channel: the transposing reads below meet no bank twice
    {
        const uint64_t w = (uint64_t)p.w + 2 * kCvTapBytes * (uint32_t)wv, w8 = (uint64_t)p.w + 8 * kCvTapBytes + 2048 * wv;
        const u32x4 rs = {(uint32_t)w, (uint32_t)(w >> 32) & 0xffffu, 0x7fffffffu, 0x00020000u};
        const u32x4 rs8 = {(uint32_t)w8, (uint32_t)(w8 >> 32) & 0xffffu, 0x7fffffffu, 0x00020000u};
        // slot 64 i + lane: input channel 8 i + lane / 8, piece lane % 8
        auto source = [&](int i) {
            const int ci = 8 * i + (lane >> 3);
            return (uint32_t)(128 * (lane >> 3) + 16 * ((lane & 7) ^ (ci & 2) ^ ((ci >> 1) & 4)));
        };
        const uint32_t even = source(0), odd = source(1);
        cv_each([&](auto index) {
            constexpr int i = decltype(index)::value;     // of 1 KB
            if constexpr (i % 4 == 0) cv_lds_base(ring0 + kCvEarly * kCvRowBytes + 1024 * i);
            cv_dma16<1024 * (i % 4)>(rs, (i % 2 ? odd : even) + 4096 * (i / 4));
        }, std::make_integer_sequence<int, 16>{});
        cv_lds_base(cv_lds_addr(s_stage) + 2048 * wv);
        cv_dma16<0>(rs8, even);
        cv_dma16<1024>(rs8, odd);
    }

    // task = column segment: image n, strip of 32 pixels, rows y0 .. y0 + len - 1.  The waves of a workgroup take tasks beside each other.
    const uint32_t task = (uint32_t)xcd_contiguous(blockIdx.x, gridDim.x) * kCvWaves + wv;
    const bool active = task < p.ntasks;
    const uint32_t per_img = (uint32_t)p.tiles_x * p.nseg;
    const uint32_t n = active ? task / per_img : 0u, rest = active ? task - n * per_img : 0u;
    const uint32_t sg = rest / (uint32_t)p.tiles_x;
    const int x0 = kCvTX * (int)(rest - sg * p.tiles_x);
    const int y0 = (int)sg * p.seg_len, len = min(p.seg_len, p.H - y0);
    const uint32_t row_bytes = (uint32_t)p.W * 128u;

    // Requests, rows y0 - 1, y0, ... one after the other: slot 64 i + lane of a row holds channel piece (lane & 7) ^ ((px >> 1) & 7) of pixel
    // px = 8 i + lane / 8 (image column x0 - 1 + px).  Pixels left and right of the image lie beyond the descriptor and arrive as zeros;
    // a row outside the image, or that the segment doesn't need, has a descriptor of length zero.
    uint32_t off[kCvRowLoads];
#pragma unroll
    for (int i = 0; i < kCvRowLoads; ++i) {
        const int px = 8 * i + (lane >> 3), x = x0 - 1 + px;
        off[i] = x >= 0 && x < p.W ? (uint32_t)(128 * (lane >> 3) + (i == 4 ? 4096 : 0) + 16 * ((lane & 7) ^ ((px >> 1) & 7))) : kCvOutside;
    }
    uint64_t from = (uint64_t)p.in + (((int64_t)n * p.H + (y0 - 1)) * p.W + (x0 - 1)) * 128;
    int from_y = y0 - 1;
    const int end_y = active ? min(p.H, y0 + len + 1) : 0;
    uint32_t from_at = ring0;
    u32x4 from_rs;
    auto aim_request = [&]() {
        from_rs = u32x4{(uint32_t)from, (uint32_t)(from >> 32) & 0xffffu, (uint32_t)from_y < (uint32_t)end_y ? 0x7fffffffu : 0u, 0x00020000u};
        cv_lds_base(from_at);
    };
    auto request = [&](auto part) {
        constexpr int i = decltype(part)::value;
        if constexpr (i < 4) {
            cv_dma16<1024 * i>(from_rs, off[i]);
        } else {
            cv_lds_base(from_at + 4096);
            cv_dma16_part<16>(from_rs, off[4]);
        }
    };
    auto next_request = [&]() {
        from += row_bytes;
        ++from_y;
        from_at += kCvRowBytes;
        if (from_at == ring0 + kCvRingBytes) from_at = ring0;
    };
    auto request_row = [&]() {
        aim_request();
        cv_each(request, std::make_integer_sequence<int, kCvRowLoads>{});
        next_request();
    };
#pragma unroll 1
    for (int r = 0; r < kCvEarly; ++r) request_row();

    // coefficient fragments: wf[ct][s] lane (c, g) = w[tap][32 kc + 8g + i][16 ct + c], s = 2 tap + kc
    half8 wf[4][18];
    cv_wait_loads<kCvEarly * kCvRowLoads>();
    lds_barrier();
    {
        // a transposing read: lane 4 r + q of 16 points at elements 4q .. 4q + 3 of row r, and lane c receives element c of the four rows
        const int ci = 8 * g + (c >> 2);                  // bits 1 and 3 are those of 32 kc + ci, and of ci + 4
        const int t = 128 * ci + 8 * (c & 3), flip = 32 * (((ci >> 1) & 1) | ((ci >> 2) & 2));
        int at[4];
#pragma unroll
        for (int ct = 0; ct < 4; ++ct) at[ct] = t + ((32 * ct) ^ flip);
        typedef short short4v __attribute__((ext_vector_type(4)));
        auto read = [&](int ct, int s, int u) {
            const int tap = s >> 1;
            const char* base = tap < 8 ? s_ring + (tap >> 1) * kCvRingBytes + kCvEarly * kCvRowBytes + (tap & 1) * kCvTapBytes : s_stage;
            return __builtin_bit_cast(half4, __builtin_amdgcn_ds_read_tr16_b64_v4i16(
                                                 (__attribute__((address_space(3))) short4v*)(base + at[ct] + 4096 * (s & 1) + 512 * u)));
        };
#pragma unroll
        for (int s = 0; s < 18; ++s)
#pragma unroll
            for (int ct = 0; ct < 4; ++ct) wf[ct][s] = join(read(ct, s, 0), read(ct, s, 1));
    }
    lds_barrier();
    if (!active) {
        cv_wait_loads<0>();                               // nothing may arrive in LDS that is no longer this workgroup's
        return;
    }
    // 64 of the 72 fragments live in the accumulation registers
#pragma unroll
    for (int ct = 0; ct < 4; ++ct)
#pragma unroll
        for (int s = 0; s < 16; ++s) asm volatile("" : "+a"(wf[ct][s]));
#pragma unroll 1
    for (int r = kCvEarly; r < kCvRing; ++r) request_row();

    // pixel fragments of the row in use: b[pt][i] lane (c, g) = channels 32 kc + 8g .. + 7 of pixel 16 pt + c + kx, i = 2 kx + kc
    half8 b[2][6];
    int part[3];
#pragma unroll
    for (int kx = 0; kx < 3; ++kx) part[kx] = (c + kx) * 128 + 16 * (g ^ (((c + kx) >> 1) & 7));
    uint32_t row_at = 0;
    auto load = [&](int pt, int i) { b[pt][i] = *reinterpret_cast<const half8*>(ring + row_at + ((part[i >> 1] ^ (64 * (i & 1))) + 2048 * pt)); };
    auto next_row = [&]() { row_at = row_at + kCvRowBytes == kCvRingBytes ? 0 : row_at + kCvRowBytes; };

    // the 48 products of a row with kernel row KY, and after product j what between(j) puts there
    auto products = [&](auto ky, floatx4 (&acc)[4][2], auto between) {
        constexpr int KY = decltype(ky)::value;
        cv_each([&](auto index) {
            constexpr int j = decltype(index)::value, pt = j / 24, ct = j / 6 % 4, i = j % 6;
            acc[ct][pt] = mfma16x16x32(wf[ct][6 * KY + i], b[pt][i], KY == 0 && i == 0 ? floatx4{0.f, 0.f, 0.f, 0.f} : acc[ct][pt]);
            cv_pin();
            between(index);
            cv_pin();
        }, std::make_integer_sequence<int, 48>{});
    };

    // way out: lane (c, g) holds channels 16 ct + 4g .. + 3 of pixel 16 pt + c
    char* const put = stage + c * kCvStagePitch + 8 * g;
    const char* const get = stage + (lane >> 3) * kCvStagePitch + 16 * (lane & 7);
    auto lay = [&](int i, const half4& v) { *reinterpret_cast<half4*>(put + 16 * kCvStagePitch * (i >> 2) + 32 * (i & 3)) = v; };      // i = 4 pt + ct
    half8 line[4];
    auto take = [&](int i) { line[i] = *reinterpret_cast<const half8*>(get + 8 * i * kCvStagePitch); };
    const uint32_t cols = (uint32_t)min(kCvTX, p.W - x0) * 128u;          // bytes of a row of the strip; what lies beyond is dropped
    uint64_t to = (uint64_t)p.out + (((int64_t)n * p.H + y0) * p.W + x0) * 128;
    auto give = [&](int i) {
        const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(reinterpret_cast<void*>(to), 0, (int)cols, 0x00020000);
        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, line[i]), rs, 16 * lane + 1024 * i, 0, kCvStream);
    };

    // Row r of the segment (-1 .. len) contributes to output rows r - 1 (kernel row 2), r (1) and r + 1 (0).
    floatx4 acc0[4][2], acc1[4][2];
    constexpr CvInt<0> ky0{};
    constexpr CvInt<1> ky1{};
    constexpr CvInt<2> ky2{};
    // kernel row 0: starts output row r + 1; row r + kCvRing is requested into the place of row r, and the fragments of row r + 1 take those of row r
    auto first = [&](floatx4 (&acc)[4][2]) {
        products(ky0, acc, [&](auto index) {
            constexpr int j = decltype(index)::value;
            if constexpr (j == 0) aim_request();
            if constexpr (j == 2) request(CvInt<0>{});
            if constexpr (j == 5) request(CvInt<1>{});
            if constexpr (j == 8) request(CvInt<2>{});
            if constexpr (j == 11) request(CvInt<3>{});
            if constexpr (j == 14) request(CvInt<4>{});
            if constexpr (j == 16) next_request();
            if constexpr (j == 17) next_row();
            if constexpr (j == 19) cv_wait_loads<kCvRowLoads * (kCvRing - 1)>();          // row r + 1 is there; with four stores a row, later ones may be waited for too
            if constexpr (j >= 24 && j < 36 && j % 2 == 0) load(0, (j - 24) / 2);
        });
    };
    auto next = [&]() {                                   // there is no output row r + 1: the fragments alone
        next_row();
        cv_wait_loads<kCvRowLoads * (kCvRing - 2)>();
#pragma unroll
        for (int i = 0; i < 6; ++i) load(0, i);
        cv_pin();
    };
    auto last = [&](floatx4 (&acc)[4][2]) {
        products(ky2, acc, [&](auto index) {
            constexpr int j = decltype(index)::value;
            if constexpr (j >= 1 && j < 13 && j % 2 == 1) load(1, j / 2);
        });
    };
    auto middle = [&](floatx4 (&acc)[4][2], const floatx4 (&done)[4][2]) {
        products(ky1, acc, [&](auto index) {
            constexpr int j = decltype(index)::value;
            if constexpr (j >= 2 && j < 26 && (j - 2) % 3 == 0) lay((j - 2) / 3, to_half4(done[(j - 2) / 3 & 3][(j - 2) / 12]));
            if constexpr (j == 25) wave_lds_fence();
            if constexpr (j >= 26 && j < 30) take(j - 26);
            if constexpr (j >= 40 && j % 2 == 0) give((j - 40) / 2);
            if constexpr (j == 47) to += row_bytes;
        });
        wave_lds_fence();
    };
    auto finish = [&](floatx4 (&done)[4][2]) {
#pragma unroll
        for (int i = 0; i < 8; ++i) lay(i, to_half4(done[i & 3][i >> 2]));
        wave_lds_fence();
#pragma unroll
        for (int i = 0; i < 4; ++i) take(i);
        cv_wait_loads<0>();                               // as above
#pragma unroll
        for (int i = 0; i < 4; ++i) give(i);
    };

    cv_wait_loads<kCvRowLoads * (kCvRing - 1)>();         // row -1
#pragma unroll
    for (int i = 0; i < 12; ++i) load(i / 6, i % 6);
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");    // read, before its place is requested over
    cv_pin();
    first(acc0);
#pragma unroll
    for (int i = 0; i < 6; ++i) load(1, i);
    cv_pin();
    products(ky1, acc0, [](auto) {});
    if (len == 1) {
        next();
        last(acc0);
        finish(acc0);
        return;
    }
    first(acc1);
    for (int r = 1;; r += 2) {
        last(acc0);
        middle(acc1, acc0);
        if (r + 1 == len) {
            next();
            last(acc1);
            finish(acc1);
            return;
        }
        first(acc0);
        last(acc1);
        middle(acc0, acc1);
        if (r + 2 == len) {
            next();
            last(acc0);
            finish(acc0);
            return;
        }
        first(acc1);
    }
}

// ---------------------------------------------------------------------------
// Vector-ALU twin: one thread per output pixel and 32 output channels, fp32 FMAs; pixels from the
// same LDS tile, weights through uniform (scalar) loads.
__global__ void __launch_bounds__(512) conv3x3_valu_kernel(ConvArgs p) {
    __shared__ __attribute__((aligned(16))) half_t s_in[kCvLdsHalves];
    const int tid = threadIdx.x;
    const int tile = blockIdx.x;
    const int n = tile / (p.tiles_x * p.tiles_y);
    const int rem = tile - n * (p.tiles_x * p.tiles_y);
    const int ty = rem / p.tiles_x, tx = rem - ty * p.tiles_x;
    const int y0 = ty * kCvTY, x0 = tx * kCvTX;
    const half_t* img = p.in + (int64_t)n * p.H * p.W * kCvC;
    for (int idx = tid; idx < kCvRows * kCvPx * 8; idx += 512) {
        const int piece = idx & 7;
        const int pr = idx >> 3;
        const int r = pr / kCvPx, px = pr - r * kCvPx;
        const int y = y0 - 1 + r, x = x0 - 1 + px;
        half8 v = {0, 0, 0, 0, 0, 0, 0, 0};
        if (y >= 0 && y < p.H && x >= 0 && x < p.W)
            v = *reinterpret_cast<const half8*>(img + ((int64_t)y * p.W + x) * kCvC + 8 * piece);
        *reinterpret_cast<half8*>(&s_in[cv_lds_index(r, piece >> 1, piece & 1, px)]) = v;
    }
    __syncthreads();
    const int cohalf = __builtin_amdgcn_readfirstlane(tid >> 8);   // waves 0-3: channels 0..31, waves 4-7: 32..63
    const int pid = tid & 255;
    const int ro = pid >> 5, xi = pid & 31;
    float acc[32];
#pragma unroll
    for (int i = 0; i < 32; ++i) acc[i] = 0.f;
    for (int tap = 0; tap < 9; ++tap) {
        const int ky = tap / 3, kx = tap - 3 * ky;
        for (int kc = 0; kc < 4; ++kc) {
            const half8 a = *reinterpret_cast<const half8*>(&s_in[cv_lds_index(ro + ky, kc, 0, xi + kx)]);
            const half8 b = *reinterpret_cast<const half8*>(&s_in[cv_lds_index(ro + ky, kc, 1, xi + kx)]);
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                const float xv = (float)(i < 8 ? a[i] : b[i - 8]);
                const half_t* wrow = p.w + ((tap * kCvC) + 16 * kc + i) * kCvC + 32 * cohalf;   // uniform
#pragma unroll
                for (int co = 0; co < 32; ++co) acc[co] = fmaf(xv, (float)wrow[co], acc[co]);
            }
        }
    }
    const int y = y0 + ro, x = x0 + xi;
    if (y < p.H && x < p.W) {
        half_t* o = p.out + (((int64_t)n * p.H + y) * p.W + x) * kCvC + 32 * cohalf;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            half8 v8;
#pragma unroll
            for (int r = 0; r < 8; ++r) v8[r] = (half_t)acc[8 * q + r];
            *reinterpret_cast<half8*>(o + 8 * q) = v8;
        }
    }
}

static hb_status conv_prepare(ConvArgs& a, const hb_half* in, const hb_half* w, hb_half* out,
                              int N, int H, int W, int Cin, int Cout) {
    if (!in || !w || !out) return HB_ERR_INVALID_ARG;
    if (N < 1 || H < 1 || W < 1 || Cin < 1 || Cout < 1) return HB_ERR_INVALID_ARG;
    if (!aligned_to(in, 16) || !aligned_to(w, 16) || !aligned_to(out, 16)) return HB_ERR_INVALID_ARG;
    if (Cin != kCvC || Cout != kCvC) return HB_ERR_UNSUPPORTED;
    const int64_t tiles = (int64_t)N * ceil_div(H, kCvTY) * ceil_div(W, kCvTX);
    if (tiles > 0x7fffffff || (int64_t)N * H * W > ((int64_t)1 << 40)) return HB_ERR_UNSUPPORTED;
    if ((int64_t)H * W * kCvC * 2 >= ((int64_t)1 << 31)) return HB_ERR_UNSUPPORTED;   // 32-bit offsets inside an image
    a.in = reinterpret_cast<const half_t*>(in);
    a.w = reinterpret_cast<const half_t*>(w);
    a.out = reinterpret_cast<half_t*>(out);
    a.N = N;
    a.H = H;
    a.W = W;
    a.tiles_x = ceil_div(W, kCvTX);
    a.tiles_y = ceil_div(H, kCvTY);
    a.ntiles = (int)tiles;
    // Column segments of the MFMA kernel: a compute unit holds four waves, so the strips are cut into as many equal segments as fill the
    // chip some whole number of times and not once more.  A round costs its segment's rows and the start of a workgroup, weights
    // and first rows, about three rows' time (a row 1 to 1.5 us); the cheapest number of rounds is taken.
    const int64_t columns = (int64_t)N * a.tiles_x, waves = (int64_t)kCvWaves * num_cu();
    const int64_t least = (columns + waves - 1) / waves;
    int len = H;
    int64_t cheapest = INT64_MAX;
    for (int64_t rounds = least; rounds < least + 16; ++rounds) {
        const int64_t segments = std::min<int64_t>(rounds * waves / columns, H);
        const int64_t rows_each = (H + segments - 1) / segments, cost = rounds * (rows_each + 3);
        if (cost < cheapest) {
            cheapest = cost;
            len = (int)rows_each;
        }
    }
    a.seg_len = len;
    a.nseg = ceil_div(H, len);
    a.ntasks = (uint32_t)(columns * a.nseg);              // at most 16 rounds more than columns
    return HB_OK;
}

}  // namespace hb

extern "C" hb_status hb_conv3x3(const hb_half* in_nhwc, const hb_half* w_hwio, hb_half* out_nhwc,
                                int N, int H, int W, int Cin, int Cout, hb_stream stream) {
    using namespace hb;
    ConvArgs a;
    hb_status s = conv_prepare(a, in_nhwc, w_hwio, out_nhwc, N, H, W, Cin, Cout);
    if (s != HB_OK) return s;
    const int64_t blocks = ((int64_t)a.ntasks + kCvWaves - 1) / kCvWaves;
    if (blocks > 0x7fffffff) return HB_ERR_UNSUPPORTED;
    hipLaunchKernelGGL(conv3x3_mfma_kernel, dim3((unsigned)blocks), dim3(64 * kCvWaves), 0,
                       reinterpret_cast<hipStream_t>(stream), a);
    return launch_status();
}

extern "C" hb_status hb_conv3x3_valu(const hb_half* in_nhwc, const hb_half* w_hwio, hb_half* out_nhwc,
                                     int N, int H, int W, int Cin, int Cout, hb_stream stream) {
    using namespace hb;
    ConvArgs a;
    hb_status s = conv_prepare(a, in_nhwc, w_hwio, out_nhwc, N, H, W, Cin, Cout);
    if (s != HB_OK) return s;
    hipLaunchKernelGGL(conv3x3_valu_kernel, dim3(a.ntiles), dim3(512), 0, reinterpret_cast<hipStream_t>(stream), a);
    return launch_status();
}
