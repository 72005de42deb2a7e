// Device-side building blocks shared by the gfx950 kernels: vector types, MFMA
// wrappers with their operand-to-lane maps, edge-aware row loads and stores.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "hb_host.hpp"

namespace hb {

typedef _Float16 half_t;
typedef _Float16 half4 __attribute__((ext_vector_type(4)));
typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// ---------------------------------------------------------------------------
// Operand-to-lane maps on a 64-lane wave (lane = 16*g + c for the 16-wide shapes).
//
// v_mfma_f32_16x16x32_f16   D[16x16] += A[16x32] * B[32x16]
//   A: lane (c, g) holds A[c][8g .. 8g+7]        (8 halves)
//   B: lane (c, g) holds B[8g .. 8g+7][c]        (8 halves)
//   D: lane (c, g) holds D[4g .. 4g+3][c]        (4 floats)
// v_mfma_f32_16x16x16_f16   D[16x16] += A[16x16] * B[16x16]
//   A: lane (c, g) holds A[c][4g .. 4g+3];  B: lane (c, g) holds B[4g .. 4g+3][c];  D as above
// v_mfma_f32_16x16x4_f32    D[16x16] += A[16x4] * B[4x16]
//   A: lane (c, g) holds A[c][g];  B: lane (c, g) holds B[g][c];  D as above
// v_mfma_f32_32x32x16_f16   D[32x32] += A[32x16] * B[16x32]      (lane = 32*h + c)
//   A: lane (c, h) holds A[c][8h .. 8h+7];  B: lane (c, h) holds B[8h .. 8h+7][c]
//   D: lane (c, h) holds D[8q + 4h + r][c] in register 4q + r  (q, r = 0..3)
//
// Because a D fragment holds, per lane, a run of the ROW index for a fixed column,
// a D fragment rounded to fp16 is already a valid A or B fragment of a following
// product that contracts over that row index: no transpose, no LDS round trip.
// Two stacked 16-row D fragments t = 0, 1 form one K = 32 operand whose k-slot
// 8g + i stands for row 16*(i/4) + 4g + (i%4); the coefficient operand is built
// with the same slot order (see krow32 below), which leaves the sum unchanged.
// ---------------------------------------------------------------------------

// These wrappers are the only matrix products the kernels can issue (a test scans the sources for
// builtins used anywhere else).  For 16 x 16 fp16 products there is ONE shape, K = 32: a
// 16x16x16 product issued straight after a 16x16x32 on the same accumulator once gave a wrong
// first tile, so an accumulator chain never mixes the two; operands with K = 16 are padded with
// zeros.  The K = 16 instruction exists only inside the self-check kernel of util.hip.
__device__ __forceinline__ floatx4 mfma16x16x32(half8 a, half8 b, floatx4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ floatx4 mfma16x16x4f32(float a, float b, floatx4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ floatx16 mfma32x32x16(half8 a, half8 b, floatx16 c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_f16(a, b, c, 0, 0, 0);
}

// Row (within a 32-row window made of two stacked 16-row D fragments) that k-slot
// 8g + i of a chained K = 32 operand stands for.
__device__ __forceinline__ int krow32(int g, int i) { return 16 * (i >> 2) + 4 * g + (i & 3); }

__device__ __forceinline__ half4 to_half4(floatx4 v) {
    half4 r;
    r[0] = (half_t)v[0]; r[1] = (half_t)v[1]; r[2] = (half_t)v[2]; r[3] = (half_t)v[3];
    return r;
}
__device__ __forceinline__ half8 join(half4 lo, half4 hi) {
    return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
}

__device__ __forceinline__ int clampi(int v, int lo, int hi) { return v < lo ? lo : (v > hi ? hi : v); }

// Vector types with element alignment only: gfx950 under HSA runs with unaligned
// access enabled, so a 16-byte access needs no more than the alignment of its elements.
typedef half8 half8_u __attribute__((aligned(2)));
typedef half4 half4_u __attribute__((aligned(2)));
typedef floatx4 floatx4_u __attribute__((aligned(4)));

// Eight consecutive pixels row[xs .. xs+7] with the column index clamped to [0, W-1].
// One 16-byte load (any 2-byte aligned address) when the run lies inside the row.
__device__ __forceinline__ half8 load8_clamp(const half_t* __restrict__ row, int xs, int W) {
    if (xs >= 0 && xs + 8 <= W) {
        return *reinterpret_cast<const half8_u*>(row + xs);
    }
    half8 r;
#pragma unroll
    for (int i = 0; i < 8; ++i) r[i] = row[clampi(xs + i, 0, W - 1)];
    return r;
}

// Border windows.  Eight pixels from column xs on, part of them outside the row, are loaded from the
// nearest column that keeps the load inside (xs - d) and moved afterwards, in registers: one 16-byte
// load where a pixel-by-pixel load with clamped columns takes eight.  Element i becomes element
// min(i + d, 7) of the loaded run, d >= 0 (what lies past the last pixel repeats it, or is zero) ...
template <bool ZERO = false>
__device__ __forceinline__ half8 shift_in_from_right(half8 v, int d) {
    u32x4 a = __builtin_bit_cast(u32x4, v);
    const uint32_t t = ZERO ? 0u : (a[3] & 0xffff0000u) | (a[3] >> 16);
    const u32x4 s8 = {t, t, t, t}, s4 = {a[2], a[3], t, t};
    a = d >= 8 ? s8 : (d & 4) ? s4 : a;
    const u32x4 s2 = {a[1], a[2], a[3], t};
    a = (d & 2) && d < 8 ? s2 : a;
    const u32x4 s1 = {__builtin_amdgcn_alignbit(a[1], a[0], 16), __builtin_amdgcn_alignbit(a[2], a[1], 16),
                      __builtin_amdgcn_alignbit(a[3], a[2], 16), ZERO ? a[3] >> 16 : t};
    a = (d & 1) && d < 8 ? s1 : a;
    return __builtin_bit_cast(half8, a);
}
// ... or element max(i - d, 0) (what lies left of pixel 0 repeats it, or is zero).
template <bool ZERO = false>
__device__ __forceinline__ half8 shift_in_from_left(half8 v, int d) {
    u32x4 a = __builtin_bit_cast(u32x4, v);
    const uint32_t t = ZERO ? 0u : (a[0] << 16) | (a[0] & 0xffffu);
    const u32x4 s8 = {t, t, t, t}, s4 = {t, t, a[0], a[1]};
    a = d >= 8 ? s8 : (d & 4) ? s4 : a;
    const u32x4 s2 = {t, a[0], a[1], a[2]};
    a = (d & 2) && d < 8 ? s2 : a;
    const u32x4 s1 = {ZERO ? a[0] << 16 : t, __builtin_amdgcn_alignbit(a[1], a[0], 16), __builtin_amdgcn_alignbit(a[2], a[1], 16),
                      __builtin_amdgcn_alignbit(a[3], a[2], 16)};
    a = (d & 1) && d < 8 ? s1 : a;
    return __builtin_bit_cast(half8, a);
}

// Store four consecutive floats at row[x .. x+3], dropping columns >= W.
__device__ __forceinline__ void store4_mask(float* __restrict__ row, int x, int W, floatx4 v) {
    if (x + 4 <= W) {
        *reinterpret_cast<floatx4_u*>(row + x) = v;
    } else {
#pragma unroll
        for (int i = 0; i < 4; ++i)
            if (x + i < W) row[x + i] = v[i];
    }
}

// Accesses through a wave-uniform base plus a 32-bit per-lane BYTE offset: the form the
// hardware addresses with a scalar base register and one vector offset register.
__device__ __forceinline__ half8 ldg8(const half_t* base, uint32_t byte_off) {
    return *reinterpret_cast<const half8_u*>(reinterpret_cast<const char*>(base) + byte_off);
}
// Output stores.  STREAM = true marks the lines non-temporal (written once, not read back by the kernel): faster wherever
// a store instruction writes whole lines, at every output size (64 MB to 256 MB per call), and for outputs that the
// memory-side cache takes in.  Large outputs that leave in parts of lines are better put together in the L2 first: see
// the rules of hb_sat2d and of hb_down2 / hb_up2.
template <bool STREAM>
__device__ __forceinline__ void stg4(float* base, uint32_t byte_off, floatx4 v) {
    floatx4_u* q = reinterpret_cast<floatx4_u*>(reinterpret_cast<char*>(base) + byte_off);
    if (STREAM) __builtin_nontemporal_store(v, q); else *q = v;
}
// LDS traffic inside one wave: what the wave wrote is there for its own lanes (LDS serves one wave's
// instructions in order); only the compiler has to be kept from reordering.
__device__ __forceinline__ void wave_lds_fence() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// LDS written by this workgroup is there for all of it; loads from memory stay in flight (the compiler puts a
// wait for everything in front of a barrier it emits).
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// Accumulator tiles leave the MFMA with a lane owning four columns of ONE row and the 16 lanes
// of a quarter-wave owning 16 DIFFERENT rows, so a store instruction would touch each row with
// 16-byte pieces only.  Passing the NW tiles (16 rows x 16*NW floats) through a wave-private LDS
// patch turns that into stores of 16 consecutive lanes x 16 bytes = one 256-byte run of one row.
// The patch has a row pitch of 16*NW + 4 floats: both the accumulator-layout writes and the
// row-major reads are bank-conflict free.  Only the owning wave touches its patch and LDS serves
// one wave's instructions in order, so no workgroup barrier is needed.
template <int NW>
struct RowPatch {
    static constexpr int kPitch = 16 * NW + 4;
    static constexpr int kFloats = 16 * kPitch;
};
template <int NW, bool STREAM>
__device__ __forceinline__ void store_rows_via_lds(float* patch, float* dst, uint32_t pitch_elems,
                                                   const floatx4 (&acc)[NW], int lane) {
    const int c = lane & 15, g = lane >> 4;
#pragma unroll
    for (int w = 0; w < NW; ++w)
        *reinterpret_cast<floatx4*>(patch + c * RowPatch<NW>::kPitch + 16 * w + 4 * g) = acc[w];
    wave_lds_fence();
    constexpr int kLanesPerRow = 4 * NW;                  // 16-byte pieces in a row of the patch
    constexpr int kRowsPerPass = 64 / kLanesPerRow;
    const int rr = lane / kLanesPerRow, xq = lane - rr * kLanesPerRow;
#pragma unroll
    for (int s = 0; s < 16 / kRowsPerPass; ++s) {
        const int row = s * kRowsPerPass + rr;
        const floatx4 v = *reinterpret_cast<const floatx4*>(patch + row * RowPatch<NW>::kPitch + 4 * xq);
        stg4<STREAM>(dst, ((uint32_t)row * pitch_elems + 4u * xq) * 4u, v);
    }
    wave_lds_fence();
}

// store_rows_via_lds for a tile group at the image border: only rows < rows and columns < cols are
// stored, still as runs of one row per 4 NW lanes.
template <int NW, bool STREAM>
__device__ __forceinline__ void store_rows_via_lds_masked(float* patch, float* dst, int64_t pitch_elems,
                                                          const floatx4 (&acc)[NW], int lane, int rows, int cols) {
    const int c = lane & 15, g = lane >> 4;
#pragma unroll
    for (int w = 0; w < NW; ++w)
        *reinterpret_cast<floatx4*>(patch + c * RowPatch<NW>::kPitch + 16 * w + 4 * g) = acc[w];
    wave_lds_fence();
    constexpr int kLanesPerRow = 4 * NW, kRowsPerPass = 64 / kLanesPerRow;
    const int rr = lane / kLanesPerRow, x = 4 * (lane - rr * kLanesPerRow);
#pragma unroll
    for (int s = 0; s < 16 / kRowsPerPass; ++s) {
        const int row = s * kRowsPerPass + rr;
        const floatx4 v = *reinterpret_cast<const floatx4*>(patch + row * RowPatch<NW>::kPitch + x);
        if (row < rows) {
            float* q = dst + (int64_t)row * pitch_elems + x;
            if (x + 4 <= cols) {
                if (STREAM) __builtin_nontemporal_store(v, reinterpret_cast<floatx4_u*>(q));
                else *reinterpret_cast<floatx4_u*>(q) = v;
            } else {
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    if (x + i < cols) q[i] = v[i];
            }
        }
    }
    wave_lds_fence();
}

// Workgroups are handed to the 8 XCDs (each with its own L2) round-robin by workgroup id.
// This maps a workgroup id to a position such that every XCD works through one contiguous
// eighth of the positions, in order: neighbouring tasks, which share halo pixels, then meet
// in the same L2 at about the same time instead of each fetching the halo from memory.
#ifndef HB_XCD_CONTIGUOUS
#define HB_XCD_CONTIGUOUS 1
#endif
__device__ __forceinline__ int xcd_contiguous(int wg, int nwg) {
    if (!HB_XCD_CONTIGUOUS) return wg;
    const int per = nwg >> 3;                             // positions per XCD (remainder handled below)
    if (wg >= per * 8) return wg;                         // tail workgroups keep their place
    return (wg & 7) * per + (wg >> 3);
}

// The same idea at a finer grain: of every 8 G consecutive workgroup ids, XCD x (which receives
// ids x, x + 8, ...) takes G consecutive positions.  Neighbours still meet in one L2, while the chip
// as a whole sweeps through the tasks in launch order, as it does with the plain order.
__device__ __forceinline__ int xcd_blocked(int wg, int nwg, int G) {
    const int span = 8 * G, first = (wg / span) * span;
    if (first + span > nwg) return wg;                    // tail workgroups keep their place
    const int r = wg - first;
    return first + (r & 7) * G + (r >> 3);
}

// Toeplitz fragment = eight consecutive entries of the zero-padded tap table that travels in the
// kernel arguments (see TapsT): one 16-byte load at a 2-byte aligned address.
__device__ __forceinline__ half8 tap_run(const uint16_t* tab, int t0) {
    return *reinterpret_cast<const half8_u*>(tab + kTapPad + t0);
}
__device__ __forceinline__ half_t tap_at(const uint16_t* tab, int t) {
    return __builtin_bit_cast(half_t, tab[kTapPad + t]);
}

}  // namespace hb
