// rows_f32.h -- blocks of 16 rows by 16 in plain f32, straight from global
// memory: what the split-operand attention kernels recompute rows with whose
// fast result is not finite.
//
// A wave holds 16 stationary rows, one per lane il = lane % 16, and walks the
// streamed side 16 rows at a time with v_mfma_f32_16x16x4_f32; lane group
// g = lane / 16 holds streamed rows 4g .. 4g + 3 of a block.  A streamed row
// that a stationary one must not see takes no part at all (a product with a
// zero weight would turn an infinity into NaN): blocks in which the mask differs
// between rows go through add16_visible.  One row at a time over the wave, as
// this was first written, an input with a NaN took 15 to 90 times a finite
// one's time; by blocks it takes 1.1 to 3 times (B8 H8 L1024 d64 causal, one
// NaN in V: forward 5.2 ms -> 157 us, backward 15.3 ms -> 442 us).
#pragma once

#include "device_common.h"

namespace mg {

// Hides where a value comes from: what is computed from it stays after this
// point, and the rare path does not change how the kernel before it is
// scheduled (B2 H6 L1500 d64 forward 71.2 us without this path, with it inlined
// 74.7, so 71.4).
__device__ __forceinline__ void hide(int &lane, int &uniform) {
    asm volatile("" : "+v"(lane), "+s"(uniform));
}

// This lane's floats [16s + 4g, +4) of its stationary row; zeros if !valid.
template <int D>
__device__ __forceinline__ void load_row16(f32x4 (&v)[D / 16], const float *row, bool valid, int g) {
#pragma unroll
    for (int s = 0; s < D / 16; ++s)
        v[s] = valid ? *reinterpret_cast<const f32x4 *>(row + 16 * s + 4 * g) : zero4();
}

// Dot products [streamed row 4g + r][stationary row il]; streamed rows at or
// beyond n read as zeros.
template <int D>
__device__ __forceinline__ f32x4 dot16(const float *rows, int n, const f32x4 (&b)[D / 16], int il,
                                       int g) {
    const auto rsrc = buffer_rsrc(rows, min(n, 16) * D * 4);
    f32x4 acc = zero4();
#pragma unroll
    for (int s = 0; s < D / 16; ++s) {
        const f32x4 a = buffer_load_f32x4(rsrc, (il * D + 16 * s + 4 * g) * 4);
#pragma unroll
        for (int e = 0; e < 4; ++e) acc = mfma16x16x4(a[e], b[s][e], acc);
    }
    return acc;
}

// acc^T[16c + 4g + r][il] += sum over the block's streamed rows x of
// rows[x][16c + 4g + r] * w[x][il]; rows at or beyond n read as zeros.
template <int D>
__device__ __forceinline__ void add16(f32x4 (&acc)[D / 16], const float *rows, int n, f32x4 w,
                                      int il, int g) {
    const auto rsrc = buffer_rsrc(rows, min(n, 16) * D * 4);
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int c = 0; c < D / 16; ++c) {
            const float a = __builtin_bit_cast(
                float, __builtin_amdgcn_raw_buffer_load_b32(
                           rsrc, ((4 * g + r) * D + 16 * c + il) * 4, 0, 0));
            acc[c] = mfma16x16x4(a, w[r], acc[c]);
        }
}

// The same over the streamed rows x with visible(x), of those below n.
template <int D, typename F>
__device__ __forceinline__ void add16_visible(f32x4 (&acc)[D / 16], const float *rows, int n,
                                              f32x4 w, int il, int g, F &&visible) {
    for (int x = 0; x < min(n, 16); ++x) {
        const int r = x & 3;   // w[x][il] lies in register r of lane il + 16 (x / 4)
        const float mine = r == 0 ? w[0] : r == 1 ? w[1] : r == 2 ? w[2] : w[3];
        const float wx = __shfl(mine, il + 16 * (x >> 2), 64);
        const bool on = visible(x);
#pragma unroll
        for (int c = 0; c < D / 16; ++c) {
            const f32x4 a = *reinterpret_cast<const f32x4 *>(rows + (size_t)x * D + 16 * c + 4 * g);
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (on) acc[c][e] = fmaf(a[e], wx, acc[c][e]);
        }
    }
}

// Every value of acc is NaN: nothing that is still to be added changes it.
template <int N>
__device__ __forceinline__ bool all_nan(const f32x4 (&acc)[N]) {
    bool nan = true;
#pragma unroll
    for (int c = 0; c < N; ++c)
#pragma unroll
        for (int e = 0; e < 4; ++e) nan = nan && acc[c][e] != acc[c][e];
    return nan;
}

}  // namespace mg
