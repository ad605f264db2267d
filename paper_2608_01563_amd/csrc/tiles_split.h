// tiles_split.h -- f32 products on the bf16 matrix cores: operands split into
// three bf16 parts, tiles of such parts in LDS.  The method is Henry, Tang and
// Heinecke, "Leveraging the bfloat16 Artificial Intelligence Datatype For
// Higher-Precision Computations" (IEEE ARITH 2019): f32 as three bf16 terms,
// six products.
//
// An f32 value x is written as x = h + m + l with h = bf16(x),
// m = bf16(x - h), l = bf16(x - h - m), all rounded to nearest even; both
// differences are exact, and what l drops is below 2^-24 |x| (8 + 8 + 8
// significant bits and the signs of m and l).  A product of two such values
// keeps the six terms of order 2^-16 and above,
//     xh yh + (xh ym + xm yh) + (xh yl + xm ym + xl yh),
// each exact in f32, summed by the matrix core in f32; the three dropped
// terms are below 2^-24 |x y| with either sign.  Measured against 64 bits on
// MI355X the sum of six v_mfma_f32_32x32x16_bf16 terms is closer than the
// v_mfma_f32_16x16x4_f32 chain it replaces (relative error over 32x32 blocks
// of normal data, six terms against f32 chain: contraction length 32
// 6.9e-8 : 1.04e-7, 64 1.10e-7 : 1.45e-7, 128 1.62e-7 : 2.03e-7, 1024
// 4.9e-7 : 5.7e-7, 4096 1.00e-6 : 1.14e-6), because one instruction adds
// sixteen products before it rounds.  At a sixteenth of the bf16 rate the f32
// instructions take 256 clocks for a 16x16x32 block, the six terms 96.
//
// Range: bf16 has f32's exponents, and parts below the smallest normal number
// (2^-126) are flushed.  So the parts are those of 2^24 x: the lowest bit of
// any f32, 2^-149, then lies in a normal part, and a product is 2^48 x y, which
// the kernels undo by exact factors (unscaled, operands below 2^-102 lose low
// bits: V about 2^-118, relative error of O 8.8e-6 against 3.3e-7).  An infinite
// or NaN operand, one above 2^103, or a sum above 2^79 makes the result
// infinite or NaN; the kernels check their results and recompute what is not
// finite with plain f32 arithmetic.
#pragma once

#include "device_common.h"
#include "tiles_bf16.h"

namespace mg {

constexpr float kUp = 0x1p24f;            // operands are split as kUp x ...
constexpr float kDown = 0x1p-24f;
constexpr float kDownProduct = 0x1p-48f;  // ... so products carry 2^48

struct Split8 {
    bf16x8 p[3];   // h, m, l of eight values
};

// Two f32 rounded to bf16 (nearest even), x in the low half.
__device__ __forceinline__ uint32_t pack2_bf16(float x, float y) {
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
    return __builtin_bit_cast(uint32_t, bf16x2{(__bf16)x, (__bf16)y});
}

// x minus the low (or high) bf16 of u, exact when u rounds x: one
// v_dot2_f32_bf16 instead of an unpack and a subtraction.  The -1 selecting
// the half sits in a register the compiler cannot see into: as an inline
// constant it would apply to both halves.
__device__ __forceinline__ float minus_bf16(float x, uint32_t u, uint32_t select) {
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
    return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, u),
                                           __builtin_bit_cast(bf16x2, select), x, false);
}

// N pairs of f32 into their parts, as packed pairs: three pair conversions and
// four exact remainders for two values.
template <int N>
__device__ __forceinline__ void split_pairs(const float (&x)[2 * N], uint32_t (&p)[3][N]) {
    uint32_t lo = 0x0000bf80u, hi = 0xbf800000u;
    asm("" : "+s"(lo), "+s"(hi));
#pragma unroll
    for (int i = 0; i < N; ++i) {
        float a = x[2 * i], b = x[2 * i + 1];
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            const uint32_t u = pack2_bf16(a, b);
            p[k][i] = u;
            if (k < 2) {
                a = minus_bf16(a, u, lo);
                b = minus_bf16(b, u, hi);
            }
        }
    }
}

__device__ __forceinline__ Split8 split8(const float (&x)[8]) {
    uint32_t p[3][4];
    split_pairs<4>(x, p);
    Split8 s;
#pragma unroll
    for (int k = 0; k < 3; ++k)
        s.p[k] = __builtin_bit_cast(bf16x8, u32x4{p[k][0], p[k][1], p[k][2], p[k][3]});
    return s;
}

__device__ __forceinline__ Split8 split8(f32x4 a, f32x4 b) {
    const float x[8] = {a[0], a[1], a[2], a[3], b[0], b[1], b[2], b[3]};
    return split8(x);
}

// Parts of an operand as it lies in memory, kUp times it.
__device__ __forceinline__ Split8 split8_up(f32x4 a, f32x4 b) { return split8(a * kUp, b * kUp); }

// The six terms (part of a, part of b), smallest first.
constexpr int kTermA[6] = {2, 1, 1, 0, 0, 0}, kTermB[6] = {0, 1, 0, 2, 1, 0};

// acc[n] += a * b[n], consecutive instructions sharing an operand ...
template <int N>
__device__ __forceinline__ void mfma_split(const Split8 &a, const Split8 (&b)[N], f32x4 (&acc)[N]) {
#pragma unroll
    for (int t = 0; t < 6; ++t)
#pragma unroll
        for (int n = 0; n < N; ++n)
            acc[n] = mfma16x16x32bf16(a.p[kTermA[t]], b[n].p[kTermB[t]], acc[n]);
}
// ... or acc[n] += a[n] * b.
template <int N>
__device__ __forceinline__ void mfma_split(const Split8 (&a)[N], const Split8 &b, f32x4 (&acc)[N]) {
#pragma unroll
    for (int t = 0; t < 6; ++t)
#pragma unroll
        for (int n = 0; n < N; ++n)
            acc[n] = mfma16x16x32bf16(a[n].p[kTermA[t]], b.p[kTermB[t]], acc[n]);
}

// An f32 [ROWS][D] tile that passes through registers, is split and lands in
// LDS (kUp times it) as three planes of TILE's layout (a Bf16Tile of the same shape), plane
// k at dst + k * TILE::kSize.  A thread moves chunks of eight floats of a row:
// two 16-byte buffer loads, three 16-byte LDS stores.  Rows at or beyond L
// arrive as zeros (the descriptor ends at row L).
template <class TILE, int ROWS, int D, int NT>
struct SplitStager {
    static constexpr int kCpr = D / 8;
    static constexpr int kChunks = ROWS * kCpr;
    static constexpr int kPer = (kChunks + NT - 1) / NT;
    static constexpr bool kExact = kChunks % NT == 0;
    f32x4 buf[kPer][2];

    __device__ __forceinline__ void load(const float *__restrict__ src, int row0, int L, int tid) {
        const int rows = min(max(L - row0, 0), ROWS);
        const auto rsrc = buffer_rsrc(src + (size_t)row0 * D, rows * D * 4);
#pragma unroll
        for (int u = 0; u < kPer; ++u) {
            const int off = 32 * (tid + u * NT);
            buf[u][0] = buffer_load_f32x4(rsrc, off);
            buf[u][1] = buffer_load_f32x4(rsrc, off + 16);
        }
    }
    __device__ __forceinline__ void store(uint16_t *dst, int tid) const {
#pragma unroll
        for (int u = 0; u < kPer; ++u) {
            const int f = tid + u * NT;
            if (!kExact && f >= kChunks) continue;
            const int r = f / kCpr;
            const int o = TILE::at(r, 8 * (f - r * kCpr));
            const Split8 s = split8_up(buf[u][0], buf[u][1]);
#pragma unroll
            for (int k = 0; k < 3; ++k)
                *reinterpret_cast<u32x4 *>(dst + k * TILE::kSize + o) =
                    __builtin_bit_cast(u32x4, s.p[k]);
        }
    }
};

// Operand reads from the three planes of a tile at u16 offset `o` of a plane.
template <class TILE>
__device__ __forceinline__ Split8 load_split(const uint16_t *t, int o) {
    Split8 s;
#pragma unroll
    for (int k = 0; k < 3; ++k) s.p[k] = load_bf16x8(t + k * TILE::kSize + o);
    return s;
}
template <class TILE>
__device__ __forceinline__ Split8 load_split_tr(const uint16_t *t, int lo, int hi) {
    Split8 s;
#pragma unroll
    for (int k = 0; k < 3; ++k)
        s.p[k] = load_tr_pair_at(t + k * TILE::kSize + lo, t + k * TILE::kSize + hi);
    return s;
}

__device__ __forceinline__ bool finite_f32(float x) {
    return (__float_as_uint(x) & 0x7f800000u) != 0x7f800000u;
}

}  // namespace mg
