// attn_few.hip -- attention forward for few query rows (a decode step, a
// handful of action tokens over a long context, a small model's layer), all
// three contracts.
//
// With at most 16 query rows per head the work is reading K and V once, and
// the query-stationary forwards leave most of their 64 or 128 rows empty;
// with few rows in all, their grids leave CUs empty and one wave walks all
// keys of its rows.  Here a workgroup takes 16 rows of one head and its NW
// waves deal the head's key tiles among themselves: wave w takes tiles w, w + NW, ...,
// keeps an online-softmax state of its own and the loads of its next tile in
// flight while it works on the current one, so the key loop has no barrier;
// the waves' states meet in LDS at the end.  There is no buffer to split a
// head's keys over workgroups, so when heads alone leave CUs idle a head's
// value columns are split instead: each of CS workgroups computes all scores
// and D/CS columns of O (its K reads hit the L2 the others fill).
//
// f32 (strict and accelerated): v_mfma_f32_16x16x4_f32 with operands straight
// from global memory, no LDS: a K row's four floats serve four products, and
// VE consecutive value columns of a row serve VE products whose output rows
// are every VE-th column.  Accelerated rounds Q, K, V and P to f16 first; the
// products of such values are exact in f32.  bf16: v_mfma_f32_16x16x32_bf16,
// K straight from global memory, V through wave-private LDS tiles (transpose
// reads).
//
// Bound at B8 H16 Lq1 Lk4096 d128, key lengths a quarter to all: bf16 83 -> 35
// us (168 MB, 4.8 TB/s; a large copy reaches 5.1), strict 268 -> 73 us,
// accelerated 107 -> 68 us (335 MB, 4.6 and 4.9 TB/s).
#include <type_traits>

#include "device_common.h"
#include "fwd_forms.h"
#include "launch.h"
#include "tiles_bf16.h"

namespace mg {
namespace {

// Online softmax of one 16-row block of queries (lane % 16), whose scores (in
// base-2 units, masked to -inf) lie in NB registers x 4 lane groups.
struct RowState {
    float m = -INFINITY, l = 0.f;

    // Turns scores into probabilities; returns the factor by which O must be
    // rescaled first (1 when no row's maximum moved).
    template <int NB>
    __device__ __forceinline__ float step(f32x4 (&s)[NB], bool &moved) {
        float mx = s[0][0];
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
            for (int r = 0; r < 4; ++r) mx = fmaxf(mx, s[b][r]);
        mx = max_over_groups(mx);
        const float mn = fmaxf(m, mx);
        const float mu = (mn == -INFINITY) ? 0.f : mn;
        const float alpha = exp2_fast(m - mu);
        moved = __any(mn != m);
        m = mn;
        float sum = 0.f;
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                s[b][r] = exp2_fast(s[b][r] - mu);
                sum += s[b][r];
            }
        l = l * alpha + sum;
        return alpha;
    }
};

// Float offset, in the waves' O states [NW][16 queries][DV], of 16-byte chunk
// c4 of query q of wave w; the chunks of a row are permuted so that the 16
// queries of a wave's store fall on different banks.
template <int DV>
__device__ __forceinline__ int state_at(int w, int q, int c4) {
    return (w * kFewRows + q) * DV + 4 * (c4 ^ (q & 7));
}

// Merge of the waves' states: wave w's m and l (per query) in ml[w], its O in
// xo.  Hands every 16-byte chunk of the result to `store` and writes LSE
// unless null.
template <int NW, int DV, typename Store>
__device__ __forceinline__ void merge_and_store(const float *xo, const float (*ml)[2][kFewRows],
                                                int tid, int rows, float *LSE, Store &&store) {
    constexpr int NT = 64 * NW;
    for (int f = tid; f < rows * (DV / 4); f += NT) {
        const int q = f / (DV / 4), c4 = f - q * (DV / 4);
        float m = -INFINITY;
#pragma unroll
        for (int w = 0; w < NW; ++w) m = fmaxf(m, ml[w][0][q]);
        const float mu = (m == -INFINITY) ? 0.f : m;
        float l = 0.f;
        f32x4 o = zero4();
#pragma unroll
        for (int w = 0; w < NW; ++w) {
            const float a = exp2_fast(ml[w][0][q] - mu);
            l += ml[w][1][q] * a;
            o += *reinterpret_cast<const f32x4 *>(&xo[state_at<DV>(w, q, c4)]) * a;
        }
        store(q, 4 * c4, o * ((l > 0.f) ? 1.f / l : 0.f));
        if (LSE != nullptr && c4 == 0) LSE[q] = row_lse(m, l);
    }
}


// ---------------------------------------------------------------------- f32 --
template <int D, int DV, int NW, int KT, bool ROUND>
__global__ __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(2, 8)))
void attn_fwd_few_f32(const float *__restrict__ Q, const float *__restrict__ K,
                      const float *__restrict__ V, float *__restrict__ O,
                      float *__restrict__ LSE, const int32_t *__restrict__ key_len, int H, int Lq,
                      int Lk, int causal, float scale_log2, int BH) {
    constexpr int NKB = KT / 16;                    // KT keys per wave and step
    constexpr int NS = D / 16;                      // 16-float pieces of a K row
    constexpr int VE = (DV / 16 < 4) ? DV / 16 : 4; // value columns per load
    constexpr int NCV = DV / (16 * VE);
    constexpr int CS = D / DV;
    typedef float vfrag __attribute__((ext_vector_type(VE)));
    __shared__ __attribute__((aligned(16))) float xo[NW > 1 ? NW * kFewRows * DV : 4];
    __shared__ float ml[NW][2][kFewRows];

    const int slot = blockIdx.x / BH;
    const int head = blockIdx.x - slot * BH;
    const int qt = slot / CS;
    const int col0 = (slot - qt * CS) * DV;
    const int tid = threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int il = lane & 15, g = lane >> 4;
    const int q0 = qt * kFewRows, qi = q0 + il;
    const int diag = Lk - Lq;
    const int klen = key_limit(key_len, head / H, Lk);
    const int kend = causal ? min(klen, min(q0 + kFewRows, Lq) + diag) : klen;
    const int ntiles = max((kend + KT - 1) / KT, 0);
    const float *Kh = K + (size_t)head * Lk * D;
    const float *Vh = V + (size_t)head * Lk * D + col0;

    // Q[qi][16s + 4g + e], strict times scale*log2e; rounded in pairs of s
    f32x4 qreg[NS];
    f16x8 qh[NS / 2];
#pragma unroll
    for (int s = 0; s < NS; ++s)
        qreg[s] = (qi < Lq) ? *reinterpret_cast<const f32x4 *>(
                                  Q + ((size_t)head * Lq + qi) * D + 16 * s + 4 * g)
                            : zero4();
#pragma unroll
    for (int s = 0; s < NS; ++s) {
        if (ROUND && (s & 1)) qh[s / 2] = to_f16x8(qreg[s - 1], qreg[s]);
        if (!ROUND) qreg[s] *= scale_log2;
    }

    struct Tile {
        f32x4 k[NKB][NS];           // K[16kb + il][16s + 4g + e]
        vfrag v[NKB][4][NCV];       // V[16kb + 4g + r][16 VE c + VE il + e]
    };
    // rows at or beyond the last allowed key read as zeros
    auto load = [&](int t, Tile &x) {
        const int row0 = t * KT, rows = min(max(kend - row0, 0), KT);
        const auto rk = buffer_rsrc(Kh + (size_t)row0 * D, rows * D * 4);
        const auto rv = buffer_rsrc(Vh + (size_t)row0 * D, rows * D * 4 - (rows > 0 ? col0 * 4 : 0));
#pragma unroll
        for (int kb = 0; kb < NKB; ++kb) {
#pragma unroll
            for (int s = 0; s < NS; ++s)
                x.k[kb][s] = buffer_load_f32x4(rk, ((16 * kb + il) * D + 16 * s + 4 * g) * 4);
#pragma unroll
            for (int r = 0; r < 4; ++r)
#pragma unroll
                for (int c = 0; c < NCV; ++c) {
                    const int off = ((16 * kb + 4 * g + r) * D + 16 * VE * c + VE * il) * 4;
                    if constexpr (VE == 4)
                        x.v[kb][r][c] = buffer_load_f32x4(rv, off);
                    else
                        x.v[kb][r][c] = __builtin_bit_cast(
                            vfrag, __builtin_amdgcn_raw_buffer_load_b64(rv, off, 0, 0));
                }
        }
    };

    RowState st;
    f32x4 oacc[NCV][VE];   // O^T[16 VE c + VE (4g + r) + e][qi]
#pragma unroll
    for (int c = 0; c < NCV; ++c)
#pragma unroll
        for (int e = 0; e < VE; ++e) oacc[c][e] = zero4();

    auto work = [&](int t, const Tile &x) {
        f32x4 s[NKB];
#pragma unroll
        for (int kb = 0; kb < NKB; ++kb) s[kb] = zero4();
#pragma unroll
        for (int i = 0; i < NS; ++i)
#pragma unroll
            for (int kb = 0; kb < NKB; ++kb) {
                if constexpr (ROUND) {
                    if (i & 1)
                        s[kb] = __builtin_amdgcn_mfma_f32_16x16x32_f16(
                            to_f16x8(x.k[kb][i - 1], x.k[kb][i]), qh[i / 2], s[kb], 0, 0, 0);
                } else {
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        s[kb] = mfma16x16x4(x.k[kb][i][e], qreg[i][e], s[kb]);
                }
            }
        const int j0 = t * KT + 4 * g;
        const int thr = causal ? min(klen - j0, qi + diag - j0 + 1) : klen - j0;
#pragma unroll
        for (int kb = 0; kb < NKB; ++kb)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const float v = ROUND ? s[kb][r] * scale_log2 : s[kb][r];
                s[kb][r] = (16 * kb + r < thr) ? v : -INFINITY;
            }
        bool moved;
        const float alpha = st.step(s, moved);
        if (moved) {
#pragma unroll
            for (int c = 0; c < NCV; ++c)
#pragma unroll
                for (int e = 0; e < VE; ++e) oacc[c][e] *= alpha;
        }
#pragma unroll
        for (int kb = 0; kb < NKB; ++kb) {
            if constexpr (ROUND) {   // the lane's four keys as one 16-deep product
                const f16x4 p = to_f16x4(s[kb]);
#pragma unroll
                for (int c = 0; c < NCV; ++c)
#pragma unroll
                    for (int e = 0; e < VE; ++e)
                        oacc[c][e] = __builtin_amdgcn_mfma_f32_16x16x16f16(
                            to_f16x4(f32x4{x.v[kb][0][c][e], x.v[kb][1][c][e], x.v[kb][2][c][e],
                                           x.v[kb][3][c][e]}),
                            p, oacc[c][e], 0, 0, 0);
            } else {
#pragma unroll
                for (int r = 0; r < 4; ++r)
#pragma unroll
                    for (int c = 0; c < NCV; ++c)
#pragma unroll
                        for (int e = 0; e < VE; ++e)
                            oacc[c][e] = mfma16x16x4(x.v[kb][r][c][e], s[kb][r], oacc[c][e]);
            }
        }
    };

    Tile a, b;
    if (w < ntiles) load(w, a);
    for (int t = w; t < ntiles; t += 2 * NW) {
        if (t + NW < ntiles) load(t + NW, b);
        work(t, a);
        if (t + NW < ntiles) {
            if (t + 2 * NW < ntiles) load(t + 2 * NW, a);
            work(t + NW, b);
        }
    }

    const float l = sum_over_groups(st.l);
    float *Oh = O + ((size_t)head * Lq + q0) * D + col0;
    float *Lh = col0 == 0 ? LSE + (size_t)head * Lq + q0 : nullptr;
    if constexpr (NW == 1) {   // the wave's state is the result
        if (qi >= Lq) return;
        const float inv = (l > 0.f) ? 1.f / l : 0.f;
#pragma unroll
        for (int c = 0; c < NCV; ++c)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                vfrag v;
#pragma unroll
                for (int e = 0; e < VE; ++e) v[e] = oacc[c][e][r] * inv;
                *reinterpret_cast<vfrag *>(Oh + (size_t)il * D + 16 * VE * c + VE * (4 * g + r)) = v;
            }
        if (Lh != nullptr && g == 0) Lh[il] = row_lse(st.m, l);
        return;
    }
    if (g == 0) {
        ml[w][0][il] = st.m;
        ml[w][1][il] = l;
    }
#pragma unroll
    for (int c = 0; c < NCV; ++c)
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
            for (int e = 0; e < VE; ++e) {
                const int col = 16 * VE * c + VE * (4 * g + r) + e;
                xo[state_at<DV>(w, il, col >> 2) + (col & 3)] = oacc[c][e][r];
            }
    __syncthreads();
    merge_and_store<NW, DV>(xo, ml, tid, min(kFewRows, Lq - q0), Lh,
                            [&](int q, int c, f32x4 v) {
                                *reinterpret_cast<f32x4 *>(Oh + (size_t)q * D + c) = v;
                            });
}

// --------------------------------------------------------------------- bf16 --
template <int D, int DV, int NW>
__global__ __launch_bounds__(64 * NW)
void attn_fwd_few_bf16(const uint16_t *__restrict__ Q, const uint16_t *__restrict__ K,
                       const uint16_t *__restrict__ V, uint16_t *__restrict__ O,
                       float *__restrict__ LSE, const int32_t *__restrict__ key_len, int H, int Lq,
                       int Lk, int causal, float scale_log2, int BH) {
    constexpr int KT = 32;
    constexpr int NKB = KT / 16;
    constexpr int NS = D / 32;
    constexpr int NC = DV / 16;
    constexpr int CS = D / DV;
    // V: [32 keys][DV] column blocks as in the dK/dV kernel's tiles, one pair
    // of tiles per wave; a wave's O state takes the place of its first tile.
    using Tile = Bf16Tile<KT, DV, 1, 32, 1, 3, 1>;
    constexpr int NL = Tile::kLoads;
    __shared__ __attribute__((aligned(16))) uint16_t V0[NW][Tile::kSize], V1[NW][Tile::kSize];
    static_assert(sizeof(V0) == NW * kFewRows * DV * sizeof(float), "states fit the tiles");
    float *const xo = reinterpret_cast<float *>(V0);
    __shared__ float ml[NW][2][kFewRows];

    const int slot = blockIdx.x / BH;
    const int head = blockIdx.x - slot * BH;
    const int qt = slot / CS;
    const int col0 = (slot - qt * CS) * DV;
    const int tid = threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int il = lane & 15, g = lane >> 4;
    const int jr = il >> 2, jc = 4 * (il & 3);
    const int q0 = qt * kFewRows, qi = q0 + il;
    const int diag = Lk - Lq;
    const int klen = key_limit(key_len, head / H, Lk);
    const int kend = causal ? min(klen, min(q0 + kFewRows, Lq) + diag) : klen;
    const int ntiles = max((kend + KT - 1) / KT, 0);
    const uint16_t *Kh = K + (size_t)head * Lk * D;
    const uint16_t *Vh = V + (size_t)head * Lk * D + col0;

    bf16x8 qreg[NS];
#pragma unroll
    for (int s = 0; s < NS; ++s)
        qreg[s] = (qi < Lq) ? load_bf16x8(Q + ((size_t)head * Lq + qi) * D + 32 * s + 8 * g)
                            : __builtin_bit_cast(bf16x8, u32x4{0u, 0u, 0u, 0u});

    using KReg = bf16x8[NKB][NS];   // K[16kb + il][32s + 8g + e]
    // this lane's byte offset within the rows of one direct-to-LDS load
    const int lr = lane / 4, lj = lane % 4;
    const int voff = lr * D * 2 + 16 * (lj ^ Tile::swz(lr));
    auto load = [&](int t, KReg &k, uint16_t *dst) {
        const int row0 = t * KT, rows = min(max(kend - row0, 0), KT);
        const auto rk = buffer_rsrc(Kh + (size_t)row0 * D, rows * D * 2);
        const auto rv = buffer_rsrc(Vh + (size_t)row0 * D, rows * D * 2 - (rows > 0 ? col0 * 2 : 0));
#pragma unroll
        for (int kb = 0; kb < NKB; ++kb)
#pragma unroll
            for (int s = 0; s < NS; ++s)
                k[kb][s] = __builtin_bit_cast(
                    bf16x8, __builtin_amdgcn_raw_buffer_load_b128(
                                rk, ((16 * kb + il) * D + 32 * s + 8 * g) * 2, 0, 0));
#pragma unroll
        for (int u = 0; u < NL; ++u) {
            const int r0 = (16 * u) % KT, blk = (16 * u) / KT;
            __builtin_amdgcn_raw_ptr_buffer_load_lds(
                rv, (__attribute__((address_space(3))) void *)(dst + 512 * u), 16,
                voff + r0 * D * 2 + 64 * blk, 0, 0, 0);
        }
    };
    const int va[2] = {Tile::at(4 * g + jr, jc), Tile::at(4 * g + jr, 16 + jc)};

    RowState st;
    f32x4 oacc[NC];   // O^T[16c + 4g + r][qi]
#pragma unroll
    for (int c = 0; c < NC; ++c) oacc[c] = zero4();

    auto work = [&](int t, const KReg &k, const uint16_t *vt) {
        f32x4 s[NKB];
#pragma unroll
        for (int kb = 0; kb < NKB; ++kb) {
            s[kb] = zero4();
#pragma unroll
            for (int i = 0; i < NS; ++i) s[kb] = mfma16x16x32bf16(k[kb][i], qreg[i], s[kb]);
        }
        const int j0 = t * KT + 4 * g;
        const int thr = causal ? min(klen - j0, qi + diag - j0 + 1) : klen - j0;
#pragma unroll
        for (int kb = 0; kb < NKB; ++kb)
#pragma unroll
            for (int r = 0; r < 4; ++r)
                s[kb][r] = (16 * kb + r < thr) ? s[kb][r] * scale_log2 : -INFINITY;
        bool moved;
        const float alpha = st.step(s, moved);
        if (moved) {
#pragma unroll
            for (int c = 0; c < NC; ++c) oacc[c] *= alpha;
        }
        const bf16x8 pb = pack_bf16(s[0], s[1]);
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            const int o = va[c & 1] + (c >> 1) * Tile::kBlock;
            oacc[c] = mfma16x16x32bf16(load_tr_pair_at(vt + o, vt + o + 32 * 16), pb, oacc[c]);
        }
    };

    // A tile's K (NKB*NS loads) and V (NL loads) are in flight while the one
    // before is consumed; V's arrival is waited for by count.
    constexpr int NV = NKB * NS + NL;
    KReg ka, kb;
    if (w < ntiles) load(w, ka, V0[w]);
    for (int t = w; t < ntiles; t += 2 * NW) {
        if (t + NW < ntiles) {
            load(t + NW, kb, V1[w]);
            wait_vmcnt<NV>();
        } else {
            wait_vmcnt<0>();
        }
        work(t, ka, V0[w]);
        if (t + NW < ntiles) {
            if (t + 2 * NW < ntiles) {
                load(t + 2 * NW, ka, V0[w]);
                wait_vmcnt<NV>();
            } else {
                wait_vmcnt<0>();
            }
            work(t + NW, kb, V1[w]);
        }
    }

    const float l = sum_over_groups(st.l);
    if (g == 0) {
        ml[w][0][il] = st.m;
        ml[w][1][il] = l;
    }
#pragma unroll
    for (int c = 0; c < NC; ++c)
        *reinterpret_cast<f32x4 *>(&xo[state_at<DV>(w, il, 4 * c + g)]) = oacc[c];
    __syncthreads();
    uint16_t *Oh = O + ((size_t)head * Lq + q0) * D + col0;
    merge_and_store<NW, DV>(xo, ml, tid, min(kFewRows, Lq - q0),
                            col0 == 0 ? LSE + (size_t)head * Lq + q0 : nullptr,
                            [&](int q, int c, f32x4 v) { store_bf16x4(Oh + (size_t)q * D + c, v); });
}

// Eight waves per workgroup where one workgroup per CU must keep a long key
// side's loads in flight, else four (two or more workgroups per CU; B2 H4
// L1024 causal strict: 24.9 us with eight, 22.1 with four).
int waves(const AttnProblem &p) {
    return few_row_blocks(p) * few_column_splits(p) <= 256 && p.Lk >= 1024 ? 8 : 4;
}

template <int X>
using Int = std::integral_constant<int, X>;

// f(d, value columns, waves) of the kernel for p.
template <typename F>
hipError_t by_shape(const AttnProblem &p, F &&f) {
    const int cs = few_column_splits(p), nw = waves(p);
#define MG_CASE(DD, CS)                                                  \
    if (p.d == DD && cs == CS)                                           \
        return nw == 8 ? f(Int<DD>{}, Int<DD / CS>{}, Int<8>{})          \
                       : f(Int<DD>{}, Int<DD / CS>{}, Int<4>{})
    MG_CASE(32, 1);
    MG_CASE(64, 1);
    MG_CASE(64, 2);
    MG_CASE(128, 1);
    MG_CASE(128, 2);
    MG_CASE(128, 4);
#undef MG_CASE
    return hipErrorInvalidValue;
}

}  // namespace

// bf16 and accelerated: a decode step (Lq <= 16) always; more rows while their
// 16-row blocks are few enough that spreading a head's keys over the waves pays
// for reading K and V once per block.  Against the query-stationary forwards
// (GPU time, this : those, us):
//   accelerated, up to 256 blocks: B4 H4 L256 5.4 : 8.8, d = 128 Lq32 Lk4096 0.8
//     of the other's time; 512: B1 H4 L2048 d128 76 : 54
//   bf16, up to 256 blocks: B4 H4 L256 4.0 : 7.2, Lq17 to 128 by Lk256 to 4096 0.3
//     to 0.8; up to 512 (1024: B8 H8 L256 8.2 : 6.5) where the blocks of a head
//     share its K and V in an L2: d = 32 (0.5 to 0.8), d = 64 to 512 keys (0.8 to
//     1.0), d = 128 to 128 keys (0.8 to 1.1), else with eight blocks a head, or
//     four of growing length, that land on at most two XCDs (heads a multiple of
//     four) or on few bytes in all: B2 H4 L1024 causal 9.8 : 16.1, B8 H8 L128 4.1 :
//     4.9; but d = 128 B1 H256 Lq32 Lk2048 1.48, B1 H73 Lq100 Lk1000 1.42, B1 H43
//     Lq128 Lk4000 1.29
bool use_few_rows(const AttnProblem &p, mg_contract_t contract) {
    const long blocks = few_row_blocks(p);
    if (p.Lq <= kFewRows || blocks <= 256) return true;
    if (contract != MG_CONTRACT_FAST_BF16 || blocks > 512) return false;
    if (p.d == 32 || p.Lk <= (p.d == 64 ? 512 : 128)) return true;
    const long BH = (long)p.B * p.H;
    return p.Lq >= (p.causal ? 64 : 128) && (BH % 4 == 0 || BH * p.Lk * p.d <= 1 << 21);
}

// The grid of a kernel of NW waves and DV value columns per workgroup.
template <typename Kern, typename T>
static hipError_t launch_few(Kern kern, const AttnProblem &p, int dv, int nw, const T *Q,
                             const T *K, const T *V, T *O, float *LSE, hipStream_t s) {
    kern<<<dim3((unsigned)(few_row_blocks(p) * (p.d / dv))), dim3(64 * nw), 0, s>>>(
        Q, K, V, O, LSE, p.key_len, p.H, p.Lq, p.Lk, p.causal, p.scale * kLog2e, p.B * p.H);
    return hipGetLastError();
}

hipError_t launch_fwd_few_f32(const AttnProblem &p, const float *Q, const float *K, const float *V,
                              float *O, float *LSE, FwdForm form, hipStream_t s) {
    auto go = [&](auto kern, int dv, int nw) {
        return launch_few(kern, p, dv, nw, Q, K, V, O, LSE, s);
    };
    if (form == FwdForm::kFewWave)
        return p.d == 32   ? go(attn_fwd_few_f32<32, 32, 1, 16, false>, 32, 1)
               : p.d == 64 ? go(attn_fwd_few_f32<64, 64, 1, 16, false>, 64, 1)
                           : go(attn_fwd_few_f32<128, 128, 1, 16, false>, 128, 1);
    if (form == FwdForm::kFew && p.d == 32) return go(attn_fwd_few_f32<32, 32, 4, 16, false>, 32, 4);
    if (form == FwdForm::kFew && p.d == 64)
        return few_column_splits(p) == 1 ? go(attn_fwd_few_f32<64, 64, 4, 16, false>, 64, 4)
                                         : go(attn_fwd_few_f32<64, 32, 4, 16, false>, 32, 4);
    return by_shape(p, [&](auto dd, auto dv, auto nw) {
        return go(attn_fwd_few_f32<dd(), dv(), nw(), 2048 / dd(), false>, dv(), nw());
    });
}

hipError_t launch_fwd_few_accel(const AttnProblem &p, const float *Q, const float *K,
                                const float *V, float *O, float *LSE, hipStream_t s) {
    return by_shape(p, [&](auto dd, auto dv, auto nw) {
        return launch_few(attn_fwd_few_f32<dd(), dv(), nw(), 2048 / dd(), true>, p, dv(), nw(), Q,
                          K, V, O, LSE, s);
    });
}

hipError_t launch_fwd_few_bf16(const AttnProblem &p, const uint16_t *Q, const uint16_t *K,
                               const uint16_t *V, uint16_t *O, float *LSE, hipStream_t s) {
    return by_shape(p, [&](auto dd, auto dv, auto nw) {
        return launch_few(attn_fwd_few_bf16<dd(), dv(), nw()>, p, dv(), nw(), Q, K, V, O, LSE, s);
    });
}

}  // namespace mg
