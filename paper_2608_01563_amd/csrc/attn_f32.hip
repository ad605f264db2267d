// attn_f32.hip -- strict-f32 attention kernels for gfx950 (f32 MFMA).
//
// The paper's attention archetype is three kernels: a tiled forward, a dQ
// kernel and a fused dK+dV kernel (Sec. 3.3; Sec. 8 makes the fused dK+dV
// kernel a compiler invariant; Sec. 7.3 profiles the backward pair).  The
// forward and the separate dK/dV and dQ kernels run on split bf16 operands
// (attn_f32x3_*.hip); here:
//
//   attn_rowdot_f32   D_i = sum_k dO_ik O_ik (HBM-bound row reduction).
//   attn_dkdvq_f32    key tile stationary: recomputes P from LSE, then
//                     dV += P^T dO, dP = dO V^T, dS = P(dP - D), dK += dS^T Q,
//                     and the dQ product of its key tile, dQ_part = dS K_tile,
//                     to the workspace, one partial per (key tile, query
//                     row) (d <= 64).
//   attn_dq_reduce_f32  dQ = scale * sum of a row's partials, in key-tile
//                     order (fixed order: bitwise-reproducible, no atomics).
//
// Every product runs on v_mfma_f32_16x16x4_f32 (f32 inputs, f32 accumulate),
// which is what the strict contract permits (Sec. 4.2).  Each wave owns 16
// rows of the stationary tile (one per lane column l%16); the other operand
// is staged through LDS, 64 rows at a time, and shared by the waves of a
// workgroup.
//
// Workgroup order: the 1-D grid is numbered rank-major over heads
// (id = slot * B*H + head) with rank 0 the tile that has the most work under
// a causal mask.  When the grid is larger than what the chip holds at once,
// slot = rank, so the longest tiles start first and the dispatcher hands the
// short ones to whichever CU frees up; when every workgroup is resident at
// once, layers of slots alternate direction (serpentine_rank) so that each
// CU holds a mix of long and short tiles.  With B*H a multiple of 8 every
// tile of a head lands on the same XCD (workgroups are dealt to the eight
// XCDs round-robin), so a head's K/V or Q/dO stay in one L2.
//
// Masking: an element's offset inside its tile is compared against one
// per-lane threshold (key length, causal diagonal).
#include <algorithm>
#include <climits>
#include <type_traits>

#include "device_common.h"
#include "launch.h"
#include "tiles_direct.h"
#include "work_order.h"

// Per-kernel launch configuration: waves per workgroup, minimum waves per
// SIMD requested from the register allocator (0 = compiler default), and
// double-buffered LDS for the streamed tile.  The defaults are
// the fastest of sweeps on MI355X at B8 H8 L1024 d64 and B16 H12 L512 d64
// (double buffering lost there: it halves the workgroups an LDS-heavy CU can
// hold); they can be overridden at build time.
#ifndef MG_DKDV_CFG
#define MG_DKDV_CFG 4, 3, false
#endif
#ifndef MG_DKDVQ_CAUSAL_CFG
#define MG_DKDVQ_CAUSAL_CFG 8, 4, false   // 128-key tiles: half the dQ partials
#endif
#ifndef MG_DKDVQ_CAUSAL_NIB
#define MG_DKDVQ_CAUSAL_NIB 2   // 16-row query blocks per step, 128-key fused kernel
#endif
#ifndef MG_DKDV_NIB
#define MG_DKDV_NIB 2   // 16-row query blocks per dK/dV step (d <= 64)
#endif

namespace mg {
namespace {

template <int NW_, int OCC_, bool DB_>
struct Cfg {
    static constexpr int NW = NW_;             // waves per workgroup
    static constexpr int NT = 64 * NW_;        // threads per workgroup
    static constexpr int ROWS = 16 * NW_;      // stationary rows per workgroup
    static constexpr int OCC = OCC_ > 0 ? OCC_ : 1;
    static constexpr int NBUF = DB_ ? 2 : 1;   // LDS buffers for the streamed tile
};
using DkdvCfg = Cfg<MG_DKDV_CFG>;
using DkdvqCausalCfg = Cfg<MG_DKDVQ_CAUSAL_CFG>;

// ------------------------------------------------- backward: D = rowsum(dO o O)
template <int D>
__global__ __launch_bounds__(256) void attn_rowdot_f32(const float *__restrict__ O,
                                                       const float *__restrict__ dO,
                                                       float *__restrict__ Dws, int rows) {
    constexpr int TPR = D / 4;   // threads per row, one 16-byte chunk each
    const int row = blockIdx.x * (256 / TPR) + threadIdx.x / TPR;
    const int c4 = threadIdx.x % TPR;
    float v = 0.f;
    if (row < rows) {
        const f32x4 o = *reinterpret_cast<const f32x4 *>(O + (size_t)row * D + 4 * c4);
        const f32x4 go = *reinterpret_cast<const f32x4 *>(dO + (size_t)row * D + 4 * c4);
        v = o[0] * go[0] + o[1] * go[1] + o[2] * go[2] + o[3] * go[3];
    }
#pragma unroll
    for (int m = TPR / 2; m >= 1; m >>= 1) v += xor_lanes(v, m);
    if (row < rows && c4 == 0) Dws[row] = v;
}

// ---------------------------------------- backward: dK, dV and dQ partials
// A workgroup keeps a key tile's K and V and walks the query tiles.  After dS
// of a query tile is known, it goes through LDS and the workgroup multiplies it
// by its own key tile, dQ_part[i][:] = sum_{j in tile} dS[i][j] K[j][:].
// Each (key tile, query row) partial is written once to the workspace and
// attn_dq_reduce_f32 adds the partials of a row in key-tile order: no atomics,
// bitwise-reproducible, and no second recompute of S and dP.
//
// The Q and dO tiles, and the LSE and D values of their rows, reach LDS by
// row-wise direct-to-LDS loads (no staging registers, padded rows); dQ partials
// leave through raw buffer stores whose descriptor ends at row Lq.  With two LDS
// buffers (C::NBUF == 2) the next tile is fetched during the whole current
// iteration; with one, during the dQ product.  A tile's dQ partials are stored
// at the start of the next iteration, so the wait for the next tile never waits
// on a just-issued store.
//
// Small grids (LOCALD): the O rows of each query tile arrive with its Q and
// dO rows, and the workgroup computes D_i = sum_k dO_ik O_ik in LDS before
// the softmax needs it, so no separate D launch precedes the kernel.  With a
// single key tile and no query split (direct_dq), the one partial of a row is
// its dQ: it is scaled and written to dQ (dQp points there), rows outside the
// tile's query range get zeros, and no reduction follows (LOCALD grids only,
// so that the large-grid instances carry none of this).
template <int D, int NIB, class C, bool LOCALD>
__global__ __launch_bounds__(C::NT) __attribute__((amdgpu_waves_per_eu(C::OCC, 8)))
void attn_dkdvq_f32(const float *__restrict__ Q, const float *__restrict__ K,
                    const float *__restrict__ V, const float *__restrict__ O,
                    const float *__restrict__ dO, const float *__restrict__ LSE,
                    const float *__restrict__ Dws, float *__restrict__ dK,
                    float *__restrict__ dV, float *__restrict__ dQp, float *__restrict__ dKVp,
                    const int32_t *__restrict__ key_len, int H, int Lq, int Lk, int causal,
                    float scale, float scale_log2, int BH, int nsplit, int nranks, int layer,
                    int work_first, int direct_dq) {
    constexpr int DQ = D / 4;
    constexpr int NC = D / 16;
    constexpr int BR = 16 * NIB;
    constexpr int KR = C::ROWS;                 // keys per workgroup
    constexpr int NBLK = NIB * NC;              // 16x16 blocks of a dQ partial tile
    constexpr int PER_WAVE = (NBLK + C::NW - 1) / C::NW;
    constexpr int NB = C::NBUF;
    constexpr int LD = D + 4;
    using Tile = RowDirectTile<BR, D, C::NW, LD>;
    __shared__ __attribute__((aligned(16))) float Qs[NB][BR][LD];
    __shared__ __attribute__((aligned(16))) float dOs[NB][BR][LD];
    __shared__ __attribute__((aligned(16))) float lse2s[NB][BR];    // LSE (natural log)
    __shared__ __attribute__((aligned(16))) float Ds[NB][BR];
    __shared__ __attribute__((aligned(16))) float Os[LOCALD ? NB : 1][LOCALD ? BR : 1][LD];
    __shared__ __attribute__((aligned(16))) float Kt[D][KR + 4];    // key tile, transposed
    __shared__ __attribute__((aligned(16))) float dSs[BR][KR + 4];  // dS of the query tile

    int slot, head;
    if (work_first) {
        work_first_tile(blockIdx.x, nranks, nsplit, C::ROWS, BH, H, Lk, key_len, slot, head);
    } else {
        slot = blockIdx.x / BH;
        head = blockIdx.x - slot * BH;
    }
    const int rank = serpentine_rank(slot, nranks, layer);
    const int kt = rank / nsplit;          // key tile
    const int split = rank - kt * nsplit;  // share of its query tiles
    const int b = head / H;
    const size_t qoff = (size_t)head * Lq * D, hoff = (size_t)head * Lk * D;
    const float *Qh = Q + qoff;
    const float *dOh = dO + qoff;
    const int diag = Lk - Lq;   // causal: row i sees keys j <= i + diag

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int il = lane & 15;
    const int g = lane >> 4;
    const int k0 = kt * KR;
    const int wkey0 = k0 + 16 * w;   // first key of this wave (wave-uniform)
    const int kj = wkey0 + il;

    const int klen = key_limit(key_len, b, Lk);
    const int nq = (Lq + BR - 1) / BR;
    // first query tile holding a row that sees key k0, and the end of the
    // range; split `split` of `nsplit` takes a contiguous share of it
    const int qfirst = causal ? min(nq, max(0, k0 - diag) / BR) : 0;
    const int qlast = (k0 < klen) ? nq : qfirst;
    const int qstart = qfirst + (int)((long)(qlast - qfirst) * split / nsplit);
    const int qstop = qfirst + (int)((long)(qlast - qfirst) * (split + 1) / nsplit);

    const Tile tile;

    // Direct-to-LDS loads of the Q and dO rows of query tile qt, and of their
    // LSE (wave 0) and D (the last wave) values, or with LOCALD of their O
    // rows instead of D; rows past Lq arrive as zeros.
    auto fetch = [&](int qt, int buf) {
        tile.issue(Qs[buf], Qh, qt * BR, Lq, w, lane);
        tile.issue(dOs[buf], dOh, qt * BR, Lq, w, lane);
        if constexpr (LOCALD) tile.issue(Os[buf], O + qoff, qt * BR, Lq, w, lane);
        if (w == 0 || (!LOCALD && w == C::NW - 1)) {
            const int row0 = qt * BR;
            const int rows = min(max(Lq - row0, 0), BR);
            const float *src = (w == 0 ? LSE : Dws) + (size_t)head * Lq + row0;
            const auto rsrc = buffer_rsrc(src, rows * 4);
            float *dst = (w == 0) ? lse2s[buf] : Ds[buf];
            if (lane < BR)
                __builtin_amdgcn_raw_ptr_buffer_load_lds(
                    rsrc, (__attribute__((address_space(3))) void *)dst, 4, lane * 4, 0, 0, 0);
        }
    };
    if (qstart < qstop) fetch(qstart, 0);

    float kreg[DQ], vreg[DQ];
#pragma unroll
    for (int s4 = 0; s4 < DQ / 4; ++s4) {
        const size_t off = hoff + (size_t)kj * D + g * DQ + 4 * s4;
        const f32x4 kv = (kj < Lk) ? *reinterpret_cast<const f32x4 *>(K + off) : zero4();
        const f32x4 vv = (kj < Lk) ? *reinterpret_cast<const f32x4 *>(V + off) : zero4();
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            kreg[4 * s4 + e] = kv[e];
            vreg[4 * s4 + e] = vv[e];
        }
    }
    // The key tile, transposed, for the A operand of the dQ product.
    for (int f = tid; f < KR * (D / 4); f += C::NT) {
        const int row = f / (D / 4);
        const int c4 = f - row * (D / 4);
        const f32x4 v = (k0 + row < Lk)
            ? *reinterpret_cast<const f32x4 *>(K + hoff + (size_t)(k0 + row) * D + 4 * c4)
            : zero4();
#pragma unroll
        for (int e = 0; e < 4; ++e) Kt[4 * c4 + e][row] = v[e];
    }

    f32x4 dkacc[NC], dvacc[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) {
        dkacc[c] = zero4();
        dvacc[c] = zero4();
    }

    // Under a causal mask element (ib, r) is query ibase + 16ib + r, allowed
    // iff it is >= kj - diag; a padded key (kj >= key length) is masked everywhere
    // so that it adds nothing to dQ.
    // (sentinels +-2^30 keep kthr - ibase free of overflow)
    constexpr int kNever = 1 << 30;
    const int kthr = (kj >= klen) ? kNever : (causal ? kj - diag : -kNever);

    // dQ partial blocks of this wave: consecutive blocks (same query rows,
    // shared dS reads) when they split evenly, else strided
    auto dq_block = [&](int bb) {
        return (NBLK % C::NW == 0) ? w * PER_WAVE + bb : w + bb * C::NW;
    };
    f32x4 dqacc[PER_WAVE];   // partials of the previous query tile, not yet stored
    // Raw buffer stores through a descriptor that covers the tile's rows below
    // Lq: stores of rows past Lq fall outside it and are dropped.
    float *dQp_head = dQp + ((size_t)kt * BH + head) * Lq * D;
    auto store_dq = [&](int qt) {
        const int row0 = qt * BR;
        const auto rsrc = buffer_rsrc(dQp_head + (size_t)row0 * D, min(Lq - row0, BR) * D * 4);
#pragma unroll
        for (int bb = 0; bb < PER_WAVE; ++bb) {
            const int blk = dq_block(bb);
            if (NBLK % C::NW != 0 && blk >= NBLK) break;
            const int ib = blk / NC;
            const int c = blk - ib * NC;
            __builtin_amdgcn_raw_buffer_store_b128(
                __builtin_bit_cast(u32x4, (LOCALD && direct_dq) ? dqacc[bb] * scale : dqacc[bb]),
                rsrc,
                ((16 * ib + il) * D + 16 * c + 4 * g) * 4, 0, 0);
        }
    };

    // D of the tile in buffer buf from its landed dO and O rows: TPR threads
    // per row, each summing every TPR-th 4-float chunk, then a butterfly.
    auto local_d = [&](int buf) {
        if constexpr (LOCALD) {
            constexpr int TPR = C::NT / BR;
            static_assert(C::NT % BR == 0 && (TPR & (TPR - 1)) == 0 && TPR <= 64,
                          "threads per row");
            const int row = tid / TPR, part = tid - (tid / TPR) * TPR;
            float acc = 0.f;
#pragma unroll
            for (int c4 = part; c4 < D / 4; c4 += TPR) {
                const f32x4 a = *reinterpret_cast<const f32x4 *>(&dOs[buf][row][4 * c4]);
                const f32x4 o = *reinterpret_cast<const f32x4 *>(&Os[buf][row][4 * c4]);
#pragma unroll
                for (int e = 0; e < 4; ++e) acc = fmaf(a[e], o[e], acc);
            }
#pragma unroll
            for (int m = TPR / 2; m >= 1; m >>= 1) acc += xor_lanes(acc, m);
            if (part == 0) Ds[buf][row] = acc;
        }
    };

    if (qstart < qstop) wait_vmcnt<0>();
    __syncthreads();   // first tile, its LSE/D and Kt visible
    if (LOCALD) {
        if (qstart < qstop) local_d(0);
        __syncthreads();   // its D visible
    }

    for (int qt = qstart; qt < qstop; ++qt) {
        const int cb = (NB == 2) ? ((qt - qstart) & 1) : 0;
        if (qt > qstart) store_dq(qt - 1);
        if (NB == 2 && qt + 1 < qstop) fetch(qt + 1, cb ^ 1);

        // A wave whose 16 keys are all masked for every row of this query
        // tile (padded keys, or keys past the tile's last row under a causal
        // mask) contributes nothing but its zero block of dS.
        const bool live = wkey0 < klen && (!causal || wkey0 - diag <= qt * BR + BR - 1);
        if (live) {
            f32x4 sacc[NIB], pacc[NIB];
#pragma unroll
            for (int ib = 0; ib < NIB; ++ib) {
                sacc[ib] = zero4();
                pacc[ib] = zero4();
            }
            // S = Q K^T, then dP = dO V^T: one product at a time keeps one
            // set of A operands live, so the kernel fits in 128 VGPRs (four
            // waves per SIMD, two 8-wave workgroups per CU).
#pragma unroll
            for (int s4 = 0; s4 < DQ / 4; ++s4) {
                f32x4 aq[NIB];
#pragma unroll
                for (int ib = 0; ib < NIB; ++ib)
                    aq[ib] = *reinterpret_cast<const f32x4 *>(&Qs[cb][16 * ib + il][g * DQ + 4 * s4]);
#pragma unroll
                for (int e = 0; e < 4; ++e)
#pragma unroll
                    for (int ib = 0; ib < NIB; ++ib)
                        sacc[ib] = mfma16x16x4(aq[ib][e], kreg[4 * s4 + e], sacc[ib]);
            }
#pragma unroll
            for (int s4 = 0; s4 < DQ / 4; ++s4) {
                f32x4 ao[NIB];
#pragma unroll
                for (int ib = 0; ib < NIB; ++ib)
                    ao[ib] = *reinterpret_cast<const f32x4 *>(&dOs[cb][16 * ib + il][g * DQ + 4 * s4]);
#pragma unroll
                for (int e = 0; e < 4; ++e)
#pragma unroll
                    for (int ib = 0; ib < NIB; ++ib)
                        pacc[ib] = mfma16x16x4(ao[ib][e], vreg[4 * s4 + e], pacc[ib]);
            }

            const int ibase = qt * BR + 4 * g;
            const int thr = kthr - ibase;
#pragma unroll
            for (int ib = 0; ib < NIB; ++ib) {
                const f32x4 l2 = *reinterpret_cast<const f32x4 *>(&lse2s[cb][16 * ib + 4 * g]) * kLog2e;
                const f32x4 dd = *reinterpret_cast<const f32x4 *>(&Ds[cb][16 * ib + 4 * g]);
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    float p = exp2_fast(sacc[ib][r] * scale_log2 - l2[r]);
                    p = (16 * ib + r >= thr) ? p : 0.f;
                    sacc[ib][r] = p;
                    pacc[ib][r] = p * (pacc[ib][r] - dd[r]);
                    dSs[16 * ib + 4 * g + r][16 * w + il] = pacc[ib][r];
                }
            }

#pragma unroll
            for (int ib = 0; ib < NIB; ++ib)
#pragma unroll
                for (int r = 0; r < 4; ++r)
#pragma unroll
                    for (int c = 0; c < NC; ++c) {
                        dvacc[c] = mfma16x16x4(dOs[cb][16 * ib + 4 * g + r][16 * c + il],
                                               sacc[ib][r], dvacc[c]);
                        dkacc[c] = mfma16x16x4(Qs[cb][16 * ib + 4 * g + r][16 * c + il],
                                               pacc[ib][r], dkacc[c]);
                    }
        } else {
#pragma unroll
            for (int ib = 0; ib < NIB; ++ib)
#pragma unroll
                for (int r = 0; r < 4; ++r) dSs[16 * ib + 4 * g + r][16 * w + il] = 0.f;
        }

        __syncthreads();   // dS complete (and, single-buffered, Q/dO consumed)
        if (NB == 1 && qt + 1 < qstop) fetch(qt + 1, 0);

        // dQ_part^T[16c + 4g + r][16ib + il] = sum_j K^T[16c + il'][j] dS^T[j][16ib + il]
        // over the 16-key blocks that hold an allowed key for some row of the
        // tile (the rest of dS is zero: past the key length, or past the
        // tile's last row under a causal mask)
        int qblocks = min(KR / 16, (klen - k0 + 15) / 16);
        if (causal) qblocks = min(qblocks, max(0, qt * BR + BR - 1 + diag - k0) / 16 + 1);
        // (full tiles keep a loop without exits, which the compiler schedules freely)
        auto dq_product = [&](auto full) {
#pragma unroll
            for (int bb = 0; bb < PER_WAVE; ++bb) {
                const int blk = dq_block(bb);
                if (NBLK % C::NW != 0 && blk >= NBLK) break;
                const int ib = blk / NC;
                const int c = blk - ib * NC;
                f32x4 acc = zero4();
#pragma unroll
                for (int q = 0; q < KR / 16; ++q) {
                    if (!decltype(full)::value && q >= qblocks) break;
                    const f32x4 bv = *reinterpret_cast<const f32x4 *>(&dSs[16 * ib + il][16 * q + 4 * g]);
                    const f32x4 av = *reinterpret_cast<const f32x4 *>(&Kt[16 * c + il][16 * q + 4 * g]);
#pragma unroll
                    for (int e = 0; e < 4; ++e) acc = mfma16x16x4(av[e], bv[e], acc);
                }
                dqacc[bb] = acc;
            }
        };
        if (qblocks == KR / 16)
            dq_product(std::true_type{});
        else
            dq_product(std::false_type{});

        if (qt + 1 < qstop) wait_vmcnt<0>();   // next Q/dO tile and its LSE/D landed
        __syncthreads();   // next tile visible; dS and this tile's buffer free
        if (LOCALD) {
            if (qt + 1 < qstop) local_d(NB == 2 ? (cb ^ 1) : 0);
            __syncthreads();   // its D visible
        }
    }
    if (qstart < qstop) store_dq(qstop - 1);
    if (LOCALD && direct_dq) {
        // rows no query tile of this workgroup wrote (none see a key) get zeros
        float *dqh = dQp + (size_t)head * Lq * D;
        const int r0 = min(qstart * BR, Lq), r1 = min(qstop * BR, Lq);
        const int nz = (r0 + (Lq - r1)) * (D / 4);
        for (int f = tid; f < nz; f += C::NT) {
            const int rr = f / (D / 4);
            const int row = rr < r0 ? rr : r1 + (rr - r0);
            *reinterpret_cast<f32x4 *>(dqh + (size_t)row * D + 4 * (f - rr * (D / 4))) = zero4();
        }
    }

    // One split writes dK and dV directly; several write partials laid out
    // [dK, dV][split][B*H][Lk][d] (every split writes its rows, zeros for an
    // empty share) for attn_bwd_reduce_f32.
    if (kj < Lk) {
        const bool keep = kj < klen;
        const size_t row = hoff + (size_t)kj * D;
        const size_t part = (size_t)BH * Lk * D;
        float *dkrow = (nsplit == 1) ? dK + row : dKVp + (size_t)split * part + row;
        float *dvrow = (nsplit == 1) ? dV + row : dKVp + (size_t)(nsplit + split) * part + row;
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            *reinterpret_cast<f32x4 *>(dkrow + 16 * c + 4 * g) = keep ? dkacc[c] * scale : zero4();
            *reinterpret_cast<f32x4 *>(dvrow + 16 * c + 4 * g) = keep ? dvacc[c] : zero4();
        }
    }
}

// dK and dV from the per-split partials of attn_dkdvq_f32, added in
// increasing split order (a fixed order).  n4 = B*H*Lk*d / 4; idx runs over
// the 2*n4 16-byte chunks of dK then dV.
__device__ __forceinline__ void dkdv_reduce_at(long idx, const float *__restrict__ dKVp,
                                               float *__restrict__ dK, float *__restrict__ dV,
                                               int nsplit, long n4) {
    if (idx >= 2 * n4) return;
    const int t = idx >= n4;           // 0: dK, 1: dV
    const long e4 = idx - t * n4;
    const f32x4 *src = reinterpret_cast<const f32x4 *>(dKVp) + (long)t * nsplit * n4 + e4;
    f32x4 sum = zero4();
    for (int s = 0; s < nsplit; ++s) sum += src[(long)s * n4];
    reinterpret_cast<f32x4 *>(t ? dV : dK)[e4] = sum;
}

// dQ[i] = scale * sum over key tiles kt that hold an allowed key for row i of
// dQ_part[kt][i], added in increasing kt (a fixed order).  Partials are laid
// out [key tile][B*H][Lq][d].
template <int D>
__device__ __forceinline__ void dq_reduce_at(size_t idx, const float *__restrict__ dQp,
                                             float *__restrict__ dQ,
                                             const int32_t *__restrict__ key_len, int H, int Lq,
                                             int Lk, int causal, float scale, int BH,
                                             int key_rows) {
    constexpr int C4 = D / 4;
    const size_t total = (size_t)BH * Lq * C4;
    if (idx >= total) return;
    const size_t rowg = idx / C4;              // head * Lq + i
    const int head = (int)(rowg / Lq);
    const int i = (int)(rowg - (size_t)head * Lq);
    const int klen = key_limit(key_len, head / H, Lk);
    const int nk = (klen + key_rows - 1) / key_rows;
    // causal: row i sees keys j <= i + Lk - Lq, i.e. key tiles up to that key's
    const int last = i + Lk - Lq;
    const int kmax = causal ? (last < 0 ? 0 : min(nk, last / key_rows + 1)) : nk;
    const size_t stride = (size_t)BH * Lq * D;
    const float *src = dQp + idx * 4;
    f32x4 sum = zero4();
    for (int kt = 0; kt < kmax; ++kt)
        sum += *reinterpret_cast<const f32x4 *>(src + (size_t)kt * stride);
    *reinterpret_cast<f32x4 *>(dQ + idx * 4) = sum * scale;
}

template <int D>
__global__ __launch_bounds__(256) void attn_dq_reduce_f32(const float *__restrict__ dQp,
                                                          float *__restrict__ dQ,
                                                          const int32_t *__restrict__ key_len,
                                                          int H, int Lq, int Lk, int causal,
                                                          float scale, int BH, int key_rows) {
    dq_reduce_at<D>((size_t)blockIdx.x * 256 + threadIdx.x, dQp, dQ, key_len, H, Lq, Lk, causal,
                    scale, BH, key_rows);
}

// Both reductions of a query-split fused backward in one launch: the first
// nb_kv workgroups add the dK/dV partials, the rest the dQ partials.
template <int D>
__global__ __launch_bounds__(256) void attn_bwd_reduce_f32(
    const float *__restrict__ dKVp, float *__restrict__ dK, float *__restrict__ dV, int nsplit,
    long n4, unsigned nb_kv, const float *__restrict__ dQp, float *__restrict__ dQ,
    const int32_t *__restrict__ key_len, int H, int Lq, int Lk, int causal, float scale, int BH,
    int key_rows) {
    if (blockIdx.x < nb_kv)
        dkdv_reduce_at((long)blockIdx.x * 256 + threadIdx.x, dKVp, dK, dV, nsplit, n4);
    else
        dq_reduce_at<D>((size_t)(blockIdx.x - nb_kv) * 256 + threadIdx.x, dQp, dQ, key_len, H,
                        Lq, Lk, causal, scale, BH, key_rows);
}

}  // namespace

// ---------------------------------------------------------------- launchers
hipError_t launch_bwd_rowdot_f32(const AttnProblem &p, const float *O, const float *dO,
                                 float *Dws, hipStream_t s) {
    const int rows = p.B * p.H * p.Lq;
    const dim3 block(256);
    switch (p.d) {
    case 32: attn_rowdot_f32<32><<<dim3(cdiv(rows, 256 / 8)), block, 0, s>>>(O, dO, Dws, rows); break;
    case 64: attn_rowdot_f32<64><<<dim3(cdiv(rows, 256 / 16)), block, 0, s>>>(O, dO, Dws, rows); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

// Fused dQ: causal problems with enough work use 128-key tiles (heavy-first
// ordering keeps the fewer workgroups balanced, and the partials halve);
// the rest keep 64-key tiles, which measured faster there.
bool wide_key_tiles(const AttnProblem &p) {
    return p.causal && (long)cdiv(p.Lk, DkdvqCausalCfg::ROWS) * p.B * p.H >= 512;
}
int fused_dq_key_rows(const AttnProblem &p) {
    return wide_key_tiles(p) ? DkdvqCausalCfg::ROWS : DkdvCfg::ROWS;
}

// Few keys (a short context, few heads) leave the key-stationary grid far
// smaller than the chip: below MG_DKDV_SPLIT_BELOW workgroups, each key
// tile's query tiles are split over up to ceil(MG_DKDV_SPLIT_TARGET / grid)
// workgroups, keeping at least MG_DKDV_SPLIT_MIN_TILES query tiles each.
#ifndef MG_DKDV_SPLIT_BELOW
#define MG_DKDV_SPLIT_BELOW 512
#endif
#ifndef MG_DKDV_SPLIT_TARGET
#define MG_DKDV_SPLIT_TARGET 1024
#endif
#ifndef MG_DKDV_SPLIT_MIN_TILES
#define MG_DKDV_SPLIT_MIN_TILES 4
#endif
int fused_dq_query_splits(const AttnProblem &p) {
    const long grid = (long)cdiv(p.Lk, fused_dq_key_rows(p)) * p.B * p.H;
    if (grid >= MG_DKDV_SPLIT_BELOW) return 1;
    const int br = 16 * (wide_key_tiles(p) ? MG_DKDVQ_CAUSAL_NIB : MG_DKDV_NIB);
    const long by_grid = (MG_DKDV_SPLIT_TARGET + grid - 1) / grid;
    // short query sides (at most 8 tiles) split down to 2 tiles per share:
    // each share is then latency-bound, and finer shares measured faster
    const int nqt = cdiv(p.Lq, br);
    const long by_tiles = nqt / (nqt <= 8 ? 2 : MG_DKDV_SPLIT_MIN_TILES);
    return (int)std::max(1L, std::min(by_grid, by_tiles));
}

// Small fused grids compute D in the kernel (LOCALD): at most this many key
// tiles per head, so that each query tile's O rows are read a few times, and
// a grid below MG_DKDV_SPLIT_BELOW workgroups.
#ifndef MG_LOCAL_D_MAX_KEY_TILES
#define MG_LOCAL_D_MAX_KEY_TILES 4
#endif
bool fused_local_d(const AttnProblem &p) {
    const long nkt = cdiv(p.Lk, fused_dq_key_rows(p));
    return nkt <= MG_LOCAL_D_MAX_KEY_TILES && nkt * p.B * p.H < MG_DKDV_SPLIT_BELOW;
}
bool fused_direct_dq(const AttnProblem &p) {
    return fused_local_d(p) && cdiv(p.Lk, fused_dq_key_rows(p)) == 1 &&
           fused_dq_query_splits(p) == 1;
}

template <class C, int NIB>
static hipError_t launch_dkdvq(const AttnProblem &p, const float *Q, const float *K,
                               const float *V, const float *O, const float *dO,
                               const float *LSE, const float *Dws, float *dK, float *dV,
                               float *dQp, float *dKVp, hipStream_t s) {
    const int BH = p.B * p.H;
    const int ns = fused_dq_query_splits(p);
    const int nr = cdiv(p.Lk, C::ROWS) * ns;   // ranks: key tile x split
    const dim3 grid(nr * BH), block(C::NT);
    const float sl2 = p.scale * kLog2e;
    const int direct = fused_direct_dq(p) ? 1 : 0;
    auto go = [&](auto kern) {
        const int ly = causal_rank_layer((const void *)kern, C::NT, grid.x, BH, p.causal);
        kern<<<grid, block, 0, s>>>(Q, K, V, O, dO, LSE, Dws, dK, dV, dQp, dKVp, p.key_len,
                                    p.H, p.Lq, p.Lk, p.causal, p.scale, sl2, BH, ns, nr, ly,
                                    padded_work_order(p), direct);
    };
    // Local D only in the 64-key form: grids small enough for it never take
    // the 128-key tiles, which need at least 512 workgroups.
    constexpr bool kLocalForm = !std::is_same<C, DkdvqCausalCfg>::value;
    const bool local = kLocalForm && fused_local_d(p);
    auto pick = [&](auto plain, auto with_local) {
        if constexpr (kLocalForm) {
            if (local) return go(with_local);
        }
        go(plain);
    };
    switch (p.d) {
    case 32: pick(attn_dkdvq_f32<32, NIB, C, false>, attn_dkdvq_f32<32, NIB, C, kLocalForm>); break;
    case 64: pick(attn_dkdvq_f32<64, NIB, C, false>, attn_dkdvq_f32<64, NIB, C, kLocalForm>); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_bwd_dkdvq_f32(const AttnProblem &p, const float *Q, const float *K,
                                const float *V, const float *O, const float *dO,
                                const float *LSE, const float *Dws, float *dK, float *dV,
                                float *dQp, float *dKVp, hipStream_t s) {
    if (fused_dq_query_splits(p) > 1 && dKVp == nullptr) return hipErrorInvalidValue;
    return wide_key_tiles(p)
        ? launch_dkdvq<DkdvqCausalCfg, MG_DKDVQ_CAUSAL_NIB>(p, Q, K, V, O, dO, LSE, Dws, dK, dV,
                                                            dQp, dKVp, s)
        : launch_dkdvq<DkdvCfg, MG_DKDV_NIB>(p, Q, K, V, O, dO, LSE, Dws, dK, dV, dQp, dKVp, s);
}

hipError_t launch_bwd_reduce_f32(const AttnProblem &p, const float *dKVp, float *dK,
                                 float *dV, const float *dQp, float *dQ, hipStream_t s) {
    const int BH = p.B * p.H;
    const long n4 = (long)BH * p.Lk * p.d / 4;
    const unsigned nb_kv = (unsigned)((2 * n4 + 255) / 256);
    const size_t total = (size_t)BH * p.Lq * (p.d / 4);
    const dim3 grid(nb_kv + (unsigned)((total + 255) / 256)), block(256);
    const int ns = fused_dq_query_splits(p), kr = fused_dq_key_rows(p);
    switch (p.d) {
    case 32: attn_bwd_reduce_f32<32><<<grid, block, 0, s>>>(dKVp, dK, dV, ns, n4, nb_kv, dQp, dQ, p.key_len, p.H, p.Lq, p.Lk, p.causal, p.scale, BH, kr); break;
    case 64: attn_bwd_reduce_f32<64><<<grid, block, 0, s>>>(dKVp, dK, dV, ns, n4, nb_kv, dQp, dQ, p.key_len, p.H, p.Lq, p.Lk, p.causal, p.scale, BH, kr); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_bwd_dq_reduce_f32(const AttnProblem &p, const float *dQp, float *dQ,
                                    hipStream_t s) {
    const int BH = p.B * p.H;
    const size_t total = (size_t)BH * p.Lq * (p.d / 4);
    const dim3 grid((unsigned)((total + 255) / 256)), block(256);
    const int kr = fused_dq_key_rows(p);
    switch (p.d) {
    case 32: attn_dq_reduce_f32<32><<<grid, block, 0, s>>>(dQp, dQ, p.key_len, p.H, p.Lq, p.Lk, p.causal, p.scale, BH, kr); break;
    case 64: attn_dq_reduce_f32<64><<<grid, block, 0, s>>>(dQp, dQ, p.key_len, p.H, p.Lq, p.Lk, p.causal, p.scale, BH, kr); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

}  // namespace mg
