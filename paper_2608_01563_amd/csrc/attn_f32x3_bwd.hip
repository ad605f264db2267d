// attn_f32x3_bwd.hip -- strict-f32 attention backward on the bf16 matrix
// cores: every product takes its f32 operands as three bf16 parts
// (tiles_split.h).
//
// Two kernels, neither of which needs partial sums in memory: a
// query-stationary dQ kernel, which also computes D_i = sum_k dO_ik O_ik for
// its rows and writes it, and the key-stationary dK/dV kernel that reads D
// after it.  Both recompute S and dP, 14 d instead of the 10 d operations per
// pair of the fused kernel in attn_f32.hip, and drop that kernel's dQ partials
// (written and read back, 151 MB at B8 H8 L1024 d64), their reduction and the
// separate D launch.
//
// Operands are split as 2^24 times their values (tiles_split.h): S and dP come
// out 2^48 times, the factors below bring dS to 2^24 times (its split) and the
// results back.
#include <algorithm>

#include "device_common.h"
#include "launch.h"
#include "rows_f32.h"
#include "tiles_split.h"
#include "work_order.h"

namespace mg {
namespace {

// Rows (dQ) or keys (dK, dV) whose fast result is not finite, in plain f32
// (rows_f32.h): 16 at a time.  Ends early where every value is NaN.
template <int D>
__device__ __forceinline__ void dq_rows_plain(const float *Q, const float *K, const float *V,
                                           const float *dO, const float *LSE, const float *Dw,
                                           float *dQ, int row0, int nrows, int Lq, int klen,
                                           int causal, int diag, float scale, float scale_log2,
                                           int lane) {
    constexpr int NC = D / 16;
    hide(lane, klen);
    const int il = lane & 15, g = lane >> 4;
    for (int i0 = row0; i0 < min(row0 + nrows, Lq); i0 += 16) {
        const int i = i0 + il;
        const bool row = i < Lq;
        f32x4 q[NC], go[NC], acc[NC];
        load_row16<D>(q, Q + (size_t)i * D, row, g);
        load_row16<D>(go, dO + (size_t)i * D, row, g);
#pragma unroll
        for (int c = 0; c < NC; ++c) acc[c] = zero4();
        const float lse2 = row ? LSE[i] * kLog2e : 0.f, Di = row ? Dw[i] : 0.f;
        const int sees = causal ? min(klen, i + diag + 1) : klen;          // keys of this row
        const int all = causal ? min(klen, i0 + diag + 1) : klen;          // ... of every row
        const int some = causal ? min(klen, min(i0 + 16, Lq) + diag) : klen;   // ... of any row
        for (int j0 = 0; j0 < some; j0 += 16) {
            const f32x4 s = dot16<D>(K + (size_t)j0 * D, klen - j0, q, il, g);
            const f32x4 dp = dot16<D>(V + (size_t)j0 * D, klen - j0, go, il, g);
            f32x4 ds;
#pragma unroll
            for (int r = 0; r < 4; ++r) ds[r] = exp2_fast(s[r] * scale_log2 - lse2) * (dp[r] - Di);
            if (j0 + 16 <= all)
                add16<D>(acc, K + (size_t)j0 * D, 16, ds, il, g);
            else
                add16_visible<D>(acc, K + (size_t)j0 * D, klen - j0, ds, il, g,
                                 [&](int x) { return j0 + x < sees; });
            if (__all(!row || all_nan(acc))) break;
        }
        if (row) {
#pragma unroll
            for (int c = 0; c < NC; ++c)
                *reinterpret_cast<f32x4 *>(dQ + (size_t)i * D + 16 * c + 4 * g) = acc[c] * scale;
        }
    }
}

template <int D>
__device__ __forceinline__ void dkdv_keys_plain(const float *Q, const float *K, const float *V,
                                             const float *dO, const float *LSE, const float *Dw,
                                             float *dK, float *dV, int key0, int klen, int Lq,
                                             int causal, int diag, float scale, float scale_log2,
                                             int lane) {
    constexpr int NC = D / 16;
    if constexpr (D < 128) hide(lane, klen);   // d = 128 has no register to spare for it
    const int il = lane & 15, g = lane >> 4;
    const int j = key0 + il;
    const bool key = j < klen;
    f32x4 k[NC], v[NC], ak[NC], av[NC];
    load_row16<D>(k, K + (size_t)j * D, key, g);
    load_row16<D>(v, V + (size_t)j * D, key, g);
#pragma unroll
    for (int c = 0; c < NC; ++c) ak[c] = av[c] = zero4();
    for (int i0 = causal ? max(0, key0 - diag) / 16 * 16 : 0; i0 < Lq; i0 += 16) {
        const f32x4 s = dot16<D>(Q + (size_t)i0 * D, Lq - i0, k, il, g);
        const f32x4 dp = dot16<D>(dO + (size_t)i0 * D, Lq - i0, v, il, g);
        f32x4 p, ds;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int i = i0 + 4 * g + r;
            p[r] = (i < Lq) ? exp2_fast(s[r] * scale_log2 - LSE[i] * kLog2e) : 0.f;
            ds[r] = (i < Lq) ? p[r] * (dp[r] - Dw[i]) : 0.f;
        }
        if (!causal || i0 + diag >= key0 + 15) {
            add16<D>(av, dO + (size_t)i0 * D, Lq - i0, p, il, g);
            add16<D>(ak, Q + (size_t)i0 * D, Lq - i0, ds, il, g);
        } else {
            const auto sees = [&](int x) { return i0 + x + diag >= j; };
            add16_visible<D>(av, dO + (size_t)i0 * D, Lq - i0, p, il, g, sees);
            add16_visible<D>(ak, Q + (size_t)i0 * D, Lq - i0, ds, il, g, sees);
        }
        if (__all(!key || (all_nan(ak) && all_nan(av)))) break;
    }
    if (key) {
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            *reinterpret_cast<f32x4 *>(dK + (size_t)j * D + 16 * c + 4 * g) = ak[c] * scale;
            *reinterpret_cast<f32x4 *>(dV + (size_t)j * D + 16 * c + 4 * g) = av[c];
        }
    }
}

// ------------------------------------------------------------------------ dQ --
// QW waves of 16 QB query rows; key tiles of KT keys, double-buffered.  G = 2: two
// groups of QW waves hold the same rows and take half of every key tile each,
// through one buffer; the second hands its sums over at the end.
template <int D, int QB, int QW, int KT, int G>
__global__ __launch_bounds__(64 * QW * G) __attribute__((amdgpu_waves_per_eu(G == 2 && D <= 64 ? 4 : 2, 8)))
void attn_dq_f32x3(const float *__restrict__ Q, const float *__restrict__ K,
                   const float *__restrict__ V, const float *__restrict__ O,
                   const float *__restrict__ dO, const float *__restrict__ LSE,
                   float *__restrict__ Dws, float *__restrict__ dQ,
                   const int32_t *__restrict__ key_len, int H, int Lq, int Lk, int causal,
                   float scale, float scale_log2, int n_qtiles, int BH, int layer,
                   int padded_order) {
    constexpr int NT = 64 * QW * G;
    constexpr int NS = D / 32, NC = D / 16, NKB = KT / (16 * G), WQ = 16 * QB;
    using Tile = Bf16Tile<KT, D, 1, 32, 1, 3, 1>;
    constexpr int BLK = Tile::kBlock, TS = 3 * Tile::kSize;
    __shared__ __attribute__((aligned(16))) uint16_t smem[(G == 1 ? 4 : 2) * TS];
    uint16_t *const Ks = smem, *const Vs = smem + TS;   // next buffers 2 TS further

    int slot, head;
    if (padded_order) {
        heavy_first_tile(blockIdx.x, n_qtiles, KT, BH, H, Lk, key_len, slot, head);
    } else {
        slot = blockIdx.x / BH;
        head = blockIdx.x - slot * BH;
    }
    const int rank = serpentine_rank(slot, n_qtiles, layer);
    const int qt = causal ? (n_qtiles - 1 - rank) : rank;
    const size_t qoff = (size_t)head * Lq * D, hoff = (size_t)head * Lk * D;
    const float *Qh = Q + qoff, *dOh = dO + qoff, *Kh = K + hoff, *Vh = V + hoff;
    const int diag = Lk - Lq;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wg = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int gr = (G == 1) ? 0 : wg / QW;   // key group: the gr-th part of each tile
    const int w = wg - gr * QW;
    const int il = lane & 15, g = lane >> 4;
    const int jr = il >> 2, jc = 4 * (il & 3);
    const int q0 = qt * WQ * QW, qw0 = q0 + WQ * w, qi = qw0 + il;

    const int klen = key_limit(key_len, head / H, Lk);
    const int kend = causal ? min(klen, q0 + WQ * QW + diag) : klen;
    const int ntiles = max((kend + KT - 1) / KT, 0);

    SplitStager<Tile, KT, D, NT> sk, sv;
    if (ntiles > 0) {
        sk.load(Kh, 0, klen, tid);
        sv.load(Vh, 0, klen, tid);
    }
    // parts of Q and dO [qi + 16qb][32s + 8g + e]; D from dO and O on the way
    Split8 qreg[NS][QB], oreg[NS][QB];
    float lse2[QB], Di[QB];
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) {
        const int q = qi + 16 * qb;
        lse2[qb] = (q < Lq) ? LSE[(size_t)head * Lq + q] * kLog2e : 0.f;
        float dsum = 0.f;
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            f32x4 a = zero4(), b = zero4(), x = zero4(), y = zero4();
            if (q < Lq) {
                const size_t off = qoff + (size_t)q * D + 32 * s + 8 * g;
                a = *reinterpret_cast<const f32x4 *>(Q + off);
                b = *reinterpret_cast<const f32x4 *>(Q + off + 4);
                x = *reinterpret_cast<const f32x4 *>(dO + off);
                y = *reinterpret_cast<const f32x4 *>(dO + off + 4);
                const f32x4 u = *reinterpret_cast<const f32x4 *>(O + off);
                const f32x4 v = *reinterpret_cast<const f32x4 *>(O + off + 4);
#pragma unroll
                for (int e = 0; e < 4; ++e) dsum = fmaf(x[e], u[e], fmaf(y[e], v[e], dsum));
            }
            qreg[s][qb] = split8_up(a, b);
            oreg[s][qb] = split8_up(x, y);
        }
        Di[qb] = sum_over_groups(dsum);
        if (q < Lq && g == 0 && gr == 0) Dws[(size_t)head * Lq + q] = Di[qb];
    }
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) Di[qb] *= kUp;
    const float s_scale = scale_log2 * kDownProduct;
    const int key0 = 16 * NKB * gr;   // this group's keys of a tile
    const int ka = Tile::at(il, 8 * g) + 32 * key0;
    const int kt_[2] = {Tile::at(4 * g + jr, jc) + 32 * key0,
                        Tile::at(4 * g + jr, 16 + jc) + 32 * key0};

    f32x4 dqacc[NC][QB];   // dQ^T[16c + 4g + r][qi + 16qb]
#pragma unroll
    for (int c = 0; c < NC; ++c)
#pragma unroll
        for (int qb = 0; qb < QB; ++qb) dqacc[c][qb] = zero4();

    if (ntiles > 0) {
        sk.store(Ks, tid);
        sv.store(Vs, tid);
        sk.load(Kh, KT, klen, tid);
        sv.load(Vh, KT, klen, tid);
    }
    __syncthreads();
    for (int kt = 0; kt < ntiles; ++kt) {
        const int cur = (G == 1 && (kt & 1)) ? 2 * TS : 0, nxt = 2 * TS - cur;
        if (G == 1 && kt + 1 < ntiles) {   // tile kt + 1 goes to the buffer the last barrier freed
            sk.store(Ks + nxt, tid);
            sv.store(Vs + nxt, tid);
            sk.load(Kh, (kt + 2) * KT, klen, tid);
            sv.load(Vh, (kt + 2) * KT, klen, tid);
        }
        const int jt = kt * KT + key0;
        if (qw0 < Lq && jt < klen && (!causal || jt <= qw0 + WQ - 1 + diag)) {
            const uint16_t *Kc = Ks + cur, *Vc = Vs + cur;
            f32x4 sacc[NKB][QB], pacc[NKB][QB];   // 2^48 S^T, dP^T[16kb + 4g + r][qi + 16qb]
#pragma unroll
            for (int kb = 0; kb < NKB; ++kb)
#pragma unroll
                for (int qb = 0; qb < QB; ++qb) {
                    sacc[kb][qb] = zero4();
                    pacc[kb][qb] = zero4();
                }
#pragma unroll
            for (int s = 0; s < NS; ++s)
#pragma unroll
                for (int kb = 0; kb < NKB; ++kb) {
                    const int o = ka + s * BLK + 32 * 16 * kb;
                    mfma_split(load_split<Tile>(Kc, o), qreg[s], sacc[kb]);
                    mfma_split(load_split<Tile>(Vc, o), oreg[s], pacc[kb]);
                }
            // two products' operand reads in flight (d = 128: 89 -> 82 us at B2 H8 L1024)
            sched_reads_ahead<6 * NS * NKB, 12 * QB * NS * NKB, 6, 3, 6 * QB, 0>();
            // 2^24 dS^T = P^T 2^24 (dP^T - D), P^T = exp2(S^T * scale*log2e - LSE*log2e)
            const bool masked = jt + 16 * NKB > klen || (causal && jt + 16 * NKB - 1 > qw0 + diag);
            const int j0 = jt + 4 * g;
#pragma unroll
            for (int qb = 0; qb < QB; ++qb) {
                const int thr = causal ? min(klen - j0, qi + 16 * qb + diag - j0 + 1) : klen - j0;
#pragma unroll
                for (int kb = 0; kb < NKB; ++kb)
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const float p = exp2_fast(fmaf(sacc[kb][qb][r], s_scale, -lse2[qb]));
                        pacc[kb][qb][r] = p * fmaf(pacc[kb][qb][r], kDown, -Di[qb]);
                    }
                if (masked) {
#pragma unroll
                    for (int kb = 0; kb < NKB; ++kb)
#pragma unroll
                        for (int r = 0; r < 4; ++r)
                            if (16 * kb + r >= thr) pacc[kb][qb][r] = 0.f;
                }
            }
            // dQ^T[16c + .][qi] += sum_j K^T[16c + il'][j] dS^T[j][qi], 32 keys per step
#pragma unroll
            for (int t = 0; t < NKB / 2; ++t) {
                Split8 ds[QB];
#pragma unroll
                for (int qb = 0; qb < QB; ++qb) ds[qb] = split8(pacc[2 * t][qb], pacc[2 * t + 1][qb]);
#pragma unroll
                for (int c = 0; c < NC; ++c) {
                    const int o = kt_[c & 1] + (c >> 1) * BLK + 32 * 32 * t;
                    // a fresh sum per tile, added once: rounds at the size of dQ once
                    // per 32 keys instead of six times (B4 H16 L2048 d64: dQ error
                    // 9.6e-7 -> 6.8e-7, 3 % of the kernel's time)
                    f32x4 part[QB];
#pragma unroll
                    for (int qb = 0; qb < QB; ++qb) part[qb] = zero4();
                    mfma_split(load_split_tr<Tile>(Kc, o, o + 32 * 16), ds, part);
#pragma unroll
                    for (int qb = 0; qb < QB; ++qb) dqacc[c][qb] += part[qb];
                }
            }
            sched_reads_ahead<6 * NC * NKB / 2, 6 * QB * NC * NKB / 2, 6, 6, 6 * QB, 1>();
        }
        __syncthreads();   // tile kt + 1 visible; tile kt's buffers free
        if (G > 1 && kt + 1 < ntiles) {
            sk.store(Ks, tid);
            sv.store(Vs, tid);
            sk.load(Kh, (kt + 2) * KT, klen, tid);
            sv.load(Vh, (kt + 2) * KT, klen, tid);
            __syncthreads();
        }
    }
    if constexpr (G == 2) {
        // the second group's sums reach the first through the tile buffers
        static_assert(sizeof(smem) >= (size_t)QW * NC * QB * 64 * sizeof(f32x4), "sums fit");
        f32x4 *x = reinterpret_cast<f32x4 *>(smem) + w * NC * QB * 64 + lane;
        if (gr == 1) {
#pragma unroll
            for (int c = 0; c < NC; ++c)
#pragma unroll
                for (int qb = 0; qb < QB; ++qb) x[64 * (QB * c + qb)] = dqacc[c][qb];
        }
        __syncthreads();
        if (gr == 1) return;   // no barrier follows
#pragma unroll
        for (int c = 0; c < NC; ++c)
#pragma unroll
            for (int qb = 0; qb < QB; ++qb) dqacc[c][qb] += x[64 * (QB * c + qb)];
    }

    bool fine = true;
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) {
        const int q = qi + 16 * qb;
        if (q < Lq) {
            float chk = 0.f;
            float *row = dQ + qoff + (size_t)q * D;
#pragma unroll
            for (int c = 0; c < NC; ++c) {
                const f32x4 v = dqacc[c][qb] * kDownProduct * scale;
                *reinterpret_cast<f32x4 *>(row + 16 * c + 4 * g) = v;
#pragma unroll
                for (int e = 0; e < 4; ++e) chk = fmaf(v[e], 0.f, chk);   // NaN if not finite
            }
            fine = fine && finite_f32(chk);
        }
    }
    if (!__all(fine)) {
        __threadfence_block();   // this wave's D rows are in memory
        dq_rows_plain<D>(Qh, Kh, Vh, dOh, LSE + (size_t)head * Lq, Dws + (size_t)head * Lq,
                         dQ + qoff, qw0, WQ, Lq, klen, causal, diag, scale, scale_log2, lane);
    }
}

// -------------------------------------------------------------------- dK, dV --
// KW waves of 16 keys; query tiles of QT rows, double-buffered (G = 2: as above,
// half of every query tile per group, through one buffer).
template <int D, int KW, int QT, int G>
__global__ __launch_bounds__(64 * KW * G) __attribute__((amdgpu_waves_per_eu(2, 8)))
void attn_dkdv_f32x3(const float *__restrict__ Q, const float *__restrict__ K,
                     const float *__restrict__ V, const float *__restrict__ dO,
                     const float *__restrict__ LSE, const float *__restrict__ Dws,
                     float *__restrict__ dK, float *__restrict__ dV,
                     const int32_t *__restrict__ key_len, int H, int Lq, int Lk, int causal,
                     float scale, float scale_log2, int n_ktiles, int BH, int layer,
                     int padded_order) {
    constexpr int NT = 64 * KW * G;
    constexpr int NS = D / 32, NC = D / 16, NIB = QT / (16 * G), KR = 16 * KW;
    using Tile = Bf16Tile<QT, D, 1, 32, 1, 3, 1>;
    constexpr int BLK = Tile::kBlock, TS = 3 * Tile::kSize;
    __shared__ __attribute__((aligned(16))) uint16_t smem[(G == 1 ? 4 : 2) * TS];
    uint16_t *const Qs = smem, *const Os = smem + TS;   // next buffers 2 TS further
    __shared__ __attribute__((aligned(16))) float lse2s[2][QT], Ds[2][QT];

    int slot, head;
    if (padded_order) {
        work_first_tile(blockIdx.x, n_ktiles, 1, KR, BH, H, Lk, key_len, slot, head);
    } else {
        slot = blockIdx.x / BH;
        head = blockIdx.x - slot * BH;
    }
    const int kt = serpentine_rank(slot, n_ktiles, layer);   // low key tiles see the most queries
    const size_t qoff = (size_t)head * Lq * D, hoff = (size_t)head * Lk * D;
    const float *Qh = Q + qoff, *dOh = dO + qoff;
    const int diag = Lk - Lq;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wg = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int gr = (G == 1) ? 0 : wg / KW;   // row group: the gr-th part of each tile
    const int w = wg - gr * KW;
    const int il = lane & 15, g = lane >> 4;
    const int jr = il >> 2, jc = 4 * (il & 3);
    const int k0 = kt * KR, wkey0 = k0 + 16 * w, kj = wkey0 + il;

    const int klen = key_limit(key_len, head / H, Lk);
    const int nq = (Lq + QT - 1) / QT;
    const int qstart = causal ? min(nq, max(0, k0 - diag) / QT) : 0;
    const int qstop = (k0 < klen) ? nq : qstart;

    SplitStager<Tile, QT, D, NT> sq, so;
    float lse_pre = 0.f, d_pre = 0.f;
    auto load = [&](int qt) {
        sq.load(Qh, qt * QT, Lq, tid);
        so.load(dOh, qt * QT, Lq, tid);
        if (tid < QT) {
            const int row = qt * QT + tid;
            lse_pre = (row < Lq) ? LSE[(size_t)head * Lq + row] : 0.f;
            d_pre = (row < Lq) ? Dws[(size_t)head * Lq + row] : 0.f;
        }
    };
    auto store = [&](int buf) {
        sq.store(Qs + buf * 2 * TS, tid);
        so.store(Os + buf * 2 * TS, tid);
        if (tid < QT) {
            lse2s[buf][tid] = lse_pre * kLog2e;
            Ds[buf][tid] = d_pre * kUp;
        }
    };
    if (qstart < qstop) load(qstart);

    // B operands of S = Q K^T and dP = dO V^T: parts of K, V[kj][32s + 8g + e]
    Split8 kreg[NS][1], vreg[NS][1];
#pragma unroll
    for (int s = 0; s < NS; ++s) {
        f32x4 a = zero4(), b = zero4(), x = zero4(), y = zero4();
        if (kj < klen) {
            const size_t off = hoff + (size_t)kj * D + 32 * s + 8 * g;
            a = *reinterpret_cast<const f32x4 *>(K + off);
            b = *reinterpret_cast<const f32x4 *>(K + off + 4);
            x = *reinterpret_cast<const f32x4 *>(V + off);
            y = *reinterpret_cast<const f32x4 *>(V + off + 4);
        }
        kreg[s][0] = split8_up(a, b);
        vreg[s][0] = split8_up(x, y);
    }
    const float s_scale = scale_log2 * kDownProduct;
    const int row0 = 16 * NIB * gr;   // this group's rows of a tile
    const int qa = Tile::at(il, 8 * g) + 32 * row0;
    const int qb_[2] = {Tile::at(4 * g + jr, jc) + 32 * row0,
                        Tile::at(4 * g + jr, 16 + jc) + 32 * row0};

    f32x4 dkacc[NC][1], dvacc[NC][1];   // dK^T, dV^T[16c + 4g + r][kj]
#pragma unroll
    for (int c = 0; c < NC; ++c) {
        dkacc[c][0] = zero4();
        dvacc[c][0] = zero4();
    }
    if (qstart < qstop) {
        store(0);
        if (qstart + 1 < qstop) load(qstart + 1);
    }
    __syncthreads();
    for (int qt = qstart; qt < qstop; ++qt) {
        const int cur = (G == 1) ? (qt - qstart) & 1 : 0;
        if (G == 1 && qt + 1 < qstop) {
            store(cur ^ 1);
            if (qt + 2 < qstop) load(qt + 2);
        }
        const int rt = qt * QT + row0;
        if (wkey0 < klen && (!causal || wkey0 - diag <= rt + 16 * NIB - 1)) {
            const uint16_t *Qc = Qs + cur * 2 * TS, *Oc = Os + cur * 2 * TS;
            f32x4 sacc[NIB][1], pacc[NIB][1];   // 2^48 S, dP[16ib + 4g + r][kj]
#pragma unroll
            for (int ib = 0; ib < NIB; ++ib) {
                sacc[ib][0] = zero4();
                pacc[ib][0] = zero4();
            }
#pragma unroll
            for (int s = 0; s < NS; ++s)
#pragma unroll
                for (int ib = 0; ib < NIB; ++ib) {
                    const int o = qa + s * BLK + 32 * 16 * ib;
                    mfma_split(load_split<Tile>(Qc, o), kreg[s], sacc[ib]);
                    mfma_split(load_split<Tile>(Oc, o), vreg[s], pacc[ib]);
                }
            if constexpr (D == 128) sched_reads_ahead<6 * NS * NIB, 12 * NS * NIB, 6, 3, 6, 2>();
            const bool masked = causal && rt + diag < wkey0 + 15;
            const int thr = kj - diag - (rt + 4 * g);
#pragma unroll
            for (int ib = 0; ib < NIB; ++ib) {
                const f32x4 l2 = *reinterpret_cast<const f32x4 *>(&lse2s[cur][row0 + 16 * ib + 4 * g]);
                const f32x4 dd = *reinterpret_cast<const f32x4 *>(&Ds[cur][row0 + 16 * ib + 4 * g]);
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    float p = exp2_fast(fmaf(sacc[ib][0][r], s_scale, -l2[r]));
                    if (masked && 16 * ib + r < thr) p = 0.f;
                    sacc[ib][0][r] = p * kUp;
                    pacc[ib][0][r] = p * fmaf(pacc[ib][0][r], kDown, -dd[r]);
                }
            }
            // dV^T[16c + .][kj] += dO^T[16c + il'][i] P[i][kj]; dK^T likewise with Q, dS
#pragma unroll
            for (int t = 0; t < NIB / 2; ++t) {
                const Split8 pb[1] = {split8(sacc[2 * t][0], sacc[2 * t + 1][0])};
                const Split8 sb[1] = {split8(pacc[2 * t][0], pacc[2 * t + 1][0])};
#pragma unroll
                for (int c = 0; c < NC; ++c) {
                    const int o = qb_[c & 1] + (c >> 1) * BLK + 32 * 32 * t;
                    mfma_split(load_split_tr<Tile>(Oc, o, o + 32 * 16), pb, dvacc[c]);
                    mfma_split(load_split_tr<Tile>(Qc, o, o + 32 * 16), sb, dkacc[c]);
                }
            }
            if constexpr (D == 128) sched_reads_ahead<12 * NC * NIB / 2, 12 * NC * NIB / 2, 6, 6, 6, 3>();
        }
        __syncthreads();   // next tile visible; this tile's buffers free
        if (G > 1 && qt + 1 < qstop) {
            store(0);
            if (qt + 2 < qstop) load(qt + 2);
            __syncthreads();
        }
    }
    if constexpr (G == 2) {
        // the second group's sums reach the first through the tile buffers
        static_assert(sizeof(smem) >= (size_t)KW * 2 * NC * 64 * sizeof(f32x4), "sums fit");
        f32x4 *x = reinterpret_cast<f32x4 *>(smem) + w * 2 * NC * 64 + lane;
        if (gr == 1) {
#pragma unroll
            for (int c = 0; c < NC; ++c) {
                x[64 * 2 * c] = dkacc[c][0];
                x[64 * (2 * c + 1)] = dvacc[c][0];
            }
        }
        __syncthreads();
        if (gr == 1) return;   // no barrier follows
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            dkacc[c][0] += x[64 * 2 * c];
            dvacc[c][0] += x[64 * (2 * c + 1)];
        }
    }

    bool fine = true;
    if (kj < Lk) {
        const bool keep = kj < klen;   // padded keys get exact zeros
        float *dkrow = dK + hoff + (size_t)kj * D, *dvrow = dV + hoff + (size_t)kj * D;
        float chk = 0.f;
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            const f32x4 a = keep ? dkacc[c][0] * kDownProduct * scale : zero4();
            const f32x4 b = keep ? dvacc[c][0] * kDownProduct : zero4();
            *reinterpret_cast<f32x4 *>(dkrow + 16 * c + 4 * g) = a;
            *reinterpret_cast<f32x4 *>(dvrow + 16 * c + 4 * g) = b;
#pragma unroll
            for (int e = 0; e < 4; ++e) chk = fmaf(a[e], 0.f, fmaf(b[e], 0.f, chk));
        }
        fine = finite_f32(chk);
    }
    if (!__all(fine))
        dkdv_keys_plain<D>(Qh, K + hoff, V + hoff, dOh, LSE + (size_t)head * Lq,
                           Dws + (size_t)head * Lq, dK + hoff, dV + hoff, wkey0, klen, Lq,
                           causal, diag, scale, scale_log2, lane);
}

}  // namespace

// Forms.  kWide: four waves of 32 query rows or 16 keys.  kPair: eight waves in
// two groups that share a 64-row tile and take half of each streamed 64-row
// tile, for grids that leave the time to the chain of tiles.  kEight (d = 128):
// eight waves that share a tile's split.
//
// d <= 64, where the alternative is the fused f32 kernel, which splits the query
// tiles of a key tile over workgroups: the whole backward of both over 1,616
// problems (GPU us, fused : this).  A tile counts only where a head fills 60 %
// of it; one tile a head (64 rows and keys) stays fused, which is the whole
// backward in one launch (but d = 32 causal, many heads: B1 H768 L32 17.3 : 15.0).
//   kWide from one 128-row query tile per CU and a third more key tiles (causal
//     grids, whose tiles differ in length, and d = 32, whose workgroups are
//     shorter, from more; two tiles a head from fewer): d = 64 B1 H192 L80 28 : 27,
//     B8 H32 L128 42 : 38, B8 H16 L256 64 : 56, B8 H8 L1024 causal 207 : 173, B4 H16
//     L2048 1489 : 1100; not B1 H128 L80 21 : 24.  With two rounds of both and
//     more than 64 rows also where tiles are less filled (B1 H622 Lq629 Lk9 171 :
//     149; but B1 H539 Lq8 Lk119 35 : 45).
//   kPair from 192 64-row tiles of both sides while the chains are short, or 448:
//     B8 H12 L128 31 : 25, B8 H8 L256 49 : 37, B8 H4 L512 73 : 58, B4 H16 L512
//     causal 75 : 66, B3 H6 Lq814 Lk1850 221 : 192; not B2 H6 L1500 (288 tiles) 186
//     : 224, B1 H4 L2500 179 : 209, B2 H6 L1200 causal 86 : 105, B1 H101 Lq149
//     Lk1910 causal d32 106 : 133.
// (Before, a tile counted whole: B1 H371 Lq25 Lk116 25 : 37, B1 H557 L20 24 : 31.)
// d = 128, against separate f32 kernels: pair up to 128 128-row tiles (B2 H8
// L1024 causal 354 -> 157, four-wave workgroups 198), then eight (B4 H8 L1024
// 270, pair 316; B4 H16 L2048 3907 -> 2006).
SplitBwdForm split_bwd_form(const AttnProblem &p) {
    const long BH = (long)p.B * p.H;
    const bool causal = p.causal != 0;
    if (p.d == 128)
        return std::max(cdiv(p.Lq, 128), cdiv(p.Lk, 128)) * BH > 128 ? SplitBwdForm::kEight
                                                                     : SplitBwdForm::kPair;
    if (p.Lq <= 64 && p.Lk <= 64)
        return p.d == 32 && causal && BH >= 512 ? SplitBwdForm::kWide : SplitBwdForm::kNone;
    const long q128 = cdiv(p.Lq, 128) * BH, q64 = cdiv(p.Lq, 64) * BH, k64 = cdiv(p.Lk, 64) * BH;
    if (p.Lq > 64 && q128 >= 512 && k64 >= 512) return SplitBwdForm::kWide;
    // 60 % of the 64-row tiles of either side filled
    if (5L * p.Lq < 3L * 64 * cdiv(p.Lq, 64) || 5L * p.Lk < 3L * 64 * cdiv(p.Lk, 64))
        return SplitBwdForm::kNone;
    const bool brief = p.Lq <= 96 && p.Lk <= 96;
    const long wide = brief        ? (causal ? 512 : p.d == 32 ? 256 : 192)
                      : p.d == 32 ? 512 : (causal ? 384 : 256);
    if (q128 >= wide && 3 * k64 >= 4 * wide) return SplitBwdForm::kWide;
    if (!brief && q64 >= 192 && k64 >= 192 && (k64 >= 448 || p.Lq <= 512) &&
        (q64 >= 448 || p.Lk <= 512))
        return SplitBwdForm::kPair;
    return SplitBwdForm::kNone;
}

hipError_t launch_bwd_dq_f32x3(const AttnProblem &p, const float *Q, const float *K,
                               const float *V, const float *O, const float *dO, const float *LSE,
                               float *Dws, float *dQ, hipStream_t s) {
    const int BH = p.B * p.H;
    auto go = [&](auto kern, int rows, int nt) {
        const int nqt = cdiv(p.Lq, rows);
        const dim3 grid(nqt * BH);
        const int ly = causal_rank_layer((const void *)kern, nt, grid.x, BH, p.causal);
        kern<<<grid, dim3(nt), 0, s>>>(Q, K, V, O, dO, LSE, Dws, dQ, p.key_len, p.H, p.Lq, p.Lk,
                                       p.causal, p.scale, p.scale * kLog2e, nqt, BH, ly,
                                       padded_work_order(p));
        return hipGetLastError();
    };
    // (none: the caller has no room for the fused kernel's partials)
    const bool pair = split_bwd_form(p) == SplitBwdForm::kPair;
    switch (p.d) {
    case 32:
        return pair ? go(attn_dq_f32x3<32, 1, 4, 64, 2>, 64, 512)
                    : go(attn_dq_f32x3<32, 2, 4, 32, 1>, 128, 256);
    case 64:
        return pair ? go(attn_dq_f32x3<64, 1, 4, 64, 2>, 64, 512)
                    : go(attn_dq_f32x3<64, 2, 4, 32, 1>, 128, 256);
    case 128:
        return pair ? go(attn_dq_f32x3<128, 1, 4, 64, 2>, 64, 512)
                    : go(attn_dq_f32x3<128, 1, 8, 32, 1>, 128, 512);
    default: return hipErrorInvalidValue;
    }
}

hipError_t launch_bwd_dkdv_f32x3(const AttnProblem &p, const float *Q, const float *K,
                                 const float *V, const float *dO, const float *LSE,
                                 const float *Dws, float *dK, float *dV, hipStream_t s) {
    const int BH = p.B * p.H;
    auto go = [&](auto kern, int rows, int nt) {
        const int nkt = cdiv(p.Lk, rows);
        const dim3 grid(nkt * BH);
        const int ly = causal_rank_layer((const void *)kern, nt, grid.x, BH, p.causal);
        kern<<<grid, dim3(nt), 0, s>>>(Q, K, V, dO, LSE, Dws, dK, dV, p.key_len, p.H, p.Lq, p.Lk,
                                       p.causal, p.scale, p.scale * kLog2e, nkt, BH, ly,
                                       padded_work_order(p));
        return hipGetLastError();
    };
    const bool pair = split_bwd_form(p) == SplitBwdForm::kPair;
    switch (p.d) {
    case 32:
        return pair ? go(attn_dkdv_f32x3<32, 4, 64, 2>, 64, 512)
                    : go(attn_dkdv_f32x3<32, 4, 32, 1>, 64, 256);
    case 64:
        return pair ? go(attn_dkdv_f32x3<64, 4, 64, 2>, 64, 512)
                    : go(attn_dkdv_f32x3<64, 4, 32, 1>, 64, 256);
    case 128:
        return pair ? go(attn_dkdv_f32x3<128, 4, 64, 2>, 64, 512)
                    : go(attn_dkdv_f32x3<128, 8, 32, 1>, 128, 512);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace mg
