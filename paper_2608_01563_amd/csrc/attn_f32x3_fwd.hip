// attn_f32x3_fwd.hip -- strict-f32 attention forward on the bf16 matrix cores.
//
// Both products take f32 operands as three bf16 parts (tiles_split.h), which
// keeps the f32 result and needs 96 instead of 256 matrix clocks per 16x16x32
// block.  K and V tiles of KT keys are split once as they are staged into LDS,
// P straight from the accumulators; every product runs on 16x16x32.
//
// The waves of a workgroup form a QW x KG grid over a tile: QW groups of
// QB 16-query blocks, KG groups of KT/KG keys.  With KG = 1 a workgroup takes
// the most queries, so a split tile serves all eight waves.  Smaller grids take
// fewer queries per workgroup and spread a tile's keys over the waves instead;
// the key groups keep online-softmax states of their own, which the first
// group merges through LDS at the end.
#include <type_traits>

#include "device_common.h"
#include "fwd_forms.h"
#include "launch.h"
#include "rows_f32.h"
#include "tiles_split.h"
#include "work_order.h"

namespace mg {
namespace {

// Rows whose fast result is not finite, in plain f32 (rows_f32.h): 16 rows from
// row0 at a time.  Ends early where every row's sum is NaN, which then is all
// its O.
template <int D>
__device__ __forceinline__ void fwd_rows_plain(const float *Q, const float *K, const float *V, float *O,
                                            float *LSE, int row0, int nrows, int Lq, int klen,
                                            int causal, int diag, float scale_log2, int lane) {
    constexpr int NC = D / 16;
    hide(lane, klen);
    const int il = lane & 15, g = lane >> 4;
    for (int i0 = row0; i0 < min(row0 + nrows, Lq); i0 += 16) {
        const int i = i0 + il;
        const bool row = i < Lq;
        f32x4 q[NC], o[NC];
        load_row16<D>(q, Q + (size_t)i * D, row, g);
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            q[c] *= scale_log2;
            o[c] = zero4();
        }
        const int sees = causal ? min(klen, i + diag + 1) : klen;          // keys of this row
        const int all = causal ? min(klen, i0 + diag + 1) : klen;          // ... of every row
        const int some = causal ? min(klen, min(i0 + 16, Lq) + diag) : klen;   // ... of any row
        float m = -INFINITY, l = 0.f;
        for (int j0 = 0; j0 < some; j0 += 16) {
            f32x4 p = dot16<D>(K + (size_t)j0 * D, klen - j0, q, il, g);
            float mx = m;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                if (j0 + 4 * g + r >= sees) p[r] = -INFINITY;
                mx = fmaxf(mx, p[r]);
            }
            mx = max_over_groups(mx);
            const float mu = (mx == -INFINITY) ? 0.f : mx;
            const float alpha = exp2_fast(m - mu);
            m = mx;
            l *= alpha;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                p[r] = exp2_fast(p[r] - mu);
                l += p[r];
            }
#pragma unroll
            for (int c = 0; c < NC; ++c) o[c] *= alpha;
            if (j0 + 16 <= all)
                add16<D>(o, V + (size_t)j0 * D, 16, p, il, g);
            else
                add16_visible<D>(o, V + (size_t)j0 * D, klen - j0, p, il, g,
                                 [&](int x) { return j0 + x < sees; });
            const float lt = sum_over_groups(l);
            if (__all(!row || lt != lt)) break;
        }
        l = sum_over_groups(l);
        const float inv = (l > 0.f) ? 1.f / l : 0.f;
        if (row) {
#pragma unroll
            for (int c = 0; c < NC; ++c)
                *reinterpret_cast<f32x4 *>(O + (size_t)i * D + 16 * c + 4 * g) = o[c] * inv;
            if (g == 0) LSE[i] = row_lse(m, l);
        }
    }
}

template <int D, int QB, int QW, int KG, int KT, bool DB, int OCC>
__global__ __launch_bounds__(64 * QW * KG) __attribute__((amdgpu_waves_per_eu(OCC, 8)))
void attn_fwd_f32x3(const float *__restrict__ Q, const float *__restrict__ K,
                    const float *__restrict__ V, float *__restrict__ O, float *__restrict__ LSE,
                    const int32_t *__restrict__ key_len, int H, int Lq, int Lk, int causal,
                    float scale_log2, int n_qtiles, int BH, int layer, int padded_order) {
    constexpr int NT = 64 * QW * KG;
    constexpr int NS = D / 32;            // 32-deep contraction steps over d
    constexpr int NC = D / 16;            // 16-column blocks of d
    constexpr int WQ = 16 * QB;           // queries per wave
    constexpr int WK = KT / KG;           // keys of a tile per wave
    constexpr int NKB = WK / 16;
    static_assert(WK % 32 == 0, "P V contracts 32 keys at a time");
    using Tile = Bf16Tile<KT, D, 1, 32, 1, 3, 1>;
    constexpr int BLK = Tile::kBlock;
    constexpr int NX = QB * (2 + 4 * NC); // a lane's merge state: m, l, O^T
    constexpr int TS = 3 * Tile::kSize;
    constexpr int kTiles = (DB ? 2 : 1) * 2 * TS * 2;
    constexpr int kMerge = (KG - 1) * QW * NX * 64 * 4;
    __shared__ __attribute__((aligned(16))) unsigned char smem[kTiles > kMerge ? kTiles : kMerge];
    uint16_t *const tiles = reinterpret_cast<uint16_t *>(smem);   // K, V (, K, V)

    int slot, head;
    if (padded_order) {
        heavy_first_tile(blockIdx.x, n_qtiles, KT, BH, H, Lk, key_len, slot, head);
    } else {
        slot = blockIdx.x / BH;
        head = blockIdx.x - slot * BH;
    }
    const int rank = serpentine_rank(slot, n_qtiles, layer);
    const int qt = causal ? (n_qtiles - 1 - rank) : rank;
    const float *Qh = Q + (size_t)head * Lq * D;
    const float *Kh = K + (size_t)head * Lk * D;
    const float *Vh = V + (size_t)head * Lk * D;
    float *Oh = O + (size_t)head * Lq * D;
    const int diag = Lk - Lq;   // causal: row i sees keys j <= i + diag

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wq = w % QW, kg = w / QW;
    const int il = lane & 15;
    const int g = lane >> 4;
    const int jr = il >> 2, jc = 4 * (il & 3);   // transpose-read block offsets
    const int q0 = qt * WQ * QW;
    const int qw0 = q0 + WQ * wq;   // first query of this wave
    const int qi = qw0 + il;        // query of block 0; block qb holds qi + 16 qb

    const int klen = key_limit(key_len, head / H, Lk);
    const int kend = causal ? min(klen, q0 + WQ * QW + diag) : klen;
    const int ntiles = max((kend + KT - 1) / KT, 0);

    // Padded keys are staged as zeros (the tiles end at the key length), so
    // whatever their rows hold takes no part.
    SplitStager<Tile, KT, D, NT> sk, sv;
    if (ntiles > 0) {
        sk.load(Kh, 0, klen, tid);
        sv.load(Vh, 0, klen, tid);
    }
    // B operand of S^T = K Q^T: parts of kUp Q[qi + 16qb][32s + 8g + e] * scale*log2(e).
    const float q_scale = scale_log2 * kUp;
    Split8 qreg[NS][QB];
#pragma unroll
    for (int qb = 0; qb < QB; ++qb)
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            f32x4 a = zero4(), b = zero4();
            if (qi + 16 * qb < Lq) {
                const float *qp = Qh + (size_t)(qi + 16 * qb) * D + 32 * s + 8 * g;
                a = *reinterpret_cast<const f32x4 *>(qp) * q_scale;
                b = *reinterpret_cast<const f32x4 *>(qp + 4) * q_scale;
            }
            qreg[s][qb] = split8(a, b);
        }
    // Lane bases of the tile reads, in this wave's keys: K rows 16kb + il,
    // columns 32s + 8g; V^T rows 32t + 4g + jr (+16), columns 16c + jc.
    const int k0w = WK * kg;
    const int ka = Tile::at(il, 8 * g) + 32 * k0w;
    const int va[2] = {Tile::at(4 * g + jr, jc) + 32 * k0w, Tile::at(4 * g + jr, 16 + jc) + 32 * k0w};

    // P stays unscaled: at most 2^kSlack, it loses no bits that reach O.
    float m_run[QB], l_run[QB];   // base-2 units
    f32x4 oacc[NC][QB];           // kUp O^T[16c + 4g + r][qi + 16qb]
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) {
        m_run[qb] = -INFINITY;
        l_run[qb] = 0.f;
#pragma unroll
        for (int c = 0; c < NC; ++c) oacc[c][qb] = zero4();
    }

    if (ntiles > 0) {
        sk.store(tiles, tid);
        sv.store(tiles + TS, tid);
        if (ntiles > 1) {
            sk.load(Kh, KT, klen, tid);
            if (DB) sv.load(Vh, KT, klen, tid);
        }
    }
    __syncthreads();

    for (int kt = 0; kt < ntiles; ++kt) {
        const int jw = kt * KT + k0w;   // first key of this wave's share
        uint16_t *const Kr = tiles + ((DB && (kt & 1)) ? 2 * TS : 0);
        uint16_t *const Vr = Kr + TS;
        if (DB && kt + 1 < ntiles) {   // tile kt + 1 goes to the buffers the last barrier freed
            uint16_t *const Kn = tiles + ((kt & 1) ? 0 : 2 * TS);
            sk.store(Kn, tid);
            sv.store(Kn + TS, tid);
            if (kt + 2 < ntiles) {
                sk.load(Kh, (kt + 2) * KT, klen, tid);
                sv.load(Vh, (kt + 2) * KT, klen, tid);
            }
        }
        // some key of the share is allowed for some query of the wave
        const bool live = qw0 < Lq && jw < klen && (!causal || jw <= qw0 + WQ - 1 + diag);
        f32x4 sacc[NKB][QB];   // kUp^2 S^T[16kb + 4g + r][qi + 16qb]
        if (live) {
#pragma unroll
            for (int kb = 0; kb < NKB; ++kb)
#pragma unroll
                for (int qb = 0; qb < QB; ++qb) sacc[kb][qb] = zero4();
#pragma unroll
            for (int s = 0; s < NS; ++s)
#pragma unroll
                for (int kb = 0; kb < NKB; ++kb)
                    mfma_split(load_split<Tile>(Kr, ka + s * BLK + 32 * 16 * kb), qreg[s], sacc[kb]);
        }
        if (!DB) __syncthreads();   // every wave is done with K(kt); V(kt) is visible
        if (!DB && kt + 1 < ntiles) {
            sk.store(Kr, tid);                         // K(kt+1), loaded during S(kt)
            sv.load(Vh, (kt + 1) * KT, klen, tid);     // V(kt+1), lands during P V(kt)
        }
        if (live) {
            // Masking only where the share crosses the diagonal or the key length.
            if (jw + WK > klen || (causal && jw + WK - 1 > qw0 + diag)) {
                const int j0 = jw + 4 * g;
#pragma unroll
                for (int qb = 0; qb < QB; ++qb) {
                    const int thr =
                        causal ? min(klen - j0, qi + 16 * qb + diag - j0 + 1) : klen - j0;
#pragma unroll
                    for (int kb = 0; kb < NKB; ++kb)
#pragma unroll
                        for (int r = 0; r < 4; ++r)
                            if (16 * kb + r >= thr) sacc[kb][qb][r] = -INFINITY;
                }
            }
            float mx[QB];
            bool grew = false;
#pragma unroll
            for (int qb = 0; qb < QB; ++qb) {
                mx[qb] = max3_f32(sacc[0][qb][0], sacc[0][qb][1], sacc[0][qb][2]);
                mx[qb] = max3_f32(mx[qb], sacc[0][qb][3], sacc[1][qb][0]);
#pragma unroll
                for (int x = 5; x + 1 < 4 * NKB; x += 2)
                    mx[qb] = max3_f32(mx[qb], sacc[x >> 2][qb][x & 3],
                                      sacc[(x + 1) >> 2][qb][(x + 1) & 3]);
                mx[qb] = max3_f32(mx[qb], sacc[NKB - 1][qb][3], sacc[NKB - 1][qb][3]);
                mx[qb] = max_over_groups(mx[qb]) * kDownProduct;
                grew = grew || mx[qb] - m_run[qb] > kSlack;
            }
            // m is only an offset, at most kSlack below the true maximum (see
            // the bf16 forward): O and l are rescaled only when some row's
            // maximum grew by more.
            if (__any(grew)) {
#pragma unroll
                for (int qb = 0; qb < QB; ++qb) {
                    const float m_new = fmaxf(m_run[qb], mx[qb]);
                    const float alpha =
                        exp2_fast(m_run[qb] - ((m_new == -INFINITY) ? 0.f : m_new));
                    l_run[qb] *= alpha;
#pragma unroll
                    for (int c = 0; c < NC; ++c) oacc[c][qb] *= alpha;
                    m_run[qb] = m_new;
                }
            }
#pragma unroll
            for (int qb = 0; qb < QB; ++qb) {
                const float m2 = (m_run[qb] == -INFINITY) ? 0.f : m_run[qb];
                float psum = 0.f;
#pragma unroll
                for (int kb = 0; kb < NKB; ++kb)
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const float p = exp2_fast(fmaf(sacc[kb][qb][r], kDownProduct, -m2));
                        sacc[kb][qb][r] = p;
                        psum += p;
                    }
                l_run[qb] += psum;
            }
            // O^T[16c + .][qi] += sum_j V^T[16c + il'][j] P^T[j][qi], 32 keys per step
#pragma unroll
            for (int t = 0; t < NKB / 2; ++t) {
                Split8 pb[QB];
#pragma unroll
                for (int qb = 0; qb < QB; ++qb) pb[qb] = split8(sacc[2 * t][qb], sacc[2 * t + 1][qb]);
#pragma unroll
                for (int c = 0; c < NC; ++c) {
                    const int o = va[c & 1] + (c >> 1) * BLK + 32 * 32 * t;
                    mfma_split(load_split_tr<Tile>(Vr, o, o + 32 * 16), pb, oacc[c]);
                }
            }
        }
        __syncthreads();   // every wave is done with V(kt); K(kt+1) is visible
        if (!DB && kt + 1 < ntiles) {
            sv.store(Vr, tid);                                           // V(kt+1)
            if (kt + 2 < ntiles) sk.load(Kh, (kt + 2) * KT, klen, tid);  // K(kt+2)
        }
        // V(kt+1) becomes visible at the next iteration's first barrier
    }

    float l[QB];
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) l[qb] = sum_over_groups(l_run[qb]);
    if constexpr (KG > 1) {
        // Groups 1 .. KG-1 leave (m, l, O) in LDS, whose tiles no wave reads
        // any more; group 0 merges the states in group order.
        float *xs = reinterpret_cast<float *>(smem) + lane;
        if (kg > 0) {
            float *x = xs + ((kg - 1) * QW + wq) * NX * 64;
#pragma unroll
            for (int qb = 0; qb < QB; ++qb) {
                *x = m_run[qb]; x += 64;
                *x = l[qb]; x += 64;
#pragma unroll
                for (int c = 0; c < NC; ++c)
#pragma unroll
                    for (int r = 0; r < 4; ++r) { *x = oacc[c][qb][r]; x += 64; }
            }
        }
        __syncthreads();
        if (kg > 0) return;   // no barrier follows
#pragma unroll
        for (int qb = 0; qb < QB; ++qb) {
            const float *x0 = xs + wq * NX * 64 + qb * (2 + 4 * NC) * 64;
            constexpr int GS = QW * NX * 64;   // floats between groups
            float mm = m_run[qb];
#pragma unroll
            for (int gg = 0; gg < KG - 1; ++gg) mm = fmaxf(mm, x0[gg * GS]);
            const float mu = (mm == -INFINITY) ? 0.f : mm;
            const float a0 = exp2_fast(m_run[qb] - mu);
            l[qb] *= a0;
#pragma unroll
            for (int c = 0; c < NC; ++c) oacc[c][qb] *= a0;
#pragma unroll
            for (int gg = 0; gg < KG - 1; ++gg) {
                const float *x = x0 + gg * GS;
                const float a = exp2_fast(x[0] - mu);
                l[qb] += x[64] * a;
#pragma unroll
                for (int c = 0; c < NC; ++c)
#pragma unroll
                    for (int r = 0; r < 4; ++r)
                        oacc[c][qb][r] = fmaf(x[(2 + 4 * c + r) * 64], a, oacc[c][qb][r]);
            }
            m_run[qb] = mm;
        }
    }

    bool fine = true;
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) {
        const int q = qi + 16 * qb;
        if (q < Lq) {
            const float inv = (l[qb] > 0.f) ? kDown / l[qb] : 0.f;
            const float lse = row_lse(m_run[qb], l[qb]);
            // l is 0 where the row sees no key, else only if every score is -inf
            const bool sees = (causal ? min(klen, q + diag + 1) : klen) > 0;
            float chk = sees ? lse : 0.f;
            float *orow = Oh + (size_t)q * D;
#pragma unroll
            for (int c = 0; c < NC; ++c) {
                const f32x4 v = oacc[c][qb] * inv;
                *reinterpret_cast<f32x4 *>(orow + 16 * c + 4 * g) = v;
#pragma unroll
                for (int e = 0; e < 4; ++e) chk = fmaf(v[e], 0.f, chk);   // NaN if not finite
            }
            if (g == 0) LSE[(size_t)head * Lq + q] = lse;
            fine = fine && finite_f32(chk);
        }
    }
    if (!__all(fine))
        fwd_rows_plain<D>(Qh, Kh, Vh, Oh, LSE + (size_t)head * Lq, qw0, WQ, Lq, klen, causal, diag,
                          scale_log2, lane);
}

}  // namespace

// Instances per form.  With one key group a tile is split once for all the
// waves of a workgroup; kRows64 streams 32-key tiles, whose LDS (24 KB at d = 64)
// leaves room for four workgroups per CU.
hipError_t launch_fwd_f32(const AttnProblem &p, const float *Q, const float *K, const float *V,
                          float *O, float *LSE, FwdForm form, hipStream_t s) {
    const int BH = p.B * p.H;
    auto go = [&](auto kern, int rows, int nt) {
        const int nqt = cdiv(p.Lq, rows);
        const dim3 grid(nqt * BH);
        const int ly = causal_rank_layer((const void *)kern, nt, grid.x, BH, p.causal);
        kern<<<grid, dim3(nt), 0, s>>>(Q, K, V, O, LSE, p.key_len, p.H, p.Lq, p.Lk, p.causal,
                                       p.scale * kLog2e, nqt, BH, ly, padded_work_order(p));
        return hipGetLastError();
    };
#define MG_GO(D, QB, QW, KG, KT, DB, OCC) \
    return go(attn_fwd_f32x3<D, QB, QW, KG, KT, DB, OCC>, 16 * QB * QW, 64 * QW * KG)
    if (p.d == 32) switch (form) {
        case FwdForm::kRows32: MG_GO(32, 1, 2, 2, 64, false, 4);
        case FwdForm::kRows32Quad: MG_GO(32, 1, 2, 4, 128, false, 4);
        case FwdForm::kRows64: MG_GO(32, 1, 4, 1, 32, false, 4);
        case FwdForm::kRows64Pair: MG_GO(32, 1, 4, 2, 64, false, 4);
        case FwdForm::kRows128: MG_GO(32, 1, 8, 1, 64, false, 4);
        default: break;
    }
    if (p.d == 64) switch (form) {
        case FwdForm::kRows32: MG_GO(64, 1, 2, 2, 64, false, 3);
        case FwdForm::kRows32Quad: MG_GO(64, 1, 2, 4, 128, false, 2);
        case FwdForm::kRows64: MG_GO(64, 1, 4, 1, 32, false, 4);
        case FwdForm::kRows64Pair: MG_GO(64, 1, 4, 2, 64, false, 4);
        case FwdForm::kRows128: MG_GO(64, 1, 8, 1, 64, false, 4);
        default: break;
    }
    if (p.d == 128) switch (form) {
        case FwdForm::kRows64: MG_GO(128, 1, 4, 1, 32, false, 2);
        case FwdForm::kRows64Pair: MG_GO(128, 1, 4, 2, 64, false, 2);
        case FwdForm::kRows128: MG_GO(128, 1, 8, 1, 32, true, 2);
        case FwdForm::kRows256: MG_GO(128, 2, 8, 1, 32, true, 2);
        default: break;
    }
#undef MG_GO
    return hipErrorInvalidValue;
}

}  // namespace mg
