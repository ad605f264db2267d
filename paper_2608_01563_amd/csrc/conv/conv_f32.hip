// conv_f32.hip -- data and filter gradients of a 2-D convolution as
// implicit GEMMs, their f32 operands split into three bf16 parts
// (tiles_split.h) for v_mfma_f32_16x16x32_bf16.
//
// Neither derivative materialises an unfolded (im2col) matrix: each
// workgroup gathers the operand rows it needs straight from the
// channels-last tensors while it stages them into LDS.
//
//   filter gradient  dW[k][j]  = sum_m dY[m][k] * Xg[m][j]
//       k = output channel, j = (r, s, c) flattened (the [K][R][S][C] order of
//       dW), m = (n, p, q) flattened, Xg[m][j] = X[n][p*sh-ph+r][q*sw-pw+s][c]
//   data gradient    dX[m][c]  = sum_j dYg[m][j] * W[j][c]
//       per stride-parity class of pixels (see DgradJob): m = (n, i, j) of
//       the class, j = (tr, ts, k) over the class's filter taps with k
//       fastest, W[j][c] = W[k][r][s][c], dYg[m][j] = dY at the output
//       position the tap reads, 0 outside dY.
//
// Both run 64x64 output tiles on 512 threads: each of the eight waves owns a
// 32x16 part as two blocks of 16x16 accumulators, and the reduction advances
// BK (32) at a time through double-buffered LDS tiles (one barrier per step;
// the global loads of steps t+1 and t+2 are in flight, in two register sets,
// during the products of step t; more sets gained nothing).  A step of the
// small grids is a chain of staging, barrier, LDS reads and products with one
// workgroup per CU, so eight waves with a quarter of the f32 form's work per
// step each beat four (N4 14x14 1024 -> 256 1x1, data gradient: f32 matrix
// cores 13.1 us, split 11.7 with four waves, 9.9 with eight; N32 28x28
// 512 3x3: 1113, 973, 895 us, both derivatives 2562 -> 2000).  Operands reach LDS
// through raw buffer loads whose offset is pushed past the end of the buffer
// for a padded or out-of-range element, which reads as zero: the padding of
// the convolution and the tails of every dimension become zeros without a
// branch.  Every output element is one fixed-order sum (within a workgroup,
// then across splits in a fixed order): no atomics.
#include <algorithm>
#include <vector>

#include "../cdiv.h"
#include "../device_common.h"
#include "../rows_f32.h"
#include "../tiles_split.h"
#include "conv_launch.h"

namespace mg {
namespace {

constexpr int BM = 64, BN = 64; // output tile of a workgroup
constexpr int BK = 32;          // reduction step
constexpr int NP = 2;           // register sets: steps of loads in flight
constexpr int NT = 512;         // eight waves, each a 32 x 16 part of the tile
constexpr int kOOB = 0x7ffffff0;   // byte offset past every buffer: reads as zero

__device__ __forceinline__ int fdiv(int n, FastDiv f) {
    return (int)((__umulhi((unsigned)n, f.mul) + (unsigned)n) >> f.shift);
}

// Divisors the kernels use in their per-step index arithmetic.
struct ConvDivs {
    FastDiv PQ, Q, K, S, C;
};

__device__ __forceinline__ float buffer_load_f32(__amdgpu_buffer_rsrc_t r, int byte_offset) {
    return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, byte_offset, 0, 0));
}

// VEC = 4: one 16-byte chunk per thread and step; VEC = 1: four floats,
// 16 apart (used when the contiguous dimension is not a multiple of 4).
template <int VEC>
__device__ __forceinline__ f32x4 load_vec(__amdgpu_buffer_rsrc_t r, const int (&off)[4]) {
    if (VEC == 4) return buffer_load_f32x4(r, off[0]);
    f32x4 v;
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] = buffer_load_f32(r, off[e]);
    return v;
}

// Staged B columns of one thread: with 16-byte chunks (VB == 4), one chunk at
// columns 4*col; with 4-byte loads (VB == 1), four floats at columns
// col + 16e.
template <int VB>
struct BCols {
    static constexpr int NE = VB == 4 ? 1 : 4;   // separately addressed elements
    __device__ static int col(int c, int e) { return VB == 4 ? 4 * c : c + 16 * e; }
};

// LDS tiles: three bf16 planes each.  RedTile is reduction-major ([32
// reduction rows][64 columns]) and read by 4-row transpose reads, so a lane
// group g holds reduction rows 4g..4g+3 and 16+4g..+3; PixTile is the data
// gradient's pixel-major A ([64 pixels][32]), whose reduction columns are
// stored in that order (column 16u + 4g + x at 8g + 4u + x) for 16-byte reads.
using RedTile = Bf16Tile<BK, BN, 1, 32, 1, 3, 1>;
using PixTile = Bf16Tile<BM, BK, 1, 32, 1, 3, 1>;
static_assert(RedTile::kSize == PixTile::kSize, "one plane size");
constexpr int kTile = 3 * RedTile::kSize;
struct ConvLds {
    uint16_t A[2][kTile], B[2][kTile];   // double-buffered operands
};

// kUp times four f32 into the three planes at u16 offset o (8-byte stores), or
// at four separate offsets.
__device__ __forceinline__ void store_split4(uint16_t *t, int o, f32x4 v) {
    const float x[4] = {v[0] * kUp, v[1] * kUp, v[2] * kUp, v[3] * kUp};
    uint32_t p[3][2];
    split_pairs<2>(x, p);
#pragma unroll
    for (int k = 0; k < 3; ++k)
        *reinterpret_cast<uint64_t *>(t + k * RedTile::kSize + o) =
            (uint64_t)p[k][0] | ((uint64_t)p[k][1] << 32);
}
__device__ __forceinline__ void store_split4(uint16_t *t, const int (&o)[4], f32x4 v) {
    const float x[4] = {v[0] * kUp, v[1] * kUp, v[2] * kUp, v[3] * kUp};
    uint32_t p[3][2];
    split_pairs<2>(x, p);
#pragma unroll
    for (int k = 0; k < 3; ++k)
#pragma unroll
        for (int e = 0; e < 4; ++e)
            t[k * RedTile::kSize + o[e]] = (uint16_t)(p[k][e >> 1] >> (16 * (e & 1)));
}

// Work of one filter-gradient launch: grid (k tile, j tile, split), split fastest.
struct WgradJob {
    const float *X, *dY;
    float *out;        // dW (one split) or the partials [split][K][R*S*C]
    int tiles_j, nsplit, nsteps, blocks;
};
// Data-gradient work of one stride-parity class.  With strides (sh, sw) the
// input pixels split into sh*sw classes h = a + sh*i, w = b + sw*j, and the
// only filter taps that reach a pixel of class (a, b) are r = r0 + sh*tr,
// s = s0 + sw*ts with r0 = (a + ph) mod sh, s0 = (b + pw) mod sw; such a tap
// reads output position p = i + da - tr, q = j + db - ts.  Each class is a
// dense GEMM over (n, i, j) x c summing only its (tr, ts, k): no tap that
// skips the pixel is ever multiplied (stride 1 is one class with every tap).
// Grid of a class: (m tile, c tile, split), split fastest.
struct DgradJob {
    const float *dY, *Wt;
    float *out;        // dX (one split) or the partials [split][N*H*W][C], dX layout
    int tiles_c, nsplit, blocks;
    int a, b, Hc, Wc, r0, s0, Rc, Sc, da, db;
    FastDiv HWc, Wc_, Sc_;
};
constexpr int kMaxClasses = 16;   // strides up to 4 x 4 in one launch
struct DgradJobs {
    DgradJob c[kMaxClasses];
    int n;
};

// Outputs whose split sum is not finite: the same terms in plain f32, padding
// left out.  Four or eight outputs of a lane that share one operand of every
// term advance together, kPlain terms' loads in flight; a wave ends where every
// sum it still wants is NaN.  One output at a time, one term in flight, NaN inputs
// took N4 14x14 256 -> 256 3x3 from 38 us to 1350, a NaN in W to 640; so 145 and 98 us.
constexpr int kPlain = 2;
template <int N>
__device__ __forceinline__ bool undecided(const float (&sum)[N], unsigned want) {
    bool any = false;
#pragma unroll
    for (int x = 0; x < N; ++x) any = any || ((want >> x & 1) && sum[x] == sum[x]);
    return any;
}

// Outputs k[x], j of the filter gradient over positions [m0, m1); bits of `want`.
__device__ __forceinline__ void wgrad_plain(float (&sum)[8], unsigned want,
                                            __amdgpu_buffer_rsrc_t rdy, __amdgpu_buffer_rsrc_t rx,
                                            const ConvProblem &p, const ConvDivs &dv, int kbase,
                                            int j, int m0, int m1) {
    const int rs = fdiv(j, dv.C), c = j - rs * p.C;
    const int r = fdiv(rs, dv.S), s = rs - r * p.S;
#pragma unroll
    for (int x = 0; x < 8; ++x) sum[x] = 0.f;
#pragma unroll 1
    for (int m = m0; m < m1; m += kPlain) {
        float a[kPlain][8], b[kPlain];
        bool ok[kPlain];
#pragma unroll
        for (int u = 0; u < kPlain; ++u) {
            const int n = fdiv(m + u, dv.PQ), pq = m + u - n * p.P * p.Q;
            const int pp = fdiv(pq, dv.Q), qq = pq - pp * p.Q;
            const int h = pp * p.sh - p.ph + r, w = qq * p.sw - p.pw + s;
            ok[u] = want != 0 && m + u < m1 && (unsigned)h < (unsigned)p.H &&
                    (unsigned)w < (unsigned)p.W;
            b[u] = buffer_load_f32(rx, ok[u] ? 4 * (((n * p.H + h) * p.W + w) * p.C + c) : kOOB);
#pragma unroll
            for (int x = 0; x < 8; ++x) {
                const int k = kbase + 16 * (x >> 2) + (x & 3);
                a[u][x] = buffer_load_f32(rdy, (want >> x & 1) ? 4 * ((m + u) * p.K + k) : kOOB);
            }
        }
#pragma unroll
        for (int u = 0; u < kPlain; ++u)
            if (ok[u]) {
#pragma unroll
                for (int x = 0; x < 8; ++x) sum[x] = fmaf(a[u][x], b[u], sum[x]);
            }
        if (!__any(undecided(sum, want))) break;
    }
}

// ------------------------------------------------------- filter gradient --
// Block `bid` of the job: split `split` of `nsplit` sums the reduction steps
// [st0, st1) of the N*P*Q positions for one 64x64 tile of dW.
template <int VA, int VB>
__device__ __forceinline__ void wgrad_tile(int bid, ConvLds &L, const WgradJob &job,
                                           const ConvProblem &p, const ConvDivs &dv) {
    using BC = BCols<VB>;
    const float *__restrict__ X = job.X;
    const float *__restrict__ dY = job.dY;
    float *__restrict__ out = job.out;
    const int tiles_j = job.tiles_j, nsplit = job.nsplit, nsteps = job.nsteps;

    const int RSC = p.R * p.S * p.C;
    const int PQ = p.P * p.Q;
    const int M = p.N * PQ;
    const int split = bid % nsplit;
    bid /= nsplit;
    const int k0 = (bid / tiles_j) * BM;
    const int j0 = (bid % tiles_j) * BN;
    const int st0 = (int)((long)nsteps * split / nsplit);
    const int st1 = (int)((long)nsteps * (split + 1) / nsplit);

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int il = lane & 15, g = lane >> 4;
    const int wm = w & 1, wn = w >> 1;
    const int lrow = tid >> 4;   // reduction row this thread stages
    const int lcol = tid & 15;

    const auto rdy = buffer_rsrc(dY, M * p.K * 4);
    const auto rx = buffer_rsrc(X, p.N * p.H * p.W * p.C * 4);

    // Columns this thread stages: k for A, j = (r, s, c) for B (fixed for
    // the whole reduction).
    int ka4[4], br[BC::NE], bsx[BC::NE], boff[BC::NE];   // byte offsets (ka4, boff), taps
    bool kok[4], bok[BC::NE];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const int ka = (VA == 4) ? k0 + 4 * lcol : k0 + lcol + 16 * e;
        ka4[e] = 4 * ka;
        kok[e] = ka < p.K;
    }
#pragma unroll
    for (int e = 0; e < BC::NE; ++e) {
        const int j = j0 + BC::col(lcol, e);
        const int rs = fdiv(j, dv.C), c = j - rs * p.C;
        br[e] = fdiv(rs, dv.S);
        bsx[e] = rs - br[e] * p.S;
        boff[e] = 4 * ((br[e] * p.W + bsx[e]) * p.C + c);
        bok[e] = j < RSC;
    }

    // Step st stages reduction row st*BK + lrow.
    using Regs = f32x4[2];   // A (dY), B (X)
    auto load = [&](int st, Regs &rg) {
        const int m = st * BK + lrow;
        const bool mok = m < M;
        const int n = fdiv(m, dv.PQ), pq = m - n * PQ;
        const int pp = fdiv(pq, dv.Q), qq = pq - pp * p.Q;
        const int hb = pp * p.sh - p.ph, wb = qq * p.sw - p.pw;
        const int xbase = ((n * p.H + hb) * p.W + wb) * p.C;
        int oa[4], ob[BC::NE];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            oa[e] = (mok && kok[e]) ? m * (4 * p.K) + ka4[e] : kOOB;
            if (VA == 4) break;
        }
#pragma unroll
        for (int e = 0; e < BC::NE; ++e) {
            const int h = hb + br[e], wi = wb + bsx[e];
            const bool ok = mok && bok[e] && (unsigned)h < (unsigned)p.H &&
                            (unsigned)wi < (unsigned)p.W;
            ob[e] = ok ? xbase * 4 + boff[e] : kOOB;
        }
        rg[0] = load_vec<VA>(rdy, oa);
        if (VB == 4) {
            rg[1] = buffer_load_f32x4(rx, ob[0]);
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e) rg[1][e] = buffer_load_f32(rx, ob[e]);
        }
    };
    auto store = [&](int buf, const Regs &rg) {
        int o[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) o[e] = RedTile::at(lrow, lcol + 16 * e);
        if (VA == 4)
            store_split4(L.A[buf], RedTile::at(lrow, 4 * lcol), rg[0]);
        else
            store_split4(L.A[buf], o, rg[0]);
        if (VB == 4)
            store_split4(L.B[buf], RedTile::at(lrow, 4 * lcol), rg[1]);
        else
            store_split4(L.B[buf], o, rg[1]);
    };

    f32x4 acc[2] = {zero4(), zero4()};

    // Lane bases of the transpose reads: reduction rows 4g + jr (+16), columns
    // 32wm + 16i + jc of A, 16wn + jc of B.
    const int jr = il >> 2, jc = 4 * (il & 3);
    const int ta[2] = {RedTile::at(4 * g + jr, 32 * wm + jc),
                       RedTile::at(4 * g + jr, 32 * wm + 16 + jc)};
    const int tb = RedTile::at(4 * g + jr, 16 * wn + jc);
    // Two register sets keep the loads of the next two steps in flight while
    // the current step, already in LDS, is multiplied.
    Regs rg[NP];
#pragma unroll
    for (int u = 0; u < NP; ++u)
        if (st0 + u < st1) load(st0 + u, rg[u]);
    if (st0 < st1) store(0, rg[0]);
    __syncthreads();
    // step st: `nx` holds step st+1 (in flight), `fr` is free
    auto body = [&](int st, Regs &nx, Regs &fr) {
        const int cur = (st - st0) & 1;
        if (st + NP < st1) load(st + NP, fr);
        const Split8 a[2] = {load_split_tr<RedTile>(L.A[cur], ta[0], ta[0] + 32 * 16),
                             load_split_tr<RedTile>(L.A[cur], ta[1], ta[1] + 32 * 16)};
        mfma_split(a, load_split_tr<RedTile>(L.B[cur], tb, tb + 32 * 16), acc);
        if (st + 1 < st1) store(cur ^ 1, nx);
        __syncthreads();
    };
    for (int st = st0; st < st1; st += NP) {
#pragma unroll
        for (int u = 0; u < NP; ++u)
            if (st + u < st1) body(st + u, rg[(u + 1) % NP], rg[u]);
    }

    float *dst = out + (size_t)split * p.K * RSC;   // split 0 of 1 is dW itself
    float chk = 0.f;
    const int j = j0 + 16 * wn + il;
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int k = k0 + 32 * wm + 16 * i + 4 * g + r;
            if (k < p.K && j < RSC) dst[(size_t)k * RSC + j] = acc[i][r] * kDownProduct;
            chk = fmaf(acc[i][r], 0.f, chk);   // NaN if not finite
        }
    if (!__all(finite_f32(chk))) {
        int gp = g, first = st0;
        hide(gp, first);
        const int kbase = k0 + 32 * wm + 4 * gp;
        unsigned want = 0;
#pragma unroll
        for (int x = 0; x < 8; ++x)
            if (kbase + 16 * (x >> 2) + (x & 3) < p.K && j < RSC && !finite_f32(acc[x >> 2][x & 3]))
                want |= 1u << x;
        float sum[8];
        wgrad_plain(sum, want, rdy, rx, p, dv, kbase, j < RSC ? j : 0, first * BK, min(st1 * BK, M));
#pragma unroll
        for (int x = 0; x < 8; ++x)
            if (want >> x & 1) dst[(size_t)(kbase + 16 * (x >> 2) + (x & 3)) * RSC + j] = sum[x];
    }
}

template <int VA, int VB>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(4, 8)))
void conv_wgrad_f32(WgradJob job, ConvProblem p, ConvDivs dv, int first) {
    __shared__ __attribute__((aligned(16))) ConvLds lds;
    wgrad_tile<VA, VB>(first + blockIdx.x, lds, job, p, dv);
}

// out[i] = sum over splits of part[split][i].  A group of G consecutive lanes
// (G a power of two, up to 64) owns four consecutive elements (one when
// total % 4 != 0): lane t of the group adds splits t, t + G, t + 2G, ... in
// increasing order, then the group combines its G sums by a butterfly over
// lane distances G/2, ..., 1.  The order of every addition is fixed by
// (nsplit, G), so results repeat bit for bit.
struct ReduceJob {
    const float *part;
    float *out;
    int nsplit, total, G, vec, blocks;
};

__device__ __forceinline__ void split_reduce(int block, const ReduceJob &job) {
    const int G = job.G;
    const int gid = (block * 256 + (int)threadIdx.x) / G;   // element group
    const int t = threadIdx.x & (G - 1);
    const int E = job.vec ? 4 : 1;
    const int i = E * gid;
    const bool live = i < job.total;
    f32x4 sum = zero4();
    if (live) {
        for (int k = t; k < job.nsplit; k += G) {
            const float *src = job.part + (size_t)k * job.total + i;
            if (job.vec)
                sum += *reinterpret_cast<const f32x4 *>(src);
            else
                sum[0] += *src;
        }
    }
    for (int d = G >> 1; d > 0; d >>= 1)
#pragma unroll
        for (int e = 0; e < 4; ++e) sum[e] += __shfl_xor(sum[e], d, 64);
    if (live && t == 0) {
        if (job.vec)
            *reinterpret_cast<f32x4 *>(job.out + i) = sum;
        else
            job.out[i] = sum[0];
    }
}

// One or two reductions in one launch (b.blocks == 0 for one).
__global__ __launch_bounds__(256) void conv_split_reduce_f32(ReduceJob a, ReduceJob b) {
    if ((int)blockIdx.x < a.blocks)
        split_reduce(blockIdx.x, a);
    else
        split_reduce(blockIdx.x - a.blocks, b);
}

// Outputs of class pixels m0 .. m0 + 3, channel c of the data gradient over the
// class's reduction columns [j0, j1), tap by tap; bits of `want`.
__device__ __forceinline__ void dgrad_plain(float (&sum)[4], unsigned want, const DgradJob &job,
                                            __amdgpu_buffer_rsrc_t rdy, __amdgpu_buffer_rsrc_t rw,
                                            const ConvProblem &p, const ConvDivs &dv, int m0,
                                            int c, int j0, int j1) {
#pragma unroll
    for (int x = 0; x < 4; ++x) sum[x] = 0.f;
#pragma unroll 1
    for (int x0 = j0; x0 < j1;) {   // columns x0 .. of one tap (tr, ts)
        const int t = fdiv(x0, dv.K), k0 = x0 - t * p.K;
        const int tr = fdiv(t, job.Sc_), ts = t - tr * job.Sc;
        const int k1 = min(p.K, k0 + j1 - x0);
        x0 += k1 - k0;
        unsigned dy[4];   // byte offset of dY[n][p][q][k0] of each pixel, kOOB outside
        bool some = false;
#pragma unroll
        for (int x = 0; x < 4; ++x) {
            const int n = fdiv(m0 + x, job.HWc), ij = m0 + x - n * (job.Hc * job.Wc);
            const int i = fdiv(ij, job.Wc_), j = ij - i * job.Wc;
            const int pp = i + job.da - tr, qq = j + job.db - ts;
            const bool ok = (want >> x & 1) && (unsigned)pp < (unsigned)p.P &&
                            (unsigned)qq < (unsigned)p.Q;
            dy[x] = ok ? 4u * (((n * p.P + pp) * p.Q + qq) * p.K + k0) : kOOB;
            some = some || ok;
        }
        if (!__any(some)) continue;
        const unsigned wstep = 4u * p.R * p.S * p.C;
        unsigned w = 4u * (((k0 * p.R + job.r0 + p.sh * tr) * p.S + job.s0 + p.sw * ts) * p.C + c);
#pragma unroll 1
        for (int k = k0; k < k1; k += kPlain) {
            float a[kPlain][4], b[kPlain];
#pragma unroll
            for (int u = 0; u < kPlain; ++u) {   // what lies past the tap is not added
                b[u] = buffer_load_f32(rw, c < p.C ? w + u * wstep : kOOB);
#pragma unroll
                for (int x = 0; x < 4; ++x)
                    a[u][x] = buffer_load_f32(rdy, dy[x] == kOOB ? kOOB : dy[x] + 4 * u);
            }
#pragma unroll
            for (int u = 0; u < kPlain; ++u)
#pragma unroll
                for (int x = 0; x < 4; ++x)
                    if (k + u < k1 && dy[x] != kOOB) sum[x] = fmaf(a[u][x], b[u], sum[x]);
#pragma unroll
            for (int x = 0; x < 4; ++x)
                if (dy[x] != kOOB) dy[x] += 4 * kPlain;
            w += kPlain * wstep;
        }
        if (!__any(undecided(sum, want))) break;
    }
}

// --------------------------------------------------------- data gradient --
// Block `bid` of a class job: split `split` of `nsplit` sums the reduction
// steps [st0, st1) of the class's (tr, ts, k) for one 64x64 tile of its
// pixels x channels.
template <int VA, int VB>
__device__ __forceinline__ void dgrad_tile(int bid, ConvLds &L, const DgradJob &job,
                                           const ConvProblem &p, const ConvDivs &dv) {
    using BC = BCols<VB>;
    const float *__restrict__ dY = job.dY;
    const float *__restrict__ Wt = job.Wt;
    float *__restrict__ out = job.out;
    const int tiles_c = job.tiles_c, nsplit = job.nsplit;

    const int HWc = job.Hc * job.Wc;
    const int Mc = p.N * HWc;
    const int RSKc = job.Rc * job.Sc * p.K;
    const int nsteps = (RSKc + BK - 1) / BK;
    const int split = bid % nsplit;
    bid /= nsplit;
    const int m0 = (bid / tiles_c) * BM;
    const int c0 = (bid % tiles_c) * BN;
    const int st0 = (int)((long)nsteps * split / nsplit);
    const int st1 = (int)((long)nsteps * (split + 1) / nsplit);

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int il = lane & 15, g = lane >> 4;
    const int wm = w & 1, wn = w >> 1;

    const auto rdy = buffer_rsrc(dY, p.N * p.P * p.Q * p.K * 4);
    const auto rw = buffer_rsrc(Wt, p.K * p.R * p.S * p.C * 4);

    // A staging: class pixel row ar (fixed), reduction columns aj .. aj + 3 of
    // a step; B staging: reduction row jr of a step, channel columns.
    const int ar = tid >> 3, aj = 4 * (tid & 7);
    const int m = m0 + ar;
    const bool mok = m < Mc;
    const int n = fdiv(m, job.HWc), ij = m - n * HWc;
    const int i = fdiv(ij, job.Wc_), jw = ij - i * job.Wc;
    const int jr = tid >> 4, cc = tid & 15;
    int cb[BC::NE];   // channel columns this thread stages
#pragma unroll
    for (int e = 0; e < BC::NE; ++e) cb[e] = c0 + BC::col(cc, e);

    const int nP = n * p.P, pi = i + job.da, qj = jw + job.db;   // p = pi - tr, q = qj - ts
    // K % BK == 0: every step lies within one tap (tr, ts), known to the
    // whole workgroup; otherwise each staged element finds its own tap.
    const bool tap_uniform = p.K % BK == 0;

    // dY offset of (tap (tr, ts), channel k) for this thread's pixel, or kOOB
    // when the tap's output position lies outside dY.
    auto dy_offset = [&](int tr, int ts, int k) {
        const int pp = pi - tr, qq = qj - ts;
        const bool ok = mok && (unsigned)pp < (unsigned)p.P && (unsigned)qq < (unsigned)p.Q;
        return ok ? (((nP + pp) * p.Q + qq) * p.K + k) * 4 : kOOB;
    };
    // first float of W[k][r][s][:] for tap (tr, ts)
    auto w_row = [&](int k, int tr, int ts) {
        return ((k * p.R + job.r0 + p.sh * tr) * p.S + job.s0 + p.sw * ts) * p.C;
    };

    using Regs = f32x4[2];   // A (dY), B (W)
    auto load = [&](int st, Regs &rg) {
        const int j0 = st * BK;
        int oa[4], ob[BC::NE];
        if (tap_uniform) {
            const int t0 = fdiv(j0, dv.K);
            const int kb = j0 - t0 * p.K;
            const int tr = fdiv(t0, job.Sc_);
            const int ts = t0 - tr * job.Sc;
            oa[0] = dy_offset(tr, ts, kb + aj);   // K % BK == 0: VA == 4
            // W[k][r][s][c] for reduction row k = kb + jr of the tap
            const int row = w_row(kb + jr, tr, ts);
#pragma unroll
            for (int e = 0; e < BC::NE; ++e) ob[e] = cb[e] < p.C ? (row + cb[e]) * 4 : kOOB;
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                // a 16-byte chunk (VA == 4, K % 4 == 0) never straddles two taps
                const int j = j0 + aj + e;
                const int t = fdiv(j, dv.K), k = j - t * p.K;
                const int tr = fdiv(t, job.Sc_), ts = t - tr * job.Sc;
                oa[e] = j < RSKc ? dy_offset(tr, ts, k) : kOOB;
                if (VA == 4) break;
            }
            const int j = j0 + jr;
            const int t = fdiv(j, dv.K), k = j - t * p.K;
            const int tr = fdiv(t, job.Sc_), ts = t - tr * job.Sc;
            const int row = w_row(k, tr, ts);
#pragma unroll
            for (int e = 0; e < BC::NE; ++e)
                ob[e] = (j < RSKc && cb[e] < p.C) ? (row + cb[e]) * 4 : kOOB;
        }
        rg[0] = load_vec<VA>(rdy, oa);
        if (VB == 4) {
            rg[1] = buffer_load_f32x4(rw, ob[0]);
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e) rg[1][e] = buffer_load_f32(rw, ob[e]);
        }
    };
    auto store = [&](int buf, const Regs &rg) {
        store_split4(L.A[buf], PixTile::at(ar, 2 * (aj & 15) + 4 * (aj >> 4)), rg[0]);
        if (VB == 4) {
            store_split4(L.B[buf], RedTile::at(jr, 4 * cc), rg[1]);
        } else {
            int o[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) o[e] = RedTile::at(jr, cc + 16 * e);
            store_split4(L.B[buf], o, rg[1]);
        }
    };

    f32x4 acc[2] = {zero4(), zero4()};

    // Lane bases of the reads: pixels 32wm + 16ii + il, reduction set of group
    // g of A; reduction rows 4g + br (+16), columns 16wn + bc of B.
    const int br = il >> 2, bc = 4 * (il & 3);
    const int ta[2] = {PixTile::at(32 * wm + il, 8 * g), PixTile::at(32 * wm + 16 + il, 8 * g)};
    const int tb = RedTile::at(4 * g + br, 16 * wn + bc);
    // Two register sets keep the loads of the next two steps in flight while
    // the current step, already in LDS, is multiplied.
    Regs rg[NP];
#pragma unroll
    for (int u = 0; u < NP; ++u)
        if (st0 + u < st1) load(st0 + u, rg[u]);
    if (st0 < st1) store(0, rg[0]);
    __syncthreads();
    // step st: `nx` holds step st+1 (in flight), `fr` is free
    auto body = [&](int st, Regs &nx, Regs &fr) {
        const int cur = (st - st0) & 1;
        if (st + NP < st1) load(st + NP, fr);
        const Split8 a[2] = {load_split<PixTile>(L.A[cur], ta[0]),
                             load_split<PixTile>(L.A[cur], ta[1])};
        mfma_split(a, load_split_tr<RedTile>(L.B[cur], tb, tb + 32 * 16), acc);
        if (st + 1 < st1) store(cur ^ 1, nx);
        __syncthreads();
    };
    for (int st = st0; st < st1; st += NP) {
#pragma unroll
        for (int u = 0; u < NP; ++u)
            if (st + u < st1) body(st + u, rg[(u + 1) % NP], rg[u]);
    }

    // rows of this lane's accumulators back to dX pixels (n, a + sh*i, b + sw*j)
    float *dst = out + (size_t)split * p.N * p.H * p.W * p.C;   // split 0 of 1 is dX
    float chk = 0.f;
    const int c = c0 + 16 * wn + il;
#pragma unroll
    for (int ii = 0; ii < 2; ++ii)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int mo = m0 + 32 * wm + 16 * ii + 4 * g + r;
            if (mo >= Mc) continue;
            const int on = fdiv(mo, job.HWc), oij = mo - on * HWc;
            const int oi = fdiv(oij, job.Wc_), oj = oij - oi * job.Wc;
            const size_t pix = ((size_t)on * p.H + job.a + p.sh * oi) * p.W + job.b + p.sw * oj;
            if (c < p.C) dst[pix * p.C + c] = acc[ii][r] * kDownProduct;
            chk = fmaf(acc[ii][r], 0.f, chk);   // NaN if not finite
        }
    if (!__all(finite_f32(chk))) {
        int gp = g, first = st0;
        hide(gp, first);
#pragma unroll 1
        for (int ii = 0; ii < 2; ++ii) {
            const int mo = m0 + 32 * wm + 16 * ii + 4 * gp;
            unsigned want = 0;
#pragma unroll
            for (int r = 0; r < 4; ++r)
                if (mo + r < Mc && c < p.C && !finite_f32(ii ? acc[1][r] : acc[0][r])) want |= 1u << r;
            float sum[4];
            dgrad_plain(sum, want, job, rdy, rw, p, dv, mo, c, first * BK, min(st1 * BK, RSKc));
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                if (!(want >> r & 1)) continue;
                const int on = fdiv(mo + r, job.HWc), oij = mo + r - on * HWc;
                const int oi = fdiv(oij, job.Wc_), oj = oij - oi * job.Wc;
                const size_t pix =
                    ((size_t)on * p.H + job.a + p.sh * oi) * p.W + job.b + p.sw * oj;
                dst[pix * p.C + c] = sum[r];
            }
        }
    }
}

// Which class job a block belongs to (job counts and sizes are uniform).
__device__ __forceinline__ int find_class(const DgradJobs &jobs, int &bid) {
    int c = 0;
    while (c + 1 < jobs.n && bid >= jobs.c[c].blocks) {
        bid -= jobs.c[c].blocks;
        ++c;
    }
    return c;
}

template <int VA, int VB>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(4, 8)))
void conv_dgrad_f32(DgradJobs jobs, ConvProblem p, ConvDivs dv, int first) {
    __shared__ __attribute__((aligned(16))) ConvLds lds;
    int bid = first + blockIdx.x;
    const int c = find_class(jobs, bid);
    dgrad_tile<VA, VB>(bid, lds, jobs.c[c], p, dv);
}

// Both derivatives of one convolution in one launch: the first `dblocks`
// workgroups run the data gradient's class jobs, the rest the filter gradient.
template <int VA, int VB>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(4, 8)))
void conv_bwd_f32(DgradJobs d, int dblocks, WgradJob w, ConvProblem p, ConvDivs dv, int first) {
    __shared__ __attribute__((aligned(16))) ConvLds lds;
    int bid = first + blockIdx.x;
    if (bid < dblocks) {
        const int c = find_class(d, bid);
        dgrad_tile<VA, VB>(bid, lds, d.c[c], p, dv);
    } else {
        wgrad_tile<VA, VB>(bid - dblocks, lds, w, p, dv);
    }
}

ConvDivs make_divs(const ConvProblem &p) {
    return ConvDivs{make_fastdiv(p.P * p.Q), make_fastdiv(p.Q), make_fastdiv(p.K),
                    make_fastdiv(p.S), make_fastdiv(p.C)};
}

}  // namespace

FastDiv make_fastdiv(unsigned d) {
    unsigned l = 0;
    while ((1ull << l) < d) ++l;
    const unsigned long long m = ((1ull << 32) * ((1ull << l) - d)) / d + 1;
    return FastDiv{(unsigned)m, l};
}

// Split a reduction when the output tiles alone fill fewer than
// MG_CONV_SPLIT_BELOW workgroups: aim at about MG_CONV_SPLIT_TARGET
// workgroups, with at least MG_CONV_SPLIT_TERMS summed terms per split.
#ifndef MG_CONV_SPLIT_BELOW
#define MG_CONV_SPLIT_BELOW 512
#endif
#ifndef MG_CONV_SPLIT_TARGET
#define MG_CONV_SPLIT_TARGET 1024
#endif
#ifndef MG_CONV_SPLIT_TERMS
#define MG_CONV_SPLIT_TERMS 256
#endif
constexpr int kStepTerms = 16;   // terms counted as one step
static int splits_for(long tiles, long steps) {
    if (tiles >= MG_CONV_SPLIT_BELOW) return 1;
    const long by_grid = (MG_CONV_SPLIT_TARGET + tiles - 1) / tiles;
    const long by_steps = steps / (MG_CONV_SPLIT_TERMS / kStepTerms);
    const long s = by_grid < by_steps ? by_grid : by_steps;
    return s < 1 ? 1 : (int)s;
}

int conv_wgrad_splits(const ConvProblem &p) {
    return splits_for((long)cdiv(p.K, BM) * cdiv(p.R * p.S * p.C, BN),
                      cdiv(p.N * p.P * p.Q, kStepTerms));
}

namespace {

// The stride-parity classes of the data gradient (see DgradJob), without
// the pointers and split; classes without pixels are left out.
std::vector<DgradJob> dgrad_classes(const ConvProblem &p) {
    std::vector<DgradJob> cls;
    for (int a = 0; a < p.sh; ++a)
        for (int b = 0; b < p.sw; ++b) {
            DgradJob j{};
            j.a = a;
            j.b = b;
            j.Hc = a < p.H ? cdiv(p.H - a, p.sh) : 0;
            j.Wc = b < p.W ? cdiv(p.W - b, p.sw) : 0;
            if (j.Hc == 0 || j.Wc == 0) continue;
            j.r0 = (a + p.ph) % p.sh;
            j.s0 = (b + p.pw) % p.sw;
            j.Rc = j.r0 < p.R ? cdiv(p.R - j.r0, p.sh) : 0;
            j.Sc = j.s0 < p.S ? cdiv(p.S - j.s0, p.sw) : 0;
            j.da = (a + p.ph - j.r0) / p.sh;
            j.db = (b + p.pw - j.s0) / p.sw;
            j.HWc = make_fastdiv(j.Hc * j.Wc);
            j.Wc_ = make_fastdiv(j.Wc);
            j.Sc_ = make_fastdiv(j.Sc > 0 ? j.Sc : 1);
            j.tiles_c = cdiv(p.C, BN);
            cls.push_back(j);
        }
    return cls;
}

}  // namespace

// One split count for every class: from the classes' total tiles and the
// longest class reduction.
int conv_dgrad_splits(const ConvProblem &p) {
    long tiles = 0, steps = 0;
    for (const DgradJob &j : dgrad_classes(p)) {
        tiles += (long)cdiv(p.N * j.Hc * j.Wc, BM) * j.tiles_c;
        steps = std::max<long>(steps, cdiv(j.Rc * j.Sc * p.K, kStepTerms));
    }
    return splits_for(tiles, steps);
}

namespace {

WgradJob wgrad_job(const ConvProblem &p, const float *X, const float *dY, float *dW,
                   float *partials) {
    const int ns = conv_wgrad_splits(p);
    const int tiles_j = cdiv(p.R * p.S * p.C, BN);
    return WgradJob{X, dY, ns > 1 ? partials : dW, tiles_j, ns, cdiv(p.N * p.P * p.Q, BK),
                    cdiv(p.K, BM) * tiles_j * ns};
}

// The data gradient's class jobs, in launches of at most kMaxClasses.
std::vector<DgradJobs> dgrad_jobs(const ConvProblem &p, const float *dY, const float *Wt,
                                  float *dX, float *partials) {
    const int ns = conv_dgrad_splits(p);
    std::vector<DgradJobs> launches;
    for (DgradJob j : dgrad_classes(p)) {
        j.dY = dY;
        j.Wt = Wt;
        j.out = ns > 1 ? partials : dX;
        j.nsplit = ns;
        j.blocks = cdiv(p.N * j.Hc * j.Wc, BM) * j.tiles_c * ns;
        if (launches.empty() || launches.back().n == kMaxClasses) launches.push_back(DgradJobs{});
        DgradJobs &l = launches.back();
        l.c[l.n++] = j;
    }
    return launches;
}

int total_blocks(const DgradJobs &d) {
    int b = 0;
    for (int i = 0; i < d.n; ++i) b += d.c[i].blocks;
    return b;
}

ReduceJob reduce_job(const float *partials, int nsplit, int total, float *out) {
    // lanes per element group: about nsplit / 4 splits each, at most 64
    int G = 1;
    while (G < 64 && 4 * G < nsplit) G *= 2;
    const int vec = total % 4 == 0;
    const long groups = vec ? total / 4 : total;
    return ReduceJob{partials, out, nsplit, total, G, vec, (int)((groups * G + 255) / 256)};
}

// The kernel instance for the operands' vector widths (16-byte loads along
// k when K % 4 == 0 and along c when C % 4 == 0, else 4-byte loads) and the
// output tile width.
template <template <int, int> class Launch, typename... Args>
hipError_t by_widths(const ConvProblem &p, Args &&...args) {
    const bool va = p.K % 4 == 0, vb = p.C % 4 == 0;
    if (va && vb) return Launch<4, 4>::run(args...);
    if (va) return Launch<4, 1>::run(args...);
    if (vb) return Launch<1, 4>::run(args...);
    return Launch<1, 1>::run(args...);
}

// launch(grid, first workgroup) over `blocks` workgroups of NT threads, in several
// launches where one grid's 2^32 threads are too few (the grid's size wraps there
// without an error).
constexpr int kMaxBlocks = 1 << 22;
static_assert((uint64_t)kMaxBlocks * NT < (1ull << 32), "threads of a grid");
template <typename F>
hipError_t in_grids(int blocks, F &&launch) {
    for (int first = 0; first < blocks; first += kMaxBlocks) {
        launch(dim3(std::min(kMaxBlocks, blocks - first)), first);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

template <int VA, int VB>
struct LaunchW {
    static hipError_t run(const WgradJob &j, const ConvProblem &p, const ConvDivs &dv,
                          hipStream_t s) {
        return in_grids(j.blocks, [&](dim3 grid, int first) {
            conv_wgrad_f32<VA, VB><<<grid, dim3(NT), 0, s>>>(j, p, dv, first);
        });
    }
};
template <int VA, int VB>
struct LaunchD {
    static hipError_t run(const DgradJobs &j, const ConvProblem &p, const ConvDivs &dv,
                          hipStream_t s) {
        return in_grids(total_blocks(j), [&](dim3 grid, int first) {
            conv_dgrad_f32<VA, VB><<<grid, dim3(NT), 0, s>>>(j, p, dv, first);
        });
    }
};
template <int VA, int VB>
struct LaunchDW {
    static hipError_t run(const DgradJobs &d, const WgradJob &w, const ConvProblem &p,
                          const ConvDivs &dv, hipStream_t s) {
        const int db = total_blocks(d);
        return in_grids(db + w.blocks, [&](dim3 grid, int first) {
            conv_bwd_f32<VA, VB><<<grid, dim3(NT), 0, s>>>(d, db, w, p, dv, first);
        });
    }
};

hipError_t launch_reduce(const ReduceJob &a, const ReduceJob &b, hipStream_t s) {
    conv_split_reduce_f32<<<dim3(a.blocks + b.blocks), dim3(256), 0, s>>>(a, b);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_conv_wgrad_f32(const ConvProblem &p, const float *X, const float *dY,
                                 float *dW, float *partials, hipStream_t s) {
    const WgradJob j = wgrad_job(p, X, dY, dW, partials);
    if (j.nsplit > 1 && partials == nullptr) return hipErrorInvalidValue;
    return by_widths<LaunchW>(p, j, p, make_divs(p), s);
}

hipError_t launch_conv_dgrad_f32(const ConvProblem &p, const float *dY, const float *Wt,
                                 float *dX, float *partials, hipStream_t s) {
    if (conv_dgrad_splits(p) > 1 && partials == nullptr) return hipErrorInvalidValue;
    const ConvDivs dv = make_divs(p);
    for (const DgradJobs &j : dgrad_jobs(p, dY, Wt, dX, partials)) {
        const hipError_t e = by_widths<LaunchD>(p, j, p, dv, s);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

hipError_t launch_conv_bwd_f32(const ConvProblem &p, const float *X, const float *Wt,
                               const float *dY, float *dX, float *dW, float *dpart,
                               float *wpart, hipStream_t s) {
    const WgradJob w = wgrad_job(p, X, dY, dW, wpart);
    if ((conv_dgrad_splits(p) > 1 && dpart == nullptr) || (w.nsplit > 1 && wpart == nullptr))
        return hipErrorInvalidValue;
    const ConvDivs dv = make_divs(p);
    const std::vector<DgradJobs> d = dgrad_jobs(p, dY, Wt, dX, dpart);
    // the filter gradient shares the first launch; strides beyond 4 x 4 add
    // data-gradient-only launches for the remaining classes
    hipError_t e = by_widths<LaunchDW>(p, d[0], w, p, dv, s);
    for (size_t i = 1; i < d.size() && e == hipSuccess; ++i) e = by_widths<LaunchD>(p, d[i], p, dv, s);
    return e;
}

hipError_t launch_conv_split_reduce_f32(const float *partials, int nsplit, int total,
                                        float *out, hipStream_t s) {
    return launch_reduce(reduce_job(partials, nsplit, total, out),
                         ReduceJob{nullptr, nullptr, 0, 0, 1, 0, 0}, s);
}

hipError_t launch_conv_split_reduce2_f32(const float *part_a, int nsplit_a, int total_a,
                                         float *out_a, const float *part_b, int nsplit_b,
                                         int total_b, float *out_b, hipStream_t s) {
    return launch_reduce(reduce_job(part_a, nsplit_a, total_a, out_a),
                         reduce_job(part_b, nsplit_b, total_b, out_b), s);
}

}  // namespace mg
