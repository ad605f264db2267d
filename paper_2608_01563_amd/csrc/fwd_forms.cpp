// fwd_forms.cpp -- which form of the strict-f32 forward a problem takes (host).
#include "fwd_forms.h"

#include <algorithm>
#include <cmath>

namespace mg {
namespace {

constexpr int kCUs = 256;

// Cost of a form, in us: `chain` per key tile of a workgroup alone on its CU;
// `start` per workgroup and `tile` + `wave` per key tile where the CU is full,
// `wave` for the share of the workgroup's waves that hold rows.
struct FormCost {
    FwdForm form;
    int rows, keys;   // per workgroup; keys: of one step of all its waves
    float chain, start, tile, wave;
};

// Fitted once per head dimension to GPU times of every form over 1,873 problems
// (B*H 1 to 2048, 17 to 2048 rows and keys, all masks; the model's error is
// about 10 %).  What the rule picks from these is 1.8 % slower than the fastest
// form on average, and on 700 random problems outside the fit 1.3 %; the
// thresholds on tile counts that stood here before, which counted the rows of a
// tile whether a head fills them or not, were 15 % slower than it (B1 H1351 L55
// d128 causal 92 -> 38 us, B32 H51 L32 d32 18.9 -> 7.1, B64 H16 L128 d128 104 ->
// 74) and up to 2.3 times as slow as the f32 matrix-core forward of 64 rows that
// these kernels replaced.
constexpr FormCost kCost32[] = {
    {FwdForm::kFew, 16, 64, 0.47f, 0.18f, 0.25f, 0.16f},
    {FwdForm::kFewWave, 16, 16, 0.41f, 0.11f, 0.07f, 0.03f},
    {FwdForm::kRows32, 32, 64, 1.20f, 0.45f, 0.44f, 0.05f},
    {FwdForm::kRows64Pair, 64, 64, 1.21f, 0.99f, 0.53f, 0.35f},
    {FwdForm::kRows32Quad, 32, 128, 1.39f, 1.10f, 0.59f, 0.45f},
    {FwdForm::kRows64, 64, 32, 1.12f, 0.55f, 0.20f, 0.23f},
};
constexpr FormCost kCost64[] = {
    {FwdForm::kFew, 16, 64, 0.83f, 0.38f, 0.23f, 0.50f},
    {FwdForm::kFewWave, 16, 16, 0.68f, 0.37f, 0.11f, 0.07f},
    {FwdForm::kRows32, 32, 64, 1.86f, 1.06f, 0.81f, 0.17f},
    {FwdForm::kRows64Pair, 64, 64, 1.96f, 1.91f, 0.97f, 0.45f},
    {FwdForm::kRows32Quad, 32, 128, 1.71f, 2.58f, 1.45f, 0.90f},
    {FwdForm::kRows64, 64, 32, 1.59f, 0.99f, 0.38f, 0.40f},
};
constexpr FormCost kCost128[] = {
    {FwdForm::kFew, 16, 64, 1.14f, 1.16f, 0.70f, 0.93f},
    {FwdForm::kFewWave, 16, 16, 1.22f, 0.98f, 0.27f, 0.07f},
    {FwdForm::kRows64Pair, 64, 64, 2.42f, 4.50f, 2.31f, 1.06f},
    {FwdForm::kRows128, 128, 32, 1.21f, 3.09f, 0.91f, 2.55f},
    {FwdForm::kRows256, 256, 32, 2.20f, 6.03f, 0.83f, 5.16f},
    {FwdForm::kRows64, 64, 32, 2.25f, 2.77f, 0.77f, 0.86f},
};

// Time of the form beyond the launch: the longer of one workgroup's chain of
// key tiles and the CUs' rounds of workgroups (both count where they are alike).
// Causal grids start their longest tiles first, so their rounds even out as far
// as the tiles' lengths differ.  Padded key sides are taken as 85 % full.
float estimate(const AttnProblem &p, const FormCost &c) {
    const int tiles = cdiv(p.Lq, c.rows);
    const int splits = c.form == FwdForm::kFew ? few_column_splits(p) : 1;
    // a column split repeats the scores, half of a tile's work
    const float part = 0.5f + 0.5f / splits;
    const float filled = few_rows(c.form) ? 1.f : 16.f * cdiv(p.Lq, 16) / ((float)tiles * c.rows);
    const int longest = cdiv(p.Lk, c.keys);
    float mean = (float)longest, even = 0.f;
    if (p.causal) {
        const int shortest = cdiv(std::max(1, std::min(p.Lk, c.rows + p.Lk - p.Lq)), c.keys);
        mean = 0.5f * (longest + shortest);
        even = 1.f - (float)shortest / longest;
    }
    if (p.key_len != nullptr) mean *= 0.85f;
    const float per_cu = (float)tiles * p.B * p.H * splits / kCUs;
    const float rounds =
        (1.f - even) * std::ceil(per_cu) + even * std::max(per_cu + 0.25f, 1.f);
    const float chain = longest * c.chain * part;
    const float rate = rounds * (c.start + mean * (c.tile + c.wave * filled) * part);
    return std::sqrt(std::sqrt(chain * chain * chain * chain + rate * rate * rate * rate));
}

// The cheapest form, of at least `rows` rows.
template <int N>
FwdForm cheapest(const AttnProblem &p, const FormCost (&costs)[N], int rows = 16) {
    FwdForm best = costs[0].form;
    float least = INFINITY;
    for (const FormCost &c : costs) {
        if (c.rows < rows) continue;
        // beyond a few steps a lone wave's chain is longer than the model has it
        if (c.form == FwdForm::kFewWave && p.Lk > 96) continue;
        const float t = estimate(p, c);
        if (t < least) {
            least = t;
            best = c.form;
        }
    }
    return best;
}

// Share of its tiles that a side of L fills.
float filled(int L, int tile) { return (float)L / (tile * cdiv(L, tile)); }

// Rows and keys beyond 256 (keys beyond 1024: rows beyond 64): tiles are full, and
// what decides is whether the grid gives every CU its share (GPU time in us at
// d = 64 unless named).
//   few: a causal grid of up to 512 16-row blocks, else 256: B4 H4 L256 6.8
//     (64-row forward 9.2), B1 H4 L2048 d128 93 (150).
//   128 rows while they give two workgroups per CU: B8 H8 L1024 causal 54.7,
//     B4 H16 L2048 341 (two groups of 64 rows 388).
//   64 rows, two key groups, below that: B2 H6 L1500 73.8 (four groups of 32
//     rows 98), B4 H8 L512 18.7, B16 H8 L512 causal 34.3.
//   32 rows, four key groups, where a row's chain of keys sets the time: B2 H6
//     L1200 causal 30.0 (two groups of 64 rows 36.2), B1 H4 L4096 causal 84.6
//     (112), B4 H6 L300 10.9 (12.7).
//   d = 128: two key groups below 192 128-row tiles (B2 H8 L1024 causal 58.2),
//     then 128 rows (B4 H16 L1024 causal 104), 256 when those fill two rounds (B4
//     H16 L2048 572, 128 rows 676).
FwdForm long_form(const AttnProblem &p) {
    const long BH = (long)p.B * p.H;
    const long rows32 = cdiv(p.Lq, 32) * BH, rows128 = cdiv(p.Lq, 128) * BH,
               rows256 = cdiv(p.Lq, 256) * BH;
    if (few_row_blocks(p) <= (p.causal || p.d == 128 ? 512 : 256))
        return p.Lk < 1024 ? FwdForm::kFew : FwdForm::kFewLong;
    if (p.d == 128)
        return rows256 >= 512   ? FwdForm::kRows256
               : rows128 >= 192 ? FwdForm::kRows128 : FwdForm::kRows64Pair;
    if (rows128 >= 512) return FwdForm::kRows128;
    const bool chain = p.d == 32 ? rows32 <= (p.causal ? 1024 : 512)
                                 : rows32 <= (p.causal && p.Lk >= 1024 ? 512 : 256);
    return chain ? FwdForm::kRows32Quad : FwdForm::kRows64Pair;
}

}  // namespace

long few_row_blocks(const AttnProblem &p) { return (long)cdiv(p.Lq, kFewRows) * p.B * p.H; }

// Workgroups per (head, row block): the value columns are split (32 or more
// each) until there is one workgroup per CU.  B8 H16 Lq1 Lk4096 d128 (128 row
// blocks): bf16 39.6 -> 35.1 us, strict 86.7 -> 72.5 us; beyond 256 workgroups
// the repeated scores cost more (B32 H16 Lq1: 184 -> 261 us).
int few_column_splits(const AttnProblem &p) {
    int cs = 1;
    while (cs * 2 <= p.d / 32 && few_row_blocks(p) * cs * 2 <= kCUs) cs *= 2;
    return cs;
}

int form_rows(FwdForm f) {
    switch (f) {
    case FwdForm::kRows32:
    case FwdForm::kRows32Quad: return 32;
    case FwdForm::kRows64:
    case FwdForm::kRows64Pair: return 64;
    case FwdForm::kRows128: return 128;
    case FwdForm::kRows256: return 256;
    default: return kFewRows;
    }
}

// One step of keys needs no second wave (until the lone waves are so many that
// starting them takes longer than 64-row workgroups: d = 64 B1 H463 Lq1154 Lk14
// 82 us, 64 rows 64); a decode step reads a long cache with the most loads in
// flight.  The model's 10 % does not tell forms apart that are alike but for
// tiles that a problem without masks and lengths fills (GPU us):
//   128 rows and 64 keys at a time where both sides fill them, from one tile per
//     CU (d = 32 B8 H32 L128 9.3 -> 8.0, L256 21.2 -> 18.2, d = 64 32.5 -> 29.7), or
//     most of them over many rounds (d = 64 B1 H1377 L229 148 -> 138); not
//     with lengths (d = 64 B64 H16 L128 1.13 times the 64 rows' time)
//   32 full rows in one round of one workgroup per CU instead of two of 16 rows
//     (B8 H8 L128 8.1 -> 7.7, B4 H8 L256 10.8 -> 10.2; causal in two rounds, d = 32
//     B8 H8 L256 8.6 -> 8.0)
// and it has no cost of K and V read again: 32 and more rows (d <= 64) where two
// rounds and more of 16-row workgroups each read 1024 keys (B1 H384 Lq17 Lk2048
// 0.73 of their time, with lengths 0.80, B1 H256 Lq48 Lk1024 0.96).
FwdForm strict_fwd_form(const AttnProblem &p) {
    if (p.Lk <= 16)
        return p.d <= 64 && p.Lq >= 64 && few_row_blocks(p) >= 4096 ? FwdForm::kRows64
                                                                    : FwdForm::kFewWave;
    if (p.Lq <= kFewRows && p.Lk >= 512) return FwdForm::kFewLong;
    if (p.Lk > 1024 ? p.Lq > 64 : p.Lq > 256 && p.Lk > 256) return long_form(p);
    const bool plain = p.d <= 64 && !p.causal && p.key_len == nullptr;
    const long BH = (long)p.B * p.H, tiles128 = cdiv(p.Lq, 128) * BH, tiles32 = cdiv(p.Lq, 32) * BH;
    const float full = std::min(filled(p.Lq, 128), filled(p.Lk, 64));
    if (plain && p.Lk > 96 &&
        ((tiles128 >= kCUs && full >= 0.9375f) || (tiles128 >= 4 * kCUs && full >= 0.85f)))
        return FwdForm::kRows128;
    const bool full32 = p.Lk >= 128 && filled(p.Lk, 64) >= 0.9375f && filled(p.Lq, 32) >= 0.9375f;
    const bool round32 = plain ? tiles32 <= kCUs && tiles32 > kCUs * 7 / 8
                               : p.causal && tiles32 > 2 * kCUs * 7 / 8;
    const bool again = p.Lk >= 1024 && few_row_blocks(p) > 2 * kCUs;
    const int rows = (full32 && round32) || again ? 32 : 16;
    const FwdForm form = p.d == 32   ? cheapest(p, kCost32, rows)
                         : p.d == 64 ? cheapest(p, kCost64, rows) : cheapest(p, kCost128);
    return form == FwdForm::kFew && p.Lk > 1024 ? FwdForm::kFewLong : form;
}

}  // namespace mg
