// fwd_forms.h -- which form of the strict-f32 forward a problem takes.
#pragma once

#include "launch.h"

namespace mg {

// 16 query rows per workgroup (attn_few.hip): one wave, or the keys dealt to
// four waves in steps of 16, or to four or eight in steps of 2048 / d; and 32 to
// 256 rows per workgroup over shared key tiles (attn_f32x3_fwd.hip).
enum class FwdForm {
    kFewWave, kFew, kFewLong,
    kRows32,       // two groups of waves, half of a key tile each
    kRows32Quad,   // four groups, 128-key tiles
    kRows64,       // one group, four waves
    kRows64Pair,   // two groups
    kRows128,
    kRows256,      // d = 128: two 16-row blocks per wave
};

FwdForm strict_fwd_form(const AttnProblem &p);
inline bool few_rows(FwdForm f) { return f <= FwdForm::kFewLong; }
int form_rows(FwdForm f);   // query rows per workgroup

constexpr int kFewRows = 16;
long few_row_blocks(const AttnProblem &p);
int few_column_splits(const AttnProblem &p);

}  // namespace mg
