// tiles_direct.h -- global->LDS tile copies that use gfx950's direct-to-LDS
// buffer loads (buffer_load_dword/dwordx4 ... lds): the loaded data is
// written to LDS by the load itself, so no staging registers and no LDS
// store instructions are needed.  Completion is tracked by the issuing
// wave's vmcnt; a barrier then makes the tile visible to the workgroup.
#pragma once

#include "device_common.h"

namespace mg {

// A [ROWS][D] f32 tile copied row by row straight into a padded LDS array
// dst[ROWS][LD]: one wave-wide 4-byte direct-to-LDS buffer load moves 64
// consecutive floats of a row (256 bytes, fully coalesced), so every row
// keeps the padded stride and all operand reads keep immediate offsets from
// one per-lane base.  For D = 32 the upper half of the wave stays idle.  Rows
// at or beyond L arrive as zeros.  Loads are dealt to the waves round-robin.
template <int ROWS, int D, int NW, int LD>
struct RowDirectTile {
    static constexpr int kPart = D < 64 ? D : 64;       // floats per load
    static constexpr int kParts = D / kPart;            // loads per row
    static constexpr int kLoads = ROWS * kParts;        // loads per tile
    static constexpr int kPerWave = (kLoads + NW - 1) / NW;
    static constexpr bool kEven = kLoads % NW == 0;
    static_assert(D % kPart == 0 && LD >= D, "row shape");

    __device__ __forceinline__ void issue(float (*dst)[LD], const float *__restrict__ src,
                                          int row0, int L, int w, int lane) const {
        const int rows = min(max(L - row0, 0), ROWS);
        const auto rsrc = buffer_rsrc(src + (size_t)row0 * D, rows * D * 4);
#pragma unroll
        for (int u = 0; u < kPerWave; ++u) {
            const int t = u * NW + w;
            if (!kEven && t >= kLoads) break;
            const int row = t / kParts;
            const int part = t - row * kParts;
            if (kPart == 64 || lane < kPart)
                __builtin_amdgcn_raw_ptr_buffer_load_lds(
                    rsrc, (__attribute__((address_space(3))) void *)&dst[row][kPart * part], 4,
                    (row * D + kPart * part + lane) * 4, 0, 0, 0);
        }
    }
};

}  // namespace mg
