// work_order.h -- order in which the workgroups of a key-padded non-causal
// grid take its tiles (strict-f32 kernels).
#pragma once

#include "device_common.h"
#include "launch.h"

namespace mg {

// ---------------------------------- work-first order for key-padded grids
// In a non-causal problem with key padding, the key tiles at or past a
// batch's key length have no query work (their workgroups only write zero
// dK/dV rows).  Numbered in plain slot-major order such idle workgroups sit
// between the working ones and leave CU slots empty while working tiles wait,
// which measured 20-40 % slower than the same number of working tiles
// dispatched back to back.  Here every XCD x takes the heads h = x (mod 8)
// (workgroups are dealt to the eight XCDs round-robin, so block 8k + x runs
// on XCD x and a head's tiles share one L2), and its k-th block takes the
// k-th working (slot, head) of those heads in slot-major order, then the
// idle ones.  Needs B*H a multiple of 8 and at most 64 heads per XCD; the
// launcher checks both.  All lanes return the same slot and head.
__device__ __forceinline__ int nth_set_bit(uint64_t mask, int n) {
    for (int t = 0; t < n; ++t) mask &= mask - 1;   // drop the n lowest set bits
    return __builtin_ctzll(mask);
}

__device__ __forceinline__ void work_first_tile(int id, int nslots, int nsplit, int key_rows,
                                                int BH, int H, int Lk,
                                                const int32_t *__restrict__ key_len, int &slot,
                                                int &head) {
    const int lane = threadIdx.x & 63;
    const int x = id & 7, k = id >> 3;
    const int G = BH >> 3;                // heads of this XCD's group
    const bool valid = lane < G;
    const int klen = valid ? key_limit(key_len, (x + 8 * lane) / H, Lk) : 0;
    int before = 0;
    for (int pass = 0; pass < 2; ++pass) {   // working tiles, then idle ones
        for (int s = 0; s < nslots; ++s) {
            const bool works = (s / nsplit) * key_rows < klen;
            const uint64_t m = __ballot(valid && works == (pass == 0));
            const int c = __popcll(m);
            if (k < before + c) {
                slot = s;
                head = x + 8 * nth_set_bit(m, k - before);
                return;
            }
            before += c;
        }
    }
    slot = 0;   // not reached: the grid holds exactly nslots * B*H blocks
    head = x;
}

// The forward's version: every query tile of a non-causal key-padded head
// costs ceil(key length / key_rows) key tiles, so the k-th block of XCD x
// takes its heads' (slot, head) pairs by decreasing cost (head by head within
// one cost), and the short ones fill in at the end (a longest-first list
// schedule per XCD).  Same requirements as work_first_tile.
__device__ __forceinline__ void heavy_first_tile(int id, int nslots, int key_rows, int BH, int H,
                                                 int Lk, const int32_t *__restrict__ key_len,
                                                 int &slot, int &head) {
    const int lane = threadIdx.x & 63;
    const int x = id & 7, k = id >> 3;
    const int G = BH >> 3;
    const bool valid = lane < G;
    const int klen = valid ? key_limit(key_len, (x + 8 * lane) / H, Lk) : 0;
    const int cost = (klen + key_rows - 1) / key_rows;
    int before = 0;
    for (int v = (Lk + key_rows - 1) / key_rows; v >= 0; --v) {
        const uint64_t m = __ballot(valid && cost == v);
        const int c = __popcll(m) * nslots;
        if (k < before + c) {
            const int j = k - before;
            head = x + 8 * nth_set_bit(m, j / nslots);
            slot = j % nslots;
            return;
        }
        before += c;
    }
    slot = 0;   // not reached
    head = x;
}

// Key-padded non-causal grids take the XCD-grouped work orders
// (heavy_first_tile, work_first_tile) when the heads split evenly over the
// eight XCDs, at most 64 per XCD, and the per-workgroup search (one ballot
// per key tile) stays short: at most 1024 tiles of 64 keys, 2048 of 32.
inline int padded_work_order(const AttnProblem &p) {
    const int BH = p.B * p.H;
    return (p.key_len != nullptr && !p.causal && BH % 8 == 0 && BH <= 512 &&
            p.Lk <= 1024 * 64) ? 1 : 0;
}

}  // namespace mg
