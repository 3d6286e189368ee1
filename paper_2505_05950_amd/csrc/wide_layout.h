// Where the kernels of wide token groups keep what they hand on (up_split.hip, up_wide.hip, wide_batch.hip).
//
// The gate kernel cuts the channels of all groups, eight at a time, into equal pieces, one workgroup each.  What a piece has of a group is
// a segment: the union of the rows that the group's tokens selected there, in pairs of 16-row tiles.  A segment's row ids (32 per pair, the
// last one repeated) and its h lie at the pair slot of its first channel, one slot further for every piece before it in the group, so that no
// two segments meet whatever their channels are and nobody has to know how many rows another segment has.  Segment (piece, group) has entry
// piece + group of the table: neighbours in the sequence differ by one in either or in both.
#pragma once

#include "floe_dev.h"
#include "launch.h"

namespace floe {

// a group's record, held by lane l of the wave, in scalars (the fields that gate and down look at)
__device__ __forceinline__ WideGroup wide_record(const WideGroup& rec, int l) {
    WideGroup g{};
    g.n = __builtin_amdgcn_readlane(rec.n, l);
    g.first = __builtin_amdgcn_readlane(rec.first, l);
    g.tile = __builtin_amdgcn_readlane(rec.tile, l);
    const uint64_t p = (uint64_t)rec.e.gd;
    g.e.gd = (const h16*)((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)p, l) |
                          (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(p >> 32), l) << 32);
    return g;
}

// token row of the tiles that position i of the order has, and its group; every lane the same
__device__ __forceinline__ int wide_token_row(const WideGroup* __restrict__ groups, int ng, int max_groups, int i, int lane, int& g) {
    for (int g0 = 0; g0 < ng; g0 += kWave) {
        const WideGroup* mine = groups + min(g0 + lane, max_groups - 1);
        const int n = mine->n, first = mine->first, tile = mine->tile;
        const unsigned long long m = __ballot(g0 + lane < ng && i >= first && i < first + n);
        if (m) {
            const int l = __ffsll((long long)m) - 1;
            g = g0 + l;
            return __builtin_amdgcn_readlane(tile * 16 + i - first, l);
        }
    }
    g = 0;
    return 0;  // (not reached: every position belongs to a group)
}

// What the gate kernel expects to find empty, a thread per task (position i of the order)
__device__ __forceinline__ void wide_clear(const WidePrep& p, int i, int task, int n_tasks) {
    p.tau[i] = p.task_tau[task];
    p.scale[i] = p.task_scale ? p.task_scale[task] : 1.0f;
    p.count[task] = 0;
    p.hmax[i] = 0u;
    p.task_rows[task] = make_int2(0, 0);  // filled in by the down kernel unless the group has no rows at all
    for (int s = i; s < p.n_segments; s += n_tasks) p.segments[s] = make_int4(0, 0, 0, 0);
}

}  // namespace floe
