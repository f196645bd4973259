// The schedule of the stream kernel (stream_spmm.hip): which B rows a workgroup brings into LDS when, and which K-steps of its row
// groups its waves multiply when.
#pragma once

#include <algorithm>
#include <cstdint>
#include <vector>

#include "vbr_internal.h"

namespace vbrk {

// The groups of one workgroup: wave w's are group_of[w * kStreamGroups ...], -1 none; `units` the units of 16 B rows they take (unit i: B rows 16 i ..), rising;
// unit(l, k, h) the place in `units` of the one that half h of the l-th's K-step k takes, and frag_of its first fragment in KiB of the values.  Writes the
// steps' records behind those in `out` and returns the number of steps, 0 if there is no schedule.
//
// A step is what happens between two barriers: every wave asks for up to kStreamUnits units of B, multiplies up to `ops` K-steps, and turns the units it asked
// for kStreamAhead steps before into LDS.  The operands of a step's first K-step are read at the end of the step before.  So a unit asked for
// in step t is there from step t + kStreamAhead + 1 on, for a first K-step a step later.  One whose last K-step is multiplied in step t is read no more
// when step t + 1 writes.  Units come in the order of their rows, into any slot that is free, and stay until their last use.  A group waits with the
// first half of at most one K-step for the second, so kStreamWaves * kStreamGroups slots can be taken and one more is enough to go on.
template <class Unit>
int64_t stream_schedule(int ops, const int32_t *group_of, const int32_t *n_ks_of, const int64_t *frag_of, const std::vector<int32_t> &units, Unit unit, int share, int sharers, std::vector<StreamRecord> &out)
{
    constexpr int kAll = kStreamWaves * kStreamGroups, kZeros = kStreamSlots * kStreamUnitBytes;
    const size_t begin = out.size();
    std::vector<int32_t> uses(units.size(), 0), slot(units.size(), -1), from(units.size(), INT32_MAX), free_slots;
    int32_t next[kAll], left[kAll], u[kAll][2];
    int64_t todo = 0;
    for (int l = 0; l < kAll; ++l) {
        next[l] = 0;
        left[l] = group_of[l] < 0 ? 0 : n_ks_of[l];
        todo += left[l];
        for (int32_t k = 0; k < left[l]; ++k)
            for (int h = 0; h < 2; ++h) ++uses[(size_t)unit(l, k, h)];
        for (int h = 0; h < 2 && left[l] > 0; ++h) u[l][h] = unit(l, 0, h);
    }
    for (int32_t s = kStreamSlots; s-- > 0;) free_slots.push_back(s);
    out.reserve(begin + 2 * kStreamWaves * std::max<size_t>(units.size() / (kStreamWaves * kStreamUnits), (size_t)todo / (kStreamWaves * ops)) * 9 / 8 + 16 * kStreamWaves);
    size_t staged = 0;
    int idle = 0;
    StreamRecord empty = {};
    for (int i = 0; i < kStreamMostOps; ++i) {
        empty.slot(i) = kZeros;
        empty.frag(i) = kStreamNone;
        empty.groups() |= (int32_t)((uint32_t)kStreamGroups << (4 * i));
    }
    empty.none() = kStreamNone;
    empty.to() = kZeros;
    empty.early(0) = empty.early(1) = -1;
    size_t ahead = 0;
    for (int64_t t = 0; todo > 0 || t % kStreamAhead > 0; ++t) {
        const size_t at = out.size();
        out.resize(at + 2 * kStreamWaves, empty);
        StreamRecord *now = out.data() + at, *before = t > 0 ? now - 2 * kStreamWaves : nullptr;
        bool moved = false;
        for (int w = 0; w < kStreamWaves; ++w)
            for (int i = 0; i < ops; ++i) {
                // of the K-steps that are there the one whose first unit comes first
                int best = -1;
                int32_t first = INT32_MAX;
                for (int l = w * kStreamGroups; l < (w + 1) * kStreamGroups; ++l) {
                    if (next[l] == left[l] || u[l][0] >= first) continue;
                    if (std::max(from[(size_t)u[l][0]], from[(size_t)u[l][1]]) > t - (i == 0 ? 1 : 0)) continue;
                    first = u[l][0];
                    best = l;
                }
                if (best < 0) continue;
                const int32_t k = next[best]++;
                --todo;
                moved = true;
                for (int h = 0; h < 2; ++h) {
                    (i > 0 ? now[2 * w + h].slot(i - 1) : before[2 * w + h].slot(ops - 1)) = slot[(size_t)u[best][h]] * kStreamUnitBytes;
                    before[2 * w + h].frag(i) = (int32_t)(uint32_t)((frag_of[best] + k) << 10);
                    now[2 * w + h].groups() ^= (int32_t)((uint32_t)(best % kStreamGroups ^ kStreamGroups) << (4 * i));
                    if (--uses[(size_t)u[best][h]] == 0) free_slots.push_back(slot[(size_t)u[best][h]]);
                    if (next[best] < left[best]) u[best][h] = unit(best, next[best], h);
                }
            }
        for (int i = 0; i < kStreamWaves * kStreamUnits && staged < units.size() && !free_slots.empty(); ++i) {
            const size_t fresh = staged++;
            slot[fresh] = free_slots.back();
            free_slots.pop_back();
            from[fresh] = (int32_t)t + kStreamAhead + 1;
            now[i].row() = units[fresh] * kSlabRows;
            now[i].none() = 0;
            now[i].to() = slot[fresh] * kStreamUnitBytes;
            moved = true;
        }
        // this workgroup's share of the units up to kStreamEarly further on, by another wave in every step
        for (int i = 0; sharers > 1 && i < 4 * kStreamWaves && ahead < std::min(units.size(), staged + kStreamEarly); ++ahead) {
            if (units[ahead] % sharers != share || ahead < staged) continue;
            now[2 * ((t + i / 4) % kStreamWaves) + (i / 2 & 1)].early(i & 1) = units[ahead] * kSlabRows;
            ++i;
        }
        idle = moved ? 0 : idle + 1;
        if (idle > 2 * kStreamAhead + 2) {
            out.resize(begin);
            return 0;
        }
    }
    return (int64_t)(out.size() - begin) / (2 * kStreamWaves);
}

}  // namespace vbrk
