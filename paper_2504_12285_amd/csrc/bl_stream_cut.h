/* How the persistent stream kernels share a table of products among their workgroups (bl_stream.hip); host code without the
 * runtime, so that a host program can check it (tests/stream_index_driver.cpp). */
#pragma once
#include <stdint.h>

#include <algorithm>
#include <vector>

/* A position in the table: product, row group. */
struct bl_cut_pos {
    int x, y;
};

/* Cuts a table of products (units[i] row groups of unit_cost[i] each, enter_cost[i] for every workgroup that enters
 * product i) into `blocks` contiguous slices of about equal cost: walk the row groups once, cutting whenever a workgroup's cost
 * reaches the target; the last workgroup takes what is left.  Every cut inside a product adds one more entry, so the target is
 * raised by the last workgroup's surplus until that one is no longer than the others.  Where a dozen times do not get there (shares of
 * a few row groups, or entries that cost more than they) the slices are filled one after the other up to the smallest target that comes
 * to the table's end, by bisection in whole rounds of the workgroup's waves, if that makes the costliest a fifth cheaper.  Returns
 * blocks + 1 positions; the last slices may be empty.
 * (The last workgroup was left with up to 6.5 times the others' work, or all of it: 12 products of 4096 x 4736 in one launch
 * 26.0 us, 13.6 like this; one of 13824 x 320, five per byte, 240 and 5.8.  Bisection for every table leaves workgroups idle where a few
 * waves of each would do: one token up to +40 %, batched tables up to +33 %.) */
static inline std::vector<bl_cut_pos> bl_cut_slices(const std::vector<int>& units, const std::vector<int64_t>& unit_cost,
                                                    const std::vector<int64_t>& enter_cost, int blocks, int waves) {
    const int count = (int)units.size();
    std::vector<bl_cut_pos> wg((size_t)blocks + 1);
    /* a round of a workgroup's waves costs the same whether each has a row group in it or not */
    auto rounds = [&](int i, int64_t n) { return (n + waves - 1) / waves * waves * unit_cost[(size_t)i]; };
    int64_t least = 1, all = 0, all_rounds = 0, left_rounds = 0;
    for (int i = 0; i < count; ++i) {
        all += units[(size_t)i] * unit_cost[(size_t)i] + enter_cost[(size_t)i];
        all_rounds += rounds(i, units[(size_t)i]) + enter_cost[(size_t)i];
        least = std::max(least, waves * unit_cost[(size_t)i] + enter_cost[(size_t)i]);
    }
    bool even = false;
    int64_t target = all / blocks + 1;
    for (int iter = 0; iter < 12 && !even; ++iter) {
        int pi = 0, unit = 0;
        for (int b = 0; b < blocks; ++b) {
            wg[(size_t)b] = {pi, unit};
            int64_t c = 0;
            bool entered = false;
            while (pi < count && b < blocks - 1) {
                if (!entered) { c += enter_cost[(size_t)pi]; entered = true; }
                const int64_t uc = unit_cost[(size_t)pi];
                const int64_t room = target - c;
                const int64_t take = room > 0 ? (room + uc - 1) / uc : 0;
                const int left = units[(size_t)pi] - unit;
                if (take >= left) {
                    c += (int64_t)left * uc;
                    ++pi;
                    unit = 0;
                    entered = false;
                    if (c >= target) break;
                } else {
                    unit += (int)take;
                    break;
                }
            }
        }
        /* cost of what is left for the last workgroup */
        int64_t last = 0;
        left_rounds = 0;
        {
            int pi = wg[(size_t)blocks - 1].x, unit = wg[(size_t)blocks - 1].y;
            for (; pi < count; ++pi, unit = 0)
                if (units[(size_t)pi] > unit) {
                    last += enter_cost[(size_t)pi] + (int64_t)(units[(size_t)pi] - unit) * unit_cost[(size_t)pi];
                    left_rounds += enter_cost[(size_t)pi] + rounds(pi, units[(size_t)pi] - unit);
                }
        }
        even = last <= target + target / 64;
        target += (last - target) / blocks + 1;
    }
    if (!even) {
        const std::vector<bl_cut_pos> walked = wg;
        auto fill = [&](int64_t most) {
            int pi = 0, unit = 0;
            for (int b = 0; b < blocks; ++b) {
                wg[(size_t)b] = {pi, unit};
                int64_t room = most;
                while (pi < count) {
                    room -= enter_cost[(size_t)pi];
                    const int64_t uc = unit_cost[(size_t)pi], left = units[(size_t)pi] - unit;
                    const int64_t fit = room < 0 ? 0 : room / (waves * uc) * waves;
                    if (fit < left) {
                        unit += (int)fit;
                        break;
                    }
                    room -= rounds(pi, left);
                    ++pi;
                    unit = 0;
                }
            }
            return pi == count;
        };
        int64_t lo = std::max(least, all / blocks), hi = std::max(least, all_rounds);     /* one workgroup alone would need `all` */
        while (lo < hi) {
            const int64_t mid = lo + (hi - lo) / 2;
            if (fill(mid)) hi = mid;
            else lo = mid + 1;
        }
        fill(lo);
        if (lo > left_rounds / 5 * 4) wg = walked;
    }
    /* normalise an end position (count, 0) to (count - 1, units): the kernel never reads entry `count` */
    for (int b = 0; b <= blocks; ++b)
        if (b == blocks || wg[(size_t)b].x >= count) wg[(size_t)b] = {count - 1, units[(size_t)count - 1]};
    return wg;
}
