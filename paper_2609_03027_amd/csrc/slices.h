// Time slices of a call: how many, and how long.
#pragma once

#include <cstdint>

namespace epic {

// Samples per slice for n_time samples (at most 2^31 - 1, whole units) on S slices of
// whole units: no more than n_time.
constexpr int slice_len(int64_t n_time, int64_t S, int64_t unit) {
    return (int)(((n_time + S - 1) / S + unit - 1) / unit * unit);
}

// Time slices of a call of a paired or row-unfolded group: `slices` of them, `len`
// samples each, the last one what is left.  `slots` workgroups run at once (one paired
// workgroup fills a CU), and a workgroup's start and end cost about six samples; more
// than one slice adds the partial image sets' write and read (at about 4 TB/s against
// 4.5 us per sample) and the reduction's launch.  Two forms: slices of equal length,
// ceil(workgroups / slots) rounds of them; or, where all slices but one fit one round,
// a short last slice, whose workgroups take turns on the slots that the others leave
// and end with them: 112 channels of 128^2 on 256 CUs are 224 workgroups of 7/8 of the
// samples and 224 of an eighth, seven after one another on each of the 32 CUs left,
// where equal slices need eight sets of sums for the same time.  Workgroups are dealt
// to 32 shader engines (of 8 XCDs) in turn, whichever has room, so the turns are
// counted for the fullest engine (counted for the chip, 24 channels of 1000 samples
// took 1119 us on a short last slice and 928 on equal ones).  The cheapest wins, fewer
// slices within 3 %: 1 where the items alone fill whole rounds (128 channels on 256
// CUs), 64 for one channel.  Frames need no partial sets, only slices of whole frames
// (`unit` samples, one or more).
struct SliceChoice {
    int slices, len;
    double cost;         // in samples of one workgroup
};
constexpr SliceChoice best_slices(int64_t n_items, int64_t slots, int64_t n_time, int s_max,
                                  int64_t part_floats, int64_t unit, bool frames) {
    SliceChoice best{1, (int)n_time, 0.0};
    for (int S = 1; S <= s_max; ++S) {
        const double sets = frames || S == 1 ? 0.0 : 1.0 + (double)S * (double)part_floats * 8.0 / 18e6;
        const int64_t equal = slice_len(n_time, S, unit);
        if ((n_time + equal - 1) / equal == S) {
            const int64_t rounds = (n_items * S + slots - 1) / slots;
            const double cost = (double)rounds * ((double)equal + 6.0) + sets;
            if (S == 1 || cost < 0.97 * best.cost) best = SliceChoice{S, (int)equal, cost};
        }
        const int64_t spare = slots / 32 - (n_items * (S - 1) + 31) / 32;
        if (S == 1 || spare <= 0) continue;
        // the shortest len whose rest r takes turns (r + 6) <= len + 6
        const int64_t turns = ((n_items + 31) / 32 + spare - 1) / spare, d = 1 + turns * (S - 1);
        const int64_t len = ((turns * (n_time + 6) - 6 + d - 1) / d + unit - 1) / unit * unit;
        const int64_t rest = n_time - (S - 1) * len;
        if (turns < 2 || rest <= 0 || rest > len) continue;
        const double cost = (double)len + 6.0 + sets;
        if (cost < 0.97 * best.cost) best = SliceChoice{S, (int)len, cost};
    }
    return best;
}

// Partial image sets of part_floats floats that an accumulator of such a group
// holds: the most that a call could use, within 64 and 96 MiB.  (112 channels of 128^2,
// 29 MB of sums, hold two, which take 11 % off long calls; with equal slices only they
// held eight.)
constexpr int reserved_slices(int64_t n_items, int64_t slots, int64_t part_floats) {
    const int64_t most = (int64_t{96} << 20) / (4 * (part_floats > 0 ? part_floats : 1));
    const int cap = (int)(most < 1 ? 1 : most < 64 ? most : 64);
    int useful = 1;
    for (int64_t n = 4; n <= 65536; n *= 2) {
        const SliceChoice c = best_slices(n_items, slots, n, cap, part_floats, 1, false);
        if (c.slices > useful) useful = c.slices;
    }
    return useful;
}

}  // namespace epic
