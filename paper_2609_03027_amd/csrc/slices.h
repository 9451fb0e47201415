// Time slices of a call: how many, and how long.
#pragma once

#include <cstdint>

namespace epic {

// Samples per slice for n_time samples (at most 2^31 - 1, whole units) on S slices of
// whole units: no more than n_time.
constexpr int slice_len(int64_t n_time, int64_t S, int64_t unit) {
    return (int)(((n_time + S - 1) / S + unit - 1) / unit * unit);
}

// Time slices of a call of a paired or row-unfolded group.  `slots` workgroups
// run at once (one paired workgroup fills a CU), so the call takes
// ceil(workgroups / slots) rounds of (samples per slice + a start and
// an end that cost about six samples); more than one slice adds the partial
// image sets' write and read (at about 4 TB/s against 4.5 us per sample) and
// the reduction's launch.  The cheapest count wins: 1 where the items alone
// fill whole rounds (128 channels on 256 CUs), 64 for one channel.  Frames
// need no partial sets, only slices of whole frames (`unit` samples, one or more).
constexpr int pair_slices(int64_t n_items, int64_t slots, int64_t n_time, int s_max,
                          int64_t part_floats, int64_t unit, bool frames) {
    int best = 1;
    double best_cost = 0.0;
    for (int S = 1; S <= s_max; ++S) {
        const int64_t tps = slice_len(n_time, S, unit);
        const int64_t used = (n_time + tps - 1) / tps;
        if (used != S) continue;
        const int64_t rounds = (n_items * used + slots - 1) / slots;
        const double sets = frames || S == 1 ? 0.0 : 1.0 + (double)S * (double)part_floats * 8.0 / 18e6;
        const double cost = (double)rounds * ((double)tps + 6.0) + sets;
        if (S == 1 || cost < 0.97 * best_cost) {
            best = S;
            best_cost = cost;
        }
    }
    return best;
}

}  // namespace epic
