// Shape of a batch's persistent Explore (host only): the tuning in force and the
// workgroups each query gets.
#pragma once

#include <algorithm>
#include <cmath>

#include "pump.h"

namespace pump {

// 256 threads, 2 workgroups per CU, largest query first, graph on.
constexpr int kDefaultTeamScale = 64;

inline pump_batch_tuning tuning_or_default(const pump_batch_tuning* t) {
    return t ? *t : pump_batch_tuning{256, 2, 1, 1, kDefaultTeamScale};
}

// Workgroups of a query's team: team_scale / 4 times its share of `grid`
// workgroups (work of all queries' work_sum), 1 .. team_cap; 0: one.  At the
// default scale a team is also no larger than three times that share, or than its
// query has use for beside others (16 workgroups at 2000 nodes, and with their
// square), whichever is more: what a round's barriers cost grows with the team.
// With 16 times the share throughout, planning 96 queries of 2000 samples took 10.8
// ms, with this 7.6 (1.5 times the share: 7.3; but 64 queries of 1000 to 8000
// samples then take 28.8 instead of 27.6, since a heavy one ends last); few queries
// keep the whole device.
inline int team_size(int team_scale, int grid, int team_cap, double work, double work_sum, double nodes) {
    if (team_scale <= 0 || !(work_sum > 0.0)) return 1;
    const double share = grid * work / work_sum;
    const int size = (int)std::min(std::max(1.0, std::floor(0.25 * team_scale * share + 0.5)), (double)team_cap);
    if (team_scale != kDefaultTeamScale) return size;
    return std::min(size, (int)std::max(1.0, std::max(3.0 * share, nodes * nodes / 2.5e5)));
}

}  // namespace pump
