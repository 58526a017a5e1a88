// Rules by which the host launches the row kernels.  Plain host code: a test runs them without a GPU.
#pragma once

#include <stdint.h>

namespace difr {

// RowPace: the workgroup of a launch of `groups` from which on they share the issue slots by what they have left, where `resident` of
// them are held at once (0: not known, none does).  The likelihood kernel's.
constexpr int pace_from(int64_t groups, int resident) { return (int)(groups - resident); }

// ... of the streams that score every entry, `entries` to a workgroup.  Up to a twelfth more workgroups than fit start where a few rows end
// early, and then it is better that some do: with short rows one priority for all.  us with one priority / sharing, bf16: Token-DiFR, 1536
// fit, 1600 x 9000 20.6 / 21.5, 1600 x 30,000 36.7 / 37.9, 1800 x 30,000 39.7 / 38.8, 1600 x 128,256 100.7 / 96.6; both scores, 1280 fit, 1300 x
// 9000 26.1 / 27.0, 1500 28.3 / 27.5, 1300 x 78,058 79.2 / 76.7; fp32, 1536 fit, 1600 x 4000 20.4 / 20.9, 1728 21.7 / 21.4, with the
// admissible set 1552 x 30,000 62.7 / 65.6; shared rows with the rank, 1050 parts of 7000 entries on 1024 places 27.6 / 28.4.
constexpr int64_t kPaceEntries = 32768;
constexpr int pace_from(int64_t groups, int resident, int64_t entries)
{
    const int64_t before = groups - resident;
    return before > 0 && 12 * before <= resident && entries < kPaceEntries ? (int)groups : (int)before;
}

}  // namespace difr
