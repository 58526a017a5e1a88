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

// Whether rows of both scores run by RowPace at all: not where a compute unit has one row at most, for which looking after the priority costs 3 to
// 4%.  us with / without, graph replays: bf16 64 x 30,000 19.8 / 19.6 (with the rank 22.3 / 21.7), 14 x 10,000 12.8 / 12.5, 64 x 2064 9.6 / 9.2, 300 x
// 30,000 21.6 / 22.1; fp32 64 x 30,000 20.1 / 19.6, 64 x 10,000 13.1 / 12.7, with the admissible set 17.8 / 17.2, 300 x 30,000 23.1 / 23.3.
constexpr bool pace_needed(int64_t N, int units) { return N > units; }

// Token-DiFR alone, fp32: waves per SIMD, 8 or the compiler's choice (1), which holds seven, with the rank six.  Eight cost scalar registers
// (104 spilled to vector lanes with the rank, 7 without) and are worth it where the rows fit at once with them only, where there are many rows that
// are not long, and where a row is its set-up alone.  us with the compiler's choice / eight: 1200 x 30,000 with the rank 30.8 / 33.1,
// 1600 x 128,256 134.5 / 135.7, with the rank 155.0 / 138.9, 1600 x 2048 with the rank 11.5 / 11.9, 2048 x 128,256 176 / 161 and 174 / 162, 2048 x 9000
// 22.1 / 20.9, 2304 x 128,256 189 / 195 and 191 / 199, 2304 x 9000 with the rank 25.6 / 26.7, 4500 x 128,256 349 / 353, 16,000 x 4000 with
// the rank 92.6 / 90.6, 10,516 x 30,000 207.6 / 202.4, 10,516 x 78,058 508 / 516, 10,516 x 1000 37.7 / 34.6, 2304 x 1600 14.3 / 14.8.
constexpr int gumbel_f32_waves(int64_t N, int units, bool rank, int64_t V)
{
    const int64_t fit = (int64_t)units * 8;
    const bool fit_only_so = N > (int64_t)units * (rank ? 6 : 7) && N <= fit && (!rank || V >= 8192);
    return fit_only_so || (2 * N > 5 * fit && V < 65536) || V < 1024 ? 8 : 1;
}

// Token-IPT-DiFR: whether a wave has three vectors in flight beside the one in use, and not one.  Where the rows are few it is what keeps the
// memory busy, where many share it they get in each other's way; a row of a few rounds ends before it pays.  us with one / three, every call
// on rows of its own (700 MB in all): bf16 64 x 9000 (4 rounds) 6.78 / 6.89, 64 x 16,000 (7) 8.05 / 7.61, 300 x 30,000 (14) 12.3 / 10.5, 700 x
// 128,256 44.3 / 36.8; fp32 64 x 4000 (3) 5.74 / 5.92, 64 x 9000 (8) 8.05 / 7.27.  By rows, 128,256 bf16: 1024 45.6 / 42.7, 1500 58.5 / 61.
constexpr bool ipt_deep(int64_t N, int resident, int64_t rounds) { return 2 * N <= resident && rounds >= 6; }

// Token-IPT-DiFR without the token: idle LDS per workgroup that keeps a compute unit at seven or six of the eight that fit, if the launch's
// last generation of rows is fuller then; a generation that starts with a few rows left takes as long as a full one.  (Five as well: 2304 x
// 128,256 96 us for 98, but 5000 x 30,000 58 for 53.)  Rows of fewer than eight rounds are set-up and latency in good part, and eight are better
// whatever the last generation is like; up to 24 rounds they are where there are more than two and a half generations.  us with eight /
// seven / six: bf16 2304 x 128,256 109 / 103 / 98, 4500 185 / 176 / 171, 2304 x 30,000 (14 rounds) 29.9 / 28.9 / 28.1, 9000 x 30,000 92.2 / 94.6 /
// 94.8, 4500 x 16,000 (7) 30.3 / 31.0 / 31.5, 9000 x 9000 38.9 / 41.3 / 44.4, 9000 x 1000 21.6 / 22.4 / 23.8; fp32 2304 x 30,000 53.9 / 51.7 / 49.3,
// 2304 x 16,000 (15) 30.7 / 30.0 / 29.4, 2304 x 9000 (8) 19.2 / 18.8 / 19.0, 9000 x 9000 58.7 / 60.2 / 61.9.
constexpr unsigned ipt_idle_lds(int64_t N, int units, int per_unit, int64_t rounds)
{
    constexpr int kFit = 8, kLeast = 6, kLdsOfUnit = 160 * 1024;  // (gfx950; the figures are for eight)
    const int64_t fit = (int64_t)units * kFit;
    if (per_unit != kFit || N <= fit || rounds < 8 || (rounds < 24 && 2 * N > 5 * fit)) return 0;
    int best = kFit;
    int64_t best_places = 0;
    for (int p = kFit; p >= kLeast; --p) {
        const int64_t at_once = (int64_t)units * p, places = (N + at_once - 1) / at_once * p;
        if (p == kFit || places < best_places) {
            best = p;
            best_places = places;
        }
    }
    return best == kFit ? 0u : (unsigned)(kLdsOfUnit / best - 1024);
}

}  // namespace difr
