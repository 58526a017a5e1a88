// How many slots a selection's buffer has, and how many stream rounds it goes without a barrier (topn.hpp).  Plain host code as well:
// the test of the schedule runs it on rows that rise along the vocabulary.
#pragma once

namespace difr {

constexpr int kTopTrigger = 512;                     // a compaction is due at the latest when this many slots are used
constexpr int kTopCapSmall = kTopTrigger + 64 * 8;   // slots per buffer: the trigger plus one round of one wave
constexpr int kTopCapMid = kTopTrigger + 128 * 8;    // ... for the larger selections of the likelihood kernel, which has two buffers
constexpr int kTopCapBig = kTopTrigger + 256 * 8;    // ... plus one round of the whole workgroup
constexpr int kTopCapOne = kTopCapBig + 256;         // ... and, in the filtered Token-IPT-DiFR kernel, what the first round may leave waiting
constexpr int kTopEpoch = 8;   // stream rounds per epoch of the filtered Token-IPT-DiFR kernel (measured: 4 and 16 are both slower)
constexpr int kLikEpoch = 16;  // ... and of the likelihood kernel: vectors that trip a test only queue up there, so a threshold that is an
                               // epoch old costs little (measured: 16, 24 and 32 alike, 8 slower by 4%)

// The epoch that begins with round `round`.  The threshold moves only between epochs, and while little of the row has been seen it
// moves a lot: after the first, and up to round `settled`, none is longer than what lies behind it.  (One longer than that tests rows that
// rise along the vocabulary against a threshold from far below them, and a buffer that runs full costs the row a second, slow pass: 1024 rows of 8
// rounds whose logits rise by 0.5 a round, s = 64, k = 50: 200 us with epochs of 2 and 6 rounds and first thresholds of y from the first
// round alone; 59 so.)
constexpr int selection_epoch(int round, int first, int settled, int full)
{
    const int len = round > first ? round : first;
    return len < settled && len < full ? len : full;
}

// Rounds in the first epoch, and `settled`; `wide` is 1 for bf16 and 2 for fp32, whose rounds have half as many entries.
//
// Likelihood kernel, us with one / two rounds for the small buffers: 4096 x 9000, k = 50, s = 16 127.5 / 125.7, s = 64 160.9 / 158.6.  The larger
// selections take one, since their first thresholds let up to a sixth of a round through, and are not settled before round 16: with k = 200 a
// few rows in a thousand fill 1536 slots in rounds 8 to 23.  (Epochs of at most two thirds of what lies behind would keep rows that rise by 0.3 a
// round from filling them, 4096 x 32,000 with k = 200 1280 / 557, but cost ordinary rows 3 to 7%: 2048 x 50,000 194 / 206.)
constexpr int likelihood_first_epoch(int cap, int wide) { return (cap == kTopCapSmall ? 2 : 1) * wide; }
constexpr int likelihood_settled(int cap, int wide) { return (cap == kTopCapSmall ? 8 : 16) * wide; }
// Filtered Token-IPT-DiFR kernel (`primed`: its threshold is from rounds spread over the row, and not from the first alone), k = 50, bf16, us
// with 2 / 4 / 8 rounds: 4096 x 9000 54.9 / 53.0 / 52.4, 2048 x 16,424 40.4 / 38.9 / 37.8; with eight, rows whose rounds 1 to 7 lie 3
// above the others run full, for k of more than 32.  More than 64 logits: two rounds fit their buffer after such a threshold (four of fp32, which have
// half the entries, for up to 128), one without.  (Vectors of the first round wait for the second where fewer than 64 of a wave's pass; for k = 256
// they hold a quarter of its entries or more in one row of forty, three eighths in one of 13,000.  1024 x 128,256, rounds 1 to 7 higher by 3:
// 283 us with kTopCapBig slots, 117 with kTopCapOne, five workgroups to a compute unit either way; ordinary rows the same.)
constexpr int filtered_first_epoch(int cap, int n, bool primed, int wide)
{
    return cap == kTopCapSmall ? (n <= 32 ? 8 : 2 + 2 * wide) : (primed && (wide == 1 || n <= 128) ? 2 : 1) * wide;
}

}  // namespace difr
