// Which sub-tiles of 32 keys a workgroup of the few-rows attention (hr_attn_rows.hip) asks for, and from which lane it has their pages'
// addresses.  The kernel and a CPU test share it: every request is made, whether its sub-tile exists or not, so every one needs an address
// that is valid for the bytes it reads.
#pragma once

#include "hr_layout.h"

namespace hr {

constexpr int kSWaves = 6, kOWaves = 2, kRowsWaves = kSWaves + kOWaves;
constexpr int kSPW = 2;                          // sub-tiles per S wavefront and round: their S and K stay in registers
constexpr int kRoundSubs = kSWaves * kSPW;       // sub-tiles per round
constexpr int kVAhead = kRoundSubs / 2;          // sub-tiles whose V is on its way
static_assert(4 * kRoundSubs <= 64, "the pages of two rounds fit one lane each");

// A wavefront's lanes hold the pages of two rounds, `round` (an even one) and the next: lane l those of this sub-tile, behind the last
// one (own keys) that one's again
HR_HD int rows_lane_sub(int round, int lane, int n_sub) {
    const int j = (2 * round * kRoundSubs + lane) >> 1;
    return j < n_sub ? j : n_sub - 1;
}
// The lane that has page `side` of sub-tile j of a round
HR_HD int rows_page_lane(int round, int j, int side) { return 2 * ((round & 1) * kRoundSubs + j) + side; }
// Whether a wavefront fetches, in round r, the addresses of the pair of rounds behind r + 1
HR_HD bool rows_fetches_pages(int r, int rounds) { return !(r & 1) && r + 2 < rounds; }
// The round that is asked for where `round` would be, one past the last included.  Behind an even number of rounds the addresses are still
// those of the last two, documents' as a rule, whose fp8 pages are half as long as an absent sub-tile's request: the first of the two again
// (fetching the next pair's for it, 20 candidates of 512 + 32 keys, 0.5B shape: 1494 -> 1511 us a call)
HR_HD int rows_asked(int round, int rounds) { return round == rounds && !(rounds & 1) ? round - 2 : round; }

// sequences << 9 | blocks << 1 | last token only: one parameter word of the kernel.  A call that it does not hold stays with the chain kernel.
HR_HD bool rows_holds(int64_t n_seq, int64_t blocks) { return n_seq < (1 << 23) && blocks <= 0xFF; }

// Workgroups that read weights ahead: the launch is short, and 160 have read them sooner.  Whole calls, 0.5B shape, 128 / 160 / 192: 5 candidates
// 960 / 946 / 951 us, 20 candidates 1508 / 1486 / 1491, 23 candidates 1587 / 1549 / 1527; where the keys of the longest sequence are many or the
// codes are to be expanded they only take from the rows: 20 documents of 2048 tokens 1998 / 2005 / 2012, of 512 in an fp8 pool 1587 / 1591 / 1593.
constexpr int kRowsManyKeys = 640;
HR_HD int rows_warm_wgs(int max_keys, bool fp8) { return fp8 || max_keys >= kRowsManyKeys ? 128 : 160; }

}  // namespace hr
