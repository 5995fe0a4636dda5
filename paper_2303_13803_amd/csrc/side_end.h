// When a side of a phase that only prepares prices ends with bidders left over (run_side in auction.hip, run_bids in core.hip).
//
// What such a side leaves undone the next phase finds: columns that nobody holds and that have to come down to price 0, all others
// with them, one of the next phase's smaller epsilons at a time.  A few of those a search places at once, however far they have to come;
// fifty of them bid.  With 900 rows, 950 columns and weights of 2^29 to 2^29 + 3 the phases on lists ended both sides
// after 64 dependent steps: the fifty columns too many were left over every time, prices stayed where the
// first phase had driven them, and the first phase that runs to the end, at 2531, was to bring them down from
// 1.8e10: billions of bids.  So such columns bid until at most `stop` are left (columns_may_wait): every such side takes some 25
// bids a line.  Other sides on lists end early, at every size: 2946 x 2946 such weights, where no column is too many, 11 ms, 24 where sides go on.
// From phase_tail_from lines on all sides on lists do, for what it saves: C4's 20,000 x 20,000, seeds 63, 83 and 97, auctions of 49, 49 and 63 ms
// that take 73, 79 and 83 where columns bid on (seed 81 116 / 37 ms, sixteen ordinary ones 15.4 / 14.6).  Prices that are far off are then left to searches
// (stuck_after): 8200 x 8240 such weights 0.9 s, 8200 x 8300, where more columns are too many than may be left over, 0.08 s.
//
// No dependence on the device: tests/side_end.cpp counts the bids of such ladders on the CPU.
#pragma once

#if defined(__HIPCC__)
#define MF_END_FN __host__ __device__ __forceinline__
#else
#define MF_END_FN inline
#endif

// How many of a solve's last phases run until nobody is left to bid.  asked: so many, whatever the number (0: nobody has).
// While nobody has: of a ladder of at most five phases (weights of a few hundred levels) the last three; the first complete one would be the
// first or second, most of its work is done again by the next, and lists do not reach far enough for it yet.  Four / three, ms, four or
// six seeds: 8-bit rounds of 20,000 x 40,000 14.8 / 11.6, 9000 x 20,000 8.6 / 7.1, 4000 x 9000 5.0 / 4.7, 600 x 1500 1.39 / 1.11, 300 x 700 0.69 / 0.69; uniform 8-bit
// matrices 12,000 x 12,000 21.5 / 7.7, 6000 x 6000 9.7 / 8.8, 3000 x 5000 2.68 / 2.69; with prefixes of a half 3613 x 3613 33 / 6.7; thresholds of 2612 x 2653
// 6.6 / 2.4, four levels of 750 x 750 9.5 / 3.8.  Some lose a little (uniform 3000 x 3000 3.46 / 3.96, 600 x 600 2.28 / 2.59), longer ladders more
// (4096 x 8192 of 2^24 levels 7.3 / 8.0).
constexpr int PHASES_TO_THE_END = 4;
MF_END_FN int phases_to_the_end(int asked, bool warm, int phases) { return asked ? asked : !warm && phases <= 5 ? 3 : PHASES_TO_THE_END; }

// Bidders that may be left over, with `after` phases to come of which the last `keep` run to the end: `stop`, times `growth` for every
// phase further from those, at least `search` (so many are placed by a search: for the phases that have to finish), at most one line in 64.
MF_END_FN int bidders_left_over(int after, int keep, long long stop, int growth, int search, int lines)
{
    if (after < keep) return 0;
    for (int k = keep; k < after && stop < lines; ++k) stop *= growth;
    if (stop > 0 && stop < search) stop = search;
    return (int)(stop < lines / 64 ? stop : lines / 64);
}

// Dependent steps after which the side (0: rows bid, 1: columns) ends all the same (0: no limit).  sides: a bit each.
MF_END_FN long long steps_of_side(int side, int sides, long long steps, int from, int lines) { return (sides >> side & 1) && lines >= from ? steps : 0; }

// Whether columns that bid may be left to the next phase after that many steps, which on lists count while at most `few` (64) of them are left.  With no more too
// many (than rows without one, and `stop`) than a search places, a search brings them down; with more than `few`, some have come down to 0 by
// then, and all others with them.  (Rounds of 1015 x 1420 2.6 ms so, 3.0 where all sides with columns too many go on, 106 x 109 1.2 and 1.5.)
MF_END_FN bool columns_may_wait(int columns, int rows, int stop, int search, int few)
{
    const int too_many = columns - rows;
    return too_many <= (stop > search ? stop : search) || too_many > few;
}

// Whether a side with `left` bidders ends, of which `stop` may be left over, after `followed` dependent steps.
MF_END_FN bool side_ends(int left, int stop, long long steps, long long followed) { return left <= stop || (stop > 0 && steps > 0 && followed >= steps); }

// Dependent steps without an eighth fewer bidders after which a search takes as many of them as it can, however many there are:
// they outbid each other by an epsilon at a time, and may have as far to go as prices reach.  (Twenty columns too many where the phases before
// might leave 23 over, 1500 x 1520 weights of 2^29 to 2^29 + 3: 2e10 at an epsilon of 1e5.)
MF_END_FN long long stuck_after(long long path_after) { return 512 + 16 * (path_after < 1ll << 40 ? path_after : 1ll << 40); }
