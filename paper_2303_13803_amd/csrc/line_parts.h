// In how many parts wavefronts read whole lines together (Core::search and Core::refine in core.hip): each takes every so many-th slice of a line.
//
// Beginning on a part costs about a quarter of a slice (1.6 us): whose line it is and from what label.  Lines that end where their
// feasible prefix does are taken by as many wavefronts as there are for each: a wavefront for every slice that the longest
// might have looked 40 times at each of 27,000 prefixes of 4000 entries, 6.7 ms of a 20,000 x 40,000 round.  Lines that are all the same
// length have no empty slices, and there that rule has most wavefronts wait: of 256, 140 lines of twenty slices keep 140 busy twenty
// slices long and 300 lines all of them, then 44; in single slices and in threes it is 11 and 25 slices.  (That
// seldom is what a solve waits for: fifteen 20,000 x 20,000 rounds, among them the slow seeds, take the same within what runs differ.)
//
// No dependence on the device: tests/line_parts.cpp tries all numbers of lines.
#pragma once

#if defined(__HIPCC__)
#define MF_PARTS_FN __host__ __device__ __forceinline__
#else
#define MF_PARTS_FN inline
#endif

// In quarters of a slice, with `each` slices a part.  (Below 2^32: 2^20 lines of 2^10 slices and eight wavefronts.)
MF_PARTS_FN unsigned parts_take(unsigned slices, unsigned lines, unsigned waves, unsigned each)
{
    return ((slices + each - 1u) / each * lines + waves - 1u) / waves * (4u * each + 1u);
}

MF_PARTS_FN int parts_of_line(int slices, int lines, int waves, bool prefixes)
{
    if (prefixes) {
        const int most = waves / lines;
        return most < 1 ? 1 : most < slices ? most : slices;
    }
    int best = 1;
    unsigned least = parts_take(slices, lines, waves, 1);
    for (int each = 2; each < 2 * slices; each += each < 4 ? 1 : each) {      // 2, 3, 4, 8, ... and all of them
        const int now = each < slices ? each : slices;
        const unsigned take = parts_take(slices, lines, waves, now);
        if (take < least) { best = now; least = take; }
    }
    return (slices + best - 1) / best;
}
