// How the pair kernel's work is cut into tasks and dealt out (score.hip).
//
// A task is 32 columns beside some rows.  Tasks are numbered by rows first, so that the two thousand under way share a
// few rows' projections and every row of the matrix is written within a short time, and dealt out in turn
// to MF_PAIR_QUEUES groups of workgroups, each with a counter of its own: the first ones by the wavefront's place, then
// whoever is done takes its group's next.  (Two thousand wavefronts that end together at one counter waited 20 us
// for it: 1024 x 1024 54 / 44 us.)
//
// A workgroup takes its compute unit whole (H = 128: all vector registers).  What another stream has to run beside a pass of 21 ms must
// not wait for its end, so of a long launch one workgroup in PAIR_TURN leaves after PAIR_STAY_ROWS rows a wavefront (0.3 ms), and one
// of those launched behind it takes its place; whatever else waits for a compute unit comes in between.  The others stay:
// they need one set-up, and they are not held up by the order in which workgroups are dispatched.
// That is not enough for launches whose workgroups wait for one another on one die (core.hip): they keep the
// compute units that change hands, and no later workgroup of this launch begins there.  Whoever sees that nobody has begun in its queue, two of
// which belong to a die, for PAIR_PATIENCE times as long as its longest task leaves as well, as long as enough workgroups are to come.  The last ones to
// come stay until nothing is left, so every task is done whoever leaves.
// Calls of a second context beside passes over 20,000 x 20,000 pairs, median ms; a workgroup per tile / workgroups that all stay / as it is:
// 10^6 additions 0.10 / 23 at most / 0.18, a 64 x 64 round 0.70 / 21 / 1.4, a round of 777 x 1501 12 / 72 to 95 / 26, matchings of 500 x 700
// 4.9 / 45 / 10 to 13 and 3000 x 3000 6.0 / 27 / 8 to 11; the pass alone 22.8 / 21.3 / 21.5 ms, 20,000 x 40,000 6.9 / 5.8 / 5.9.  Tried: all of them leave
// after 64, 128, 256, 512 rows: pass 22.2, 22.0, 21.8, 21.8, 777 x 1501 11, 20, 34, 57; one in 8: 777 x 1501 31, matching of 500 x 700 20; one in 2: 20,000 x
// 40,000 0.3 ms more.
//
// No dependence on the device: tests/pair_tasks.cpp deals tasks out on the CPU.
#pragma once
#include <math.h>

#if defined(__HIPCC__)
#define MF_PAIR_FN __host__ __device__ __forceinline__
#else
#define MF_PAIR_FN inline
#endif

// Counters of a launch, and words from one to the next: a line of 128 bytes each.  Its words: the counter; whether nothing is left;
// workgroups beyond the first that have begun; when the last one did.
constexpr int MF_PAIR_QUEUES = 16, MF_PAIR_QUEUE_STEP = 32;

// Rows of a task, a power of two up to 64.  row_blocks: rows beside blocks of 32 columns that there are to score, as many
// as fit in memory order; units: compute units.
//
// A task costs what its rows cost and its columns' projections, as long as c rows; at the end of the launch a SIMD waits
// for about k of a task.  With R rows for each of the device's SIMDs that is R (1 + c / t) + k t for t rows, least at the square
// root of R c / k, and c / k fits as 2.7 for 128 hidden units and 4 for 64, where rows take a quarter as long: of 2, 4, 8, ... 64 rows
// the rule takes the fastest or one within 6 % of it at 25 sizes from 64 x 64 to 20,000 x 40,000.  It counts what fits: a rule that had
// every block of columns for a task took 64 rows where nine pairs in ten do not fit and most wavefronts had none
// (pair kernel, us, before / now: 1000 x 2000 91 / 36, 2000 x 4000 182 / 92, 12,000 x 300 181 / 78; 1000 x 2000 where three in four fit 154 / 138).
MF_PAIR_FN int pair_task_rows(int hidden, float row_blocks, float units)
{
    const float share = row_blocks / (4.0f * units) * (hidden == 128 ? 2.7f : 4.0f);
    int bits;
    frexpf(share, &bits);               // share < 2^bits
    bits >>= 1;
    return bits < 1 ? 2 : bits > 6 ? 64 : 1 << bits;
}

// first: workgroups that begin with the launch.
MF_PAIR_FN int pair_queue_bits(int first) { return first < MF_PAIR_QUEUES ? 0 : 4; }
MF_PAIR_FN int pair_queues(int first) { return 1 << pair_queue_bits(first); }
MF_PAIR_FN int pair_queue(int workgroup, int first) { return workgroup & (pair_queues(first) - 1); }

// The task that a wavefront of such a workgroup begins with, and the one that the taken-th to take from the counter goes on with.
MF_PAIR_FN int pair_task_by_place(int workgroup, int wave, int first)
{
    const int bits = pair_queue_bits(first), queue = pair_queue(workgroup, first), team = (first - queue + pair_queues(first) - 1) >> bits;
    return queue + (((workgroup >> bits) + team * wave) << bits);
}
MF_PAIR_FN int pair_task_taken(int queue, int taken, int first, int waves)
{
    const int bits = pair_queue_bits(first), team = (first - queue + pair_queues(first) - 1) >> bits;
    return queue + ((team * waves + taken) << bits);
}

// One workgroup in PAIR_TURN, 32 neighbours at a time: they are dispatched to the eight dies in turn and on a die to its four
// shader engines, in this order, so as many leave each engine (where they left two of the four, the next ones in line waited for a place
// in the others, and no compute unit changed hands).
constexpr int PAIR_TURN = 4, PAIR_TURN_GROUP = 32, PAIR_STAY_ROWS = 64, PAIR_PATIENCE = 3;

// Tasks a wavefront from which a launch is long (2 ms for H = 128): up to there all stay.
constexpr int PAIR_LONG = 8;

// Workgroups that are launched beyond the first: half as many as do all that there may be to do, 64 rows a wavefront, and the last ones, as many as the first.
MF_PAIR_FN long long pair_later(long long tasks, long long first_waves, int waves, int rows, int blocks, int first)
{
    return tasks > PAIR_LONG * first_waves ? first + (long long)rows * blocks / (2 * PAIR_STAY_ROWS * waves) : 0;
}

// Whether a workgroup leaves after PAIR_STAY_ROWS rows.
MF_PAIR_FN bool pair_takes_turns(int workgroup, int first, int later)
{
    return workgroup < first ? later > 0 && workgroup / PAIR_TURN_GROUP % PAIR_TURN == PAIR_TURN - 1 : workgroup < later;
}

// Whether a workgroup that stays may leave all the same.  begun: of the later ones of its queue.
MF_PAIR_FN bool pair_may_leave(int workgroup, int first, int later, int begun)
{
    return workgroup < first && pair_queues(first) * begun < later - first;
}
