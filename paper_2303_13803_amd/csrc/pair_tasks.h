// How the pair kernel's work is cut into tasks and dealt out (score.hip).
//
// A task is 32 columns beside some rows.  Tasks are numbered by rows first, so that the two thousand under way share a
// few rows' projections and every row of the matrix is written within a short time, and dealt out in turn
// to MF_PAIR_QUEUES groups of workgroups, each with a counter of its own: the first ones by the wavefront's place, then
// whoever is done takes its group's next.  (Two thousand wavefronts that end together at one counter waited 20 us
// for it: 1024 x 1024 54 / 44 us.)
//
// No dependence on the device: tests/pair_tasks.cpp deals tasks out on the CPU.
#pragma once

#if defined(__HIPCC__)
#define MF_PAIR_FN __host__ __device__ __forceinline__
#else
#define MF_PAIR_FN inline
#endif

// Counters of a launch, and words from one to the next: a line of 128 bytes each.
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
    int t = 2;
    while (t < 64 && share > (float)(2 * t * t)) t *= 2;
    return t;
}

// first: workgroups that begin with the launch.
MF_PAIR_FN int pair_queues(int first) { return first < MF_PAIR_QUEUES ? 1 : MF_PAIR_QUEUES; }

// The task that a wavefront of such a workgroup begins with, and the one that the taken-th to take from the counter goes on with.
MF_PAIR_FN int pair_task_by_place(int workgroup, int wave, int first)
{
    const int queues = pair_queues(first), queue = workgroup % queues, team = (first - queue + queues - 1) / queues;
    return queue + queues * (workgroup / queues + team * wave);
}
MF_PAIR_FN int pair_task_taken(int queue, int taken, int first, int waves)
{
    const int queues = pair_queues(first), team = (first - queue + queues - 1) / queues;
    return queue + queues * (team * waves + taken);
}
