// Deals tasks of csrc/pair_tasks.h out on the CPU (test_pair_tasks.py): wavefronts take turns at random, and every task has
// to be done once, whoever is slow.  And there are enough tasks, also where few pairs fit.
//
//   pair_tasks CASES SEED     prints the first case in which a task was not done once, and ends with 1
#include <stdio.h>
#include <stdlib.h>
#include <random>
#include <vector>
#include "pair_tasks.h"

int main(int argc, char **argv)
{
    const int cases = argc > 1 ? atoi(argv[1]) : 1000;
    std::mt19937 rng(argc > 2 ? atoi(argv[2]) : 1);
    const auto upto = [&](int most) { return (int)(rng() % (unsigned)(most + 1)); };
    for (int c = 0; c < cases; ++c) {
        const int waves = upto(1) ? 8 : 4, first = 1 + upto(upto(1) ? 20 : 300), tasks = upto(upto(1) ? 50 : 6 * first * waves);
        std::vector<int> done(tasks, 0), counter(MF_PAIR_QUEUES, 0);
        struct Wave { int workgroup, task; };
        std::vector<Wave> busy;
        for (int w = 0; w < first; ++w)
            for (int v = 0; v < waves; ++v) busy.push_back({w, pair_task_by_place(w, v, first)});
        while (!busy.empty()) {
            const size_t k = rng() % busy.size();
            Wave &wave = busy[k];
            if (wave.task >= tasks) { wave = busy.back(); busy.pop_back(); continue; }
            ++done[wave.task];
            const int queue = wave.workgroup % pair_queues(first);
            wave.task = pair_task_taken(queue, counter[queue]++, first, waves);
        }
        for (int t = 0; t < tasks; ++t)
            if (done[t] != 1) {
                printf("case %d: %d workgroups of %d, task %d of %d done %d times\n", c, first, waves, t, tasks, done[t]);
                return 1;
            }
    }
    // In memory order: rows whose prefixes of columns that fit shrink, evenly or not.  With a dozen rows beside 32 columns for each of a
    // device's SIMDs there is a task for each.
    for (int c = 0; c < cases; ++c) {
        const int units = 256, n = 64 + upto(8000), m = 64 + upto(16000), kind = upto(2), part = 1 + upto(9);
        std::vector<int> fits(n);
        double feasible = 0;
        for (int i = 0; i < n; ++i) {
            const double x = 1.0 - (double)i / n, y = part / 10.0;
            fits[i] = (int)(m * (kind == 0 ? x * y : kind == 1 ? y : x > 1.0 - y ? x : 0.0));
            feasible += fits[i];
        }
        const float row_blocks = (float)feasible / (32.0f * n) + 0.5f;
        for (int hidden = 64; hidden <= 128; hidden += 64) {
            const int t = pair_task_rows(hidden, n * row_blocks, (float)units);
            long long tasks = 0;
            for (int i = 0; i < n; i += t) tasks += (fits[i] + 31) / 32;
            if (feasible / 32.0 >= 12.0 * 4 * units && tasks < 4 * units) {
                printf("%d x %d, %.0f pairs fit: %lld tasks of %d rows\n", n, m, feasible, tasks, t);
                return 1;
            }
        }
    }
    for (int hidden = 64; hidden <= 128; hidden += 64)
        for (float work = 1.0f; work < 1e12f; work *= 1.07f)
            for (int units : {1, 38, 256, 304}) {
                const int t = pair_task_rows(hidden, work, (float)units);
                if (t < 2 || t > 64 || (t & (t - 1)) || t < pair_task_rows(hidden, work / 2.0f, (float)units)) { printf("rows of a task: %d\n", t); return 1; }
            }
    return 0;
}
