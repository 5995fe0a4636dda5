// Deals tasks of csrc/pair_tasks.h out on the CPU (test_pair_tasks.py): wavefronts take turns at random, and every task has
// to be done once, whoever is slow and whoever leaves.  And there are enough tasks, also where few pairs fit.
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
        // places for `first` workgroups or fewer; later ones take turns with others or not, and how readily the first ones leave differs
        const int later = upto(2) ? first + upto(upto(1) ? 10 : 300) : 0, places = 1 + upto(first - 1), each = 1 + upto(3), ready = upto(3);
        std::vector<int> none(MF_PAIR_QUEUES, 0), begun(MF_PAIR_QUEUES, 0), leaves(first + later, 0), waves_of(first + later, 0);
        struct Wave { int workgroup, task, left; };
        std::vector<Wave> busy;
        int launched = 0, here = 0;
        const auto taken = [&](int queue) { return pair_task_taken(queue, counter[queue]++, first, waves); };
        while (true) {
            while (here < places && launched < first + later) {
                const int w = launched++, queue = pair_queue(w, first);
                if (w >= first && none[queue]) continue;
                if (w >= first) ++begun[queue];
                for (int v = 0; v < waves; ++v)
                    busy.push_back({w, w < first ? pair_task_by_place(w, v, first) : taken(queue), pair_takes_turns(w, first, later) ? each : 1 << 30});
                waves_of[w] = waves;
                ++here;
            }
            if (busy.empty()) break;
            const size_t k = rng() % busy.size();
            Wave wave = busy[k];
            const int queue = pair_queue(wave.workgroup, first);
            bool ends = wave.task >= tasks;
            if (ends) none[queue] = 1;
            else {
                ++done[wave.task];
                ends = --wave.left == 0 || leaves[wave.workgroup];
                if (!ends && wave.left > 1 << 20 && later > 0 && pair_may_leave(wave.workgroup, first, later, begun[queue]) && upto(3) < ready)
                    ends = leaves[wave.workgroup] = 1;
                if (!ends) wave.task = taken(queue);
            }
            if (!ends) busy[k] = wave;
            else {
                busy[k] = busy.back();
                busy.pop_back();
                if (--waves_of[wave.workgroup] == 0) --here;
            }
        }
        for (int t = 0; t < tasks; ++t)
            if (done[t] != 1) {
                printf("case %d: %d and %d workgroups of %d, task %d of %d done %d times\n", c, first, later, waves, t, tasks, done[t]);
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
