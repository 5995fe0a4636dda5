// Runs csrc/team_join.h on threads (test_team_join.py): a thread stands for a compute unit, which runs
// one workgroup at a time and takes the next that may run there when that one has left.
//
//   team_join PATIENCE GIVE_UP   looks at the team's size before it is closed / before the wait ends
#include <sched.h>
#include <stdio.h>
#include <stdlib.h>
#include <mutex>
#include <set>
#include <thread>
#include <vector>
#include "team_join.h"

struct Memory {
    unsigned load(const unsigned *p) const { sched_yield(); return __atomic_load_n(p, __ATOMIC_SEQ_CST); }
    void store(unsigned *p, unsigned v) const { __atomic_store_n(p, v, __ATOMIC_SEQ_CST); }
    unsigned add(unsigned *p, unsigned v) const { return __atomic_fetch_add(p, v, __ATOMIC_SEQ_CST); }
    unsigned set_bits(unsigned *p, unsigned v) const { return __atomic_fetch_or(p, v, __ATOMIC_SEQ_CST); }
    int swap_if(int *p, int from, int to) const { __atomic_compare_exchange_n(p, &from, to, false, __ATOMIC_SEQ_CST, __ATOMIC_SEQ_CST); return from; }
    void settle() const {}
};

struct Launch {
    int die = -1;
    unsigned joined = 0, arrived = 0, members = 0, through = 0;
    unsigned most = 0;
    bool any_die = false;
    std::set<unsigned> numbers;
    unsigned size = 0;
    int gave_up = 0, wrong = 0;
};

static const int DIES = 2, UNITS = 4;                    // compute units a die
static unsigned patience, give_up;

// order[d]: the launches whose workgroups die d is given, in that order
static bool run(std::vector<Launch> &launches, const std::vector<std::vector<int>> &order, const char *what)
{
    std::mutex guard;
    std::vector<size_t> next(DIES, 0);
    std::vector<std::thread> units;
    for (int u = 0; u < DIES * UNITS; ++u)
        units.emplace_back([&, u]() {
            const int die = u / UNITS;
            for (;;) {
                Launch *l;
                {
                    std::lock_guard<std::mutex> hold(guard);
                    if (next[die] == order[die].size()) return;
                    l = &launches[order[die][next[die]++]];
                }
                unsigned number = 0, size = 0;
                const int mine = join_team(Memory{}, TeamWords{&l->die, &l->joined, &l->arrived, &l->members}, die, l->any_die,
                                           DIES * UNITS, l->most, patience, give_up, &number, &size);
                if (mine >= 0) {                         // a barrier over the team, in the place of its work
                    Memory{}.add(&l->through, 1u);
                    unsigned looks = 0;
                    while (Memory{}.load(&l->through) < size && ++looks <= 10u * give_up) {}
                    if (looks > 10u * give_up) { std::lock_guard<std::mutex> hold(guard); ++l->wrong; }
                }
                std::lock_guard<std::mutex> hold(guard);
                if (mine == -2) ++l->gave_up;
                if (mine >= 0) {
                    if (l->size != 0 && l->size != size) ++l->wrong;
                    l->size = size;
                    if (!l->numbers.insert((unsigned)mine).second || (unsigned)mine >= size) ++l->wrong;
                }
            }
        });
    for (std::thread &t : units) t.join();
    bool good = true;
    for (const Launch &l : launches) {
        printf("%s: %u members, %d gave up, %d wrong\n", what, l.size, l.gave_up, l.wrong);
        good = good && l.size > 0 && l.numbers.size() == l.size && l.gave_up == 0 && l.wrong == 0;
    }
    return good;
}

int main(int argc, char **argv)
{
    if (argc != 3) return 2;
    patience = (unsigned)atoi(argv[1]);
    give_up = (unsigned)atoi(argv[2]);
    const std::vector<int> own(UNITS, 0);
    bool good = true;
    const unsigned looks = patience;
    patience = give_up;                                  // (however late a thread starts: all of them are waited for)
    for (unsigned most : {8u, 3u})
        for (bool any : {true, false}) {
            std::vector<Launch> one(1);
            one[0].any_die = any;
            one[0].most = most;
            good = run(one, {own, own}, "alone") && good;
            const unsigned all = any ? DIES * UNITS : UNITS;
            good = one[0].size == (all < most ? all : most) && good;
        }
    patience = looks;
    {
        // both span the dies, and each gets half of every die
        std::vector<Launch> two(2);
        for (Launch &l : two) { l.any_die = true; l.most = 8; }
        const std::vector<int> half = {0, 0, 1, 1, 0, 0, 1, 1};
        good = run(two, {half, half}, "halves") && good;
    }
    {
        // both want one die, and each has another one full
        std::vector<Launch> two(2);
        for (Launch &l : two) l.most = 8;
        good = run(two, {{0, 0, 0, 0, 1, 1, 1, 1}, {1, 1, 1, 1, 0, 0, 0, 0}}, "a die each") && good;
    }
    return good ? 0 : 1;
}
