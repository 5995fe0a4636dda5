// Runs csrc/team_steps.h on threads (test_team_steps.py): a thread stands for a workgroup, and one of them is held up
// after every barrier until all others have come to the next one.  At each barrier all have to say that they
// are in the same place.
//
//   team_steps RULE     "labels", "stages": as the header has them; "labels read late": the count of rows read behind the
//                       barrier; "stages begin anew": every stage clears the whole ring; "cleared when read":
//                       the member that clears does so with a count it has just read
#include <stdio.h>
#include <string.h>
#include <condition_variable>
#include <mutex>
#include <thread>
#include <vector>
#include "team_steps.h"

// The barrier.  `apart`: two members came to it from different places; everybody leaves then.
struct Meeting {
    std::mutex guard;
    std::condition_variable turned;
    int members, late;                  // late: the member that is held up
    int waiting = 0, number = 0, place = 0;
    bool apart = false;

    Meeting(int m, int l) : members(m), late(l) {}

    bool barrier(int who, int where)
    {
        std::unique_lock<std::mutex> hold(guard);
        if (waiting == 0) place = where;
        else if (place != where) apart = true;
        const int mine = number;
        if (++waiting == members) { waiting = 0; ++number; }
        turned.notify_all();
        turned.wait(hold, [&]() { return apart || number != mine; });
        if (who == late) turned.wait(hold, [&]() { return apart || waiting == members - 1; });
        return !apart;
    }
    void leave()
    {
        std::lock_guard<std::mutex> hold(guard);
        if (--members == waiting && waiting > 0) { waiting = 0; ++number; }
        turned.notify_all();
    }
};

struct Shared {
    unsigned long long rows = 0;
    int ring[STEP_RING] = {0, 0, 0, 0};
};

// places a barrier can be at
enum { SERVED = 1, MAKING = 100, OFFERED = 1000, BIDDING = 2000, SIDE_DONE = 3000, SETTLED, PHASE, PROVING };

struct Member {
    Meeting &meeting;
    Shared &shared;
    int number, place = 0, tree = 0, trees;

    unsigned long long rows_looked_at() { return __atomic_load_n(&shared.rows, __ATOMIC_SEQ_CST); }
    void add_rows_looked_at(int n) { place = OFFERED; __atomic_fetch_add(&shared.rows, (unsigned long long)n, __ATOMIC_SEQ_CST); }
    bool bidders_left() const { return tree < trees; }
    bool barrier() { return meeting.barrier(number, place); }
};

template <class Team, class Clear, class Make, class Offer>
static bool labels_read_late(Team &team, bool &by_column, bool must, unsigned long long most, const Clear &clear, const Make &make, const Offer &offer)
{
    clear();
    if (!team.barrier()) return false;
    if (!team.bidders_left()) return true;
    if (!by_column && (must || team.rows_looked_at() > most)) {
        if (!make()) return false;
        by_column = true;
    }
    team.add_rows_looked_at(offer(by_column));
    return team.barrier();
}

static bool serve_trees(Member &m, bool read_late, unsigned long long most, int *made_for)
{
    bool by_column = false;
    const auto clear = [&]() { m.place = SERVED; };
    const auto make = [&]() {
        for (int k = 0; k < 4; ++k) {
            m.place = MAKING + k;
            if (!m.barrier()) return false;
        }
        *made_for = m.tree;
        return true;
    };
    const auto offer = [&](bool columns) { return columns ? 0 : 2 + m.number; };
    while (m.tree < m.trees) {
        ++m.tree;
        if (!(read_late ? labels_read_late(m, by_column, false, most, clear, make, offer)
                        : labels_of_served_tree(m, by_column, false, most, clear, make, offer)))
            return false;
    }
    return true;
}

// The stages of a launch as core.hip goes through them, with nothing but their counts: what each step hands on, of how
// many are left, decides which barriers come next.  Member 0 is the one that clears.
struct Stages {
    Member &m;
    bool anew, when_read;
    unsigned step = 0;
    std::vector<int> &seen;

    int *ring() { return m.shared.ring; }
    void add(int n) { __atomic_fetch_add(&ring()[step_fills(step)], n, __ATOMIC_SEQ_CST); }
    void set(unsigned at, int n) { if (m.number == 0) __atomic_store_n(&ring()[at], n, __ATOMIC_SEQ_CST); }
    int read()
    {
        ++step;
        seen.push_back(__atomic_load_n(&ring()[step_reads(step)], __ATOMIC_SEQ_CST));
        if (when_read) set(step_reads(step), 0);
        return seen.back();
    }
    void clear_ahead() { set(step_clears(step), 0); }
    void begin(int lines)
    {
        if (!anew) return;
        step = 0;
        for (unsigned q = 0; q < STEP_RING; ++q) set(q, q == 0 ? lines : 0);
    }
    bool at(int where) { m.place = where; return m.barrier(); }

    // a side: a quarter of the bidders is handed on by every step
    bool side(int &count, int stop)
    {
        if (!at(PHASE) || !at(PHASE + 1)) return false;
        for (int k = 0; count > stop; ++k) {
            clear_ahead();
            add(count / 16);
            if (!at(BIDDING + k)) return false;
            count = read();
        }
        return true;
    }
    bool run(int lines, int phases)
    {
        for (int ph = 0; ph < phases; ++ph) {
            const int stop = ph == phases - 1 ? 0 : 24 >> ph;
            int count = lines;
            begin(lines);
            if (!side(count, stop)) return false;
            const int left = count;
            begin(0);
            clear_ahead();
            if (!at(SIDE_DONE)) return false;
            if (anew) __atomic_fetch_add(&ring()[0], 2 + 4 * ph, __ATOMIC_SEQ_CST);
            else add(2 + 4 * ph);
            if (!at(SIDE_DONE + 10)) return false;
            if (anew) { step = STEP_RING - 1; count = read(); step = 0; }
            else count = read();
            if (left > 0 && count > stop && !at(SETTLED)) return false;
            if (count > stop && !side(count, stop)) return false;
            if (left == 0 && count == 0) {              // a proof: rounds with fewer and fewer rows
                begin(0);
                count = lines;
                if (!at(PHASE)) return false;
                for (int round = 0; count > 0 && round < 2 + ph; ++round) {
                    clear_ahead();
                    add(count / 16);
                    if (!at(PROVING + round)) return false;
                    count = read();
                }
            }
        }
        return true;
    }
};

int main(int argc, char **argv)
{
    if (argc != 2) return 2;
    const bool read_late = !strcmp(argv[1], "labels read late"), labels = read_late || !strcmp(argv[1], "labels");
    const bool anew = !strcmp(argv[1], "stages begin anew"), when_read = !strcmp(argv[1], "cleared when read");
    const bool stages = anew || when_read || !strcmp(argv[1], "stages");
    if (!labels && !stages) return 2;
    const int members = 4, trees = 6;
    int together = 0, apart = 0, wrong = 0;
    for (int late = 0; late < members; ++late)
        for (int most = 0; most < 80; ++most) {
            Meeting meeting(members, late);
            Shared shared;
            std::vector<int> made_for(members, 0);
            std::vector<std::vector<int>> seen(members);
            std::vector<std::thread> team;
            for (int k = 0; k < members; ++k)
                team.emplace_back([&, k]() {
                    Member m{meeting, shared, k};
                    m.trees = trees;
                    if (labels) (void)serve_trees(m, read_late, (unsigned long long)most, &made_for[k]);
                    else {
                        Stages launch{m, anew, when_read, 0, seen[k]};
                        (void)launch.run(64 + 16 * most, 4);
                    }
                    meeting.leave();
                });
            for (std::thread &t : team) t.join();
            if (meeting.apart) { ++apart; continue; }
            ++together;
            // a tree adds 2 + 3 + 4 + 5 rows; the last one places the last bidder, and nobody asks for labels
            int expect = labels ? most / 14 + 2 : 0;
            if (expect >= trees) expect = 0;
            for (int k = 0; k < members; ++k) wrong += made_for[k] != expect || seen[k] != seen[0];
        }
    printf("%d together, %d apart, %d wrong\n", together, apart, wrong);
    return apart == 0 && wrong == 0 ? 0 : 1;
}
