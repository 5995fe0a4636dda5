// Puts what csrc/search_words.h publishes through every order of its memory accesses (test_search_words.py).
//
// Some wavefronts look at one row in the same step, each from the label its column had when that
// wavefront read it.  Every access is one operation on shared memory; the orders of two or three
// wavefronts' operations are all tried, and after each the pass over all columns must find nothing too
// long and nothing hidden.  With "stores" the minima are plain stores, and with "moved" a reading of a
// whole line counts whatever label the column has by then: both have to fail, or the orders tried
// would not be those that matter.
#include <stdint.h>
#include <stdio.h>
#include <string.h>
#include <vector>
#include "search_words.h"

typedef unsigned long long u64;

static const double FAR = 1.0e300;
static const u64 NEVER = ~0ull;
static const double PROFIT = 7.0, EPS = 1.0;

struct Words {
    double base, dropped, left;
    u64 expanded, read_from;
};

struct Op {
    double *real;
    u64 *whole;
    double d;
    u64 u;
};

// notes the operations instead of making them
struct Recorder {
    std::vector<Op> *ops;
    void set(double *p, double v) const { *p = v; }     // (by the pass over all columns, alone)
    void set(u64 *p, u64 v) const { *p = v; }
    void lower(double *p, double v) const { ops->push_back(Op{p, nullptr, v, 0}); }
    void lower(u64 *p, u64 v) const { ops->push_back(Op{nullptr, p, 0.0, v}); }
};

static void apply(const Op &op, bool stores)
{
    if (op.real) { if (stores || op.d < *op.real) *op.real = op.d; }
    else if (stores || op.u < *op.whole) *op.whole = op.u;
}

// what(): after every order of the lists' operations, each list's own order kept
template <class What>
static void every_order(Words &w, const std::vector<std::vector<Op>> &lists, std::vector<size_t> &at, bool stores, const What &what)
{
    bool any = false;
    for (size_t k = 0; k < lists.size(); ++k) {
        if (at[k] == lists[k].size()) continue;
        any = true;
        const Words before = w;
        apply(lists[k][at[k]++], stores);
        every_order(w, lists, at, stores, what);
        --at[k];
        w = before;
    }
    if (!any) what();
}

struct Scan { u64 length; double bound; };              // the label it reads, the nearest path end it knows of

static long orders, broken;

// A row's scans in one step; `listed`: how far off its entries are when its path has length 0.
static void scans(const std::vector<Scan> &all, const std::vector<double> &listed, bool stores)
{
    Words w{FAR, FAR, FAR, NEVER, NEVER};
    std::vector<std::vector<Op>> lists(all.size());
    std::vector<double> offered(listed.size(), FAR);
    u64 label = NEVER;
    for (size_t k = 0; k < all.size(); ++k) {
        const double length = (double)all[k].length;
        double left_out = FAR;
        for (size_t e = 0; e < listed.size(); ++e) {
            const double x = length + listed[e];
            if (x < all[k].bound) offered[e] = x < offered[e] ? x : offered[e];
            else left_out = x < left_out ? x : left_out;
        }
        publish_scan(Recorder{&lists[k]}, ScanWords{&w.base, &w.dropped, &w.expanded}, all[k].length, length + PROFIT + EPS, left_out);
        label = all[k].length < label ? all[k].length : label;
    }
    std::vector<size_t> at(all.size(), 0);
    every_order(w, lists, at, stores, [&]() {
        ++orders;
        if (!scanned_from(label, w.expanded)) return;   // it will be scanned again
        bool good = w.base == (double)label + PROFIT + EPS;
        for (size_t e = 0; e < listed.size(); ++e) {
            const double x = (double)label + listed[e];
            good = good && (offered[e] <= x || w.dropped <= x);
        }
        if (!good) ++broken;
    });
}

// A pass over all columns has had the row, scanned from `length`, put on the list of whole lines and on the
// frontier; in the next step one slice for each of `slices` reads half of the unlisted entries, and the
// row is scanned from each of `again`.
static void whole_line(u64 length, const std::vector<Scan> &slices, const std::vector<Scan> &again, const std::vector<double> &unlisted,
                       bool stores, bool moved)
{
    double nearest = FAR;
    for (double d : unlisted) nearest = d < nearest ? d : nearest;
    Words w{(double)length + PROFIT + EPS, FAR, (double)length, NEVER, NEVER};
    const ScanWords scan_at{&w.base, &w.dropped, &w.expanded};
    const WholeLine line_at{&w.read_from, &w.left};
    std::vector<std::vector<Op>> lists(slices.size() + again.size());
    begin_whole_line(Recorder{nullptr}, line_at, length, FAR);
    std::vector<double> offered(unlisted.size(), FAR);
    u64 label = length;
    double least_bound = FAR;
    for (size_t k = 0; k < slices.size(); ++k) {
        double left_out = FAR;
        for (size_t e = k; e < unlisted.size(); e += slices.size()) {
            const double x = (double)slices[k].length + unlisted[e];
            if (x < slices[k].bound) offered[e] = x;
            else left_out = x < left_out ? x : left_out;
        }
        if (left_out < FAR) publish_slice(Recorder{&lists[k]}, line_at, left_out);
        label = slices[k].length < label ? slices[k].length : label;
        least_bound = slices[k].bound < least_bound ? slices[k].bound : least_bound;
    }
    for (size_t k = 0; k < again.size(); ++k) {
        publish_scan(Recorder{&lists[slices.size() + k]}, scan_at, again[k].length, (double)again[k].length + PROFIT + EPS, FAR);
        label = again[k].length < label ? again[k].length : label;
    }
    std::vector<size_t> at(lists.size(), 0);
    every_order(w, lists, at, stores, [&]() {
        ++orders;
        // (not scanned from its label yet: it is, before anything is concluded about what is not on its list)
        const double by_bound = (double)label + nearest;
        const double rem = unlisted_from(label, moved ? 0 : w.read_from, w.left, by_bound);
        bool good = true;
        for (size_t e = 0; e < unlisted.size(); ++e) {
            const double x = (double)label + unlisted[e];
            good = good && (offered[e] <= x || rem <= x);
        }
        if (label == length) good = good && rem >= least_bound;        // the line is not read again while no path end is farther
        if (!good) ++broken;
    });
}

int main(int argc, char **argv)
{
    const bool stores = argc > 1 && strcmp(argv[1], "stores") == 0, moved = argc > 1 && strcmp(argv[1], "moved") == 0;
    const std::vector<double> listed = {8.0, 9.0, 15.0, 40.0};
    const double bounds[] = {20.0, 30.0, 90.0};
    for (double b0 : bounds)
        for (double b1 : bounds) {
            scans({{20, b0}, {12, b1}}, listed, stores);
            for (double b2 : bounds) scans({{20, b0}, {12, b1}, {5, b2}}, listed, stores);
        }
    printf("scans: %ld orders, %ld broken\n", orders, broken);
    orders = broken = 0;
    const std::vector<double> unlisted = {11.0, 25.0, 14.0, 70.0};
    const u64 labels[] = {20, 12};
    for (double b0 : bounds)
        for (double b1 : bounds)
            for (u64 l0 : labels)
                for (u64 l1 : labels) {
                    whole_line(20, {{l0, b0}, {l1, b1}}, {}, unlisted, stores, moved);
                    for (u64 l2 : labels) {
                        whole_line(20, {{l0, b0}, {l1, b1}}, {{l2, b0}}, unlisted, stores, moved);
                        whole_line(20, {{l0, b0}, {l1, b1}}, {{20, b0}, {l2, b1}}, unlisted, stores, moved);
                    }
                }
    printf("whole lines: %ld orders, %ld broken\n", orders, broken);
    return 0;
}
