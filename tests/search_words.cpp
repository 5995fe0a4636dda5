// Puts what csrc/search_words.h publishes through every order of its memory accesses (test_search_words.py).
//
// Some wavefronts look at one row in the same step, each from the label its column had when that
// wavefront read it.  Every access is one operation on shared memory; the orders of two or three
// wavefronts' operations are all tried, and after each the pass over all columns must find nothing too
// long and nothing hidden.  With "stores" the minima are plain stores, which has to fail: the orders
// tried are those that matter.
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
    double base, dropped;
    u64 expanded;
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
    Words w{FAR, FAR, NEVER};
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

int main(int argc, char **argv)
{
    const bool stores = argc > 1 && strcmp(argv[1], "stores") == 0;
    const std::vector<double> listed = {8.0, 9.0, 15.0, 40.0};
    const double bounds[] = {20.0, 30.0, 90.0};
    for (double b0 : bounds)
        for (double b1 : bounds) {
            scans({{20, b0}, {12, b1}}, listed, stores);
            for (double b2 : bounds) scans({{20, b0}, {12, b1}, {5, b2}}, listed, stores);
        }
    printf("scans: %ld orders, %ld broken\n", orders, broken);
    return 0;
}
