// search_words.h, pending_rise: a search over several bidders at once that ends before all of them are placed leaves every row within
// epsilon of the best it could hold.  usage: search_end [left out]
//
// Rows bid until a few are left; those are searched for together, as in paths.hip: labels of all trees, the nearest end of a
// path served, its tree's columns labelled once more, the others left as they are; after some of them the search ends.
#include <algorithm>
#include <cstdio>
#include <cstring>
#include <random>
#include <vector>
#include "search_words.h"

namespace {

constexpr int ID_BITS = 20;
constexpr unsigned long long INF = ~0ull;

struct Problem {
    int n, m;
    long long eps;
    std::vector<long long> value, price;        // value: K w, row by row
    std::vector<int> held, holder;              // column of a row, row of a column (-1: none)
    long long worth(int i, int k) const { return value[(size_t)i * m + k] - price[k]; }
    long long best(int i) const { long long b = worth(i, 0); for (int k = 1; k < m; ++k) b = std::max(b, worth(i, k)); return b; }
    void bid(int i)
    {
        int at = 0;
        long long first = -(1ll << 60), second = first;
        for (int k = 0; k < m; ++k) {
            const long long v = worth(i, k);
            if (v > first) { second = first; first = v; at = k; }
            else second = std::max(second, v);
        }
        price[at] += first - second + eps;
        if (holder[at] >= 0) held[holder[at]] = -1;
        holder[at] = i;
        held[i] = at;
    }
    long long off() const                       // by how much more than epsilon a row would rather have another column
    {
        long long most = 0;
        for (int i = 0; i < n; ++i) if (held[i] >= 0) most = std::max(most, best(i) - worth(i, held[i]) - eps);
        return most;
    }
};

// Serves `paths` of the bidders' paths (rows do not rest: columns are enough) and ends.
void search(Problem &p, std::vector<int> bidders, int paths, bool left_out)
{
    std::vector<unsigned long long> label(p.m, INF);
    std::vector<long long> profit(p.n, 0);
    unsigned long long served = 0;
    for (int r : bidders) profit[r] = p.best(r) - p.eps;
    auto length_of = [&](int k) { return (long long)(label[k] >> ID_BITS); };
    auto relax = [&](int i, long long from, long long pi) {
        bool any = false;
        for (int k = 0; k < p.m; ++k) {
            if (p.held[i] == k) continue;
            const long long to = from + pi - p.worth(i, k) + p.eps;
            if (label[k] == INF || to < length_of(k)) { label[k] = ((unsigned long long)to << ID_BITS) | (unsigned)i; any = true; }
        }
        return any;
    };
    for (int done = 0; done < paths && !bidders.empty(); ++done) {
        for (bool any = true; any;) {
            any = false;
            for (int r : bidders) any |= relax(r, 0, profit[r]);
            for (int k = 0; k < p.m; ++k)
                if (label[k] != INF && p.holder[k] >= 0) any |= relax(p.holder[k], length_of(k), p.worth(p.holder[k], k));
        }
        int end = -1;
        for (int k = 0; k < p.m; ++k) if (p.holder[k] < 0 && label[k] != INF && (end < 0 || length_of(k) < length_of(end))) end = k;
        auto root_of = [&](int k) {
            for (;;) {
                const int i = (int)(label[k] & ((1u << ID_BITS) - 1u));
                if (p.held[i] < 0) return i;
                k = p.held[i];
            }
        };
        const int root = root_of(end);
        const long long d = length_of(end);
        std::vector<int> tree;
        for (int k = 0; k < p.m; ++k) if (label[k] != INF && root_of(k) == root) tree.push_back(k);
        for (int k : tree) if (length_of(k) < d) p.price[k] += d - length_of(k);
        for (int k = end; k >= 0;) {
            const int i = (int)(label[k] & ((1u << ID_BITS) - 1u)), before = p.held[i];
            p.price[k] += p.eps;
            p.holder[k] = i;
            p.held[i] = k;
            k = before;
        }
        for (int k : tree) label[k] = INF;
        for (int k = 0; k < p.m; ++k)                               // (labels beyond the path may come from its tree's rows as they were)
            if (label[k] != INF && length_of(k) >= d) label[k] = INF;
        bidders.erase(std::find(bidders.begin(), bidders.end(), root));
        served = (unsigned long long)d;
    }
    if (!left_out)
        for (int k = 0; k < p.m; ++k) p.price[k] += (long long)pending_rise(label[k], INF, ID_BITS, served);
}

}  // namespace

int main(int argc, char **argv)
{
    const bool left_out = argc > 1 && !strcmp(argv[1], "left out");
    std::mt19937 rng(11);
    int tried = 0, wrong = 0;
    for (int t = 0; t < 3000; ++t) {
        Problem p;
        p.n = 6 + (int)(rng() % 30);
        p.m = p.n + (int)(rng() % 4);
        p.eps = 1 + (int)(rng() % 50);
        const int kind = (int)(rng() % 3);
        std::vector<long long> a(p.n), b(p.m);
        for (auto &x : a) x = rng() % 1000;
        for (auto &x : b) x = rng() % 1000;
        p.value.resize((size_t)p.n * p.m);
        for (int i = 0; i < p.n; ++i)
            for (int k = 0; k < p.m; ++k) p.value[(size_t)i * p.m + k] = 2000000 + (kind == 0 ? (long long)(rng() % 100000) : kind == 1 ? a[i] * b[k] : 1000 * (long long)(rng() % 4));
        p.price.assign(p.m, 0);
        p.held.assign(p.n, -1);
        p.holder.assign(p.m, -1);
        const int left = 2 + (int)(rng() % 4);
        for (int turn = 0; turn < 100000; ++turn) {
            std::vector<int> open;
            for (int i = 0; i < p.n; ++i) if (p.held[i] < 0) open.push_back(i);
            if ((int)open.size() <= left) break;
            p.bid(open[rng() % open.size()]);
        }
        std::vector<int> open;
        for (int i = 0; i < p.n; ++i) if (p.held[i] < 0) open.push_back(i);
        if (p.off() > 0) { ++wrong; continue; }                     // (bids keep to it)
        search(p, open, 1 + (int)(rng() % (open.size() - 1)), left_out);
        ++tried;
        wrong += p.off() > 0;
    }
    printf("%d searches ended early, %d wrong\n", tried, wrong);
    return wrong != 0;
}
