// side_end.h: the bids of a ladder of phases whose sides end by its rules, as the phases on lists take them.
//
// Every phase begins with nobody placed and the prices of the one before; rows bid, then the columns that nobody holds and that still
// have a price.  Bidders follow their chains for some steps between two looks at the list, side by side.  What searches do in the
// phases that run to the end is left out: the model stops where the first of them begins, and says how many of its epsilons the
// prices of columns that somebody holds have still to come down (no columns but those in use have one at the optimum of weights that
// are nearly the same).
// usage: side_end rows columns base spread rule; rule "every side": the limit on steps holds on both sides at every size
#include <algorithm>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <random>
#include <vector>
#include "side_end.h"

namespace {

struct Side {
    const std::vector<int> &weight;     // line by line, negative: infeasible
    int lines, len;
    std::vector<double> &dual;          // of the other side
    std::vector<int> &holder;
};

constexpr int WAVES = 240, STEPS_MANY = 4, STEPS_FEW = 32, FEW = 64;

long long run(const Side &s, double K, std::vector<int> bidders, double eps, int stop, long long steps, long long most, int &left)
{
    long long bids = 0, followed = 0;
    while (!side_ends((int)bidders.size(), stop, steps, followed) && bids < most) {
        const int count = (int)bidders.size(), turns = count > WAVES ? STEPS_MANY : STEPS_FEW;
        std::vector<int> next;
        for (int first = 0; first < count; first += WAVES) {
            std::vector<int> now(bidders.begin() + first, bidders.begin() + std::min(count, first + WAVES));
            for (int t = 0; t < turns; ++t)
                for (int &b : now) {
                    if (b < 0) continue;
                    ++bids;
                    const int *w = &s.weight[(size_t)b * s.len], from = (int)((unsigned)b * 2654435761u >> 12) % s.len;
                    double best = -1e300, second = -1e300;
                    int at = -1;
                    for (int k = 0; k < s.len; ++k) {
                        const int j = from + k < s.len ? from + k : from + k - s.len;
                        if (w[j] < 0) continue;
                        const double v = K * w[j] - s.dual[j];
                        if (v > best) { second = best; best = v; at = j; }
                        else second = std::max(second, v);
                    }
                    if (best <= eps) { b = -1; continue; }
                    s.dual[at] = K * w[at] - std::max(second - eps, 0.0);
                    const int evicted = s.holder[at];
                    s.holder[at] = b;
                    b = evicted;
                }
            for (int b : now) if (b >= 0) next.push_back(b);
        }
        if (count <= FEW) followed += turns;
        bidders = next;
    }
    left = (int)bidders.size();
    return bids;
}

}  // namespace

int main(int argc, char **argv)
{
    if (argc == 4 && !strcmp(argv[1], "asked")) {               // so many asked for of so many phases
        printf("%d\n", phases_to_the_end(atoi(argv[2]), false, atoi(argv[3])));
        return 0;
    }
    if (argc < 6) return 2;
    const int n = atoi(argv[1]), m = atoi(argv[2]), base = atoi(argv[3]), spread = atoi(argv[4]), theta = 24, keep = 4;
    const bool every_side = !strcmp(argv[5], "every side");
    std::mt19937 rng(1);
    std::vector<int> W((size_t)n * m), T((size_t)n * m);
    int largest = 0;
    for (int i = 0; i < n; ++i)
        for (int j = 0; j < m; ++j) {
            const int w = base + (int)(rng() % (unsigned)(spread + 1));
            W[(size_t)i * m + j] = T[(size_t)j * n + i] = rng() % 10 < 3 ? -1 : w;
            largest = std::max(largest, w);
        }
    const double K = n + 1.0;
    std::vector<long long> ladder;
    for (long long e = (n + 1ll) * largest / theta;; e /= theta) { ladder.push_back(std::max(e, 1ll)); if (e <= 1) break; }
    const int phases = (int)ladder.size(), preparing = phases - keep;
    std::vector<double> price(m, 0.0), profit(n, 0.0);
    long long bids = 0;
    const long long most = 200ll * (n + m);                     // a side
    for (int ph = 0; ph < preparing; ++ph) {
        const double eps = (double)ladder[ph];
        const int stop = bidders_left_over(phases - 1 - ph, keep, 16, 2, 16, n);
        std::vector<int> all(n), holder(m, -1), row_holder(n, -1), unused;
        for (int i = 0; i < n; ++i) all[i] = i;
        int rows_left = 0, columns_left = 0;
        bids += run(Side{W, n, m, price, holder}, K, all, eps, stop, ph == 0 ? 0 : 64, most, rows_left);      // (the first phase is on whole lines)
        std::fill(profit.begin(), profit.end(), -1.0);
        for (int k = 0; k < m; ++k) {
            if (holder[k] >= 0) { row_holder[holder[k]] = k; profit[holder[k]] = K * W[(size_t)holder[k] * m + k] - price[k]; }
            else if (price[k] > 0.0) unused.push_back(k);
        }
        for (int i = 0; i < n; ++i)
            if (profit[i] < 0.0)
                for (int k = 0; k < m; ++k)
                    if (W[(size_t)i * m + k] >= 0) profit[i] = std::max(profit[i], K * W[(size_t)i * m + k] - price[k]);
        const bool next_runs_to_the_end = ph + 1 >= preparing;
        if ((int)unused.size() > (stop > 0 && !next_runs_to_the_end ? stop + rows_left : stop)) {
            const bool early = ph > 0 && (every_side || columns_may_wait((int)unused.size(), rows_left, stop, 16, FEW));
            bids += run(Side{T, m, n, profit, row_holder}, K, unused, eps, stop, early ? 64 : 0, most, columns_left);
            std::fill(price.begin(), price.end(), 0.0);
            for (int i = 0; i < n; ++i) if (row_holder[i] >= 0) price[row_holder[i]] = K * W[(size_t)i * m + row_holder[i]] - profit[i];
        }
    }
    const double highest = *std::max_element(price.begin(), price.end());
    printf("%d phases, %lld bids, prices up to %.0f epsilons of the first that runs to the end\n", preparing, bids, highest / (double)ladder[preparing]);
    const bool bounded = bids < 120ll * preparing * (n + m) && highest < 2.0 * theta * (double)ladder[preparing];
    return bounded ? 0 : 1;
}
