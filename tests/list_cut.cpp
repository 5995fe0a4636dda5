// list_cut.h: no entry worth a cut is left out, whatever the size of the numbers, and few others are let through.
#include <cstdint>
#include <cstdio>
#include <random>
#include "list_cut.h"

int main()
{
    std::mt19937_64 rng(7);
    long long wrong = 0, tried = 0, through = 0, below = 0;
    for (int t = 0; t < 4000000; ++t) {
        // K and the largest weight with K w < 2^43, a weight up to it, a cut of either sign near or far from what the weight can be worth
        const long long K = 2 + (long long)(rng() % (1ull << (1 + rng() % 20)));
        const long long top = ((1ll << 43) - 1) / K, largest = 1 + (long long)(rng() % (uint64_t)(top < INT32_MAX ? top : INT32_MAX));
        const long long w = rng() % 4 ? largest - (long long)(rng() % (uint64_t)(1 + largest / (1ll << (rng() % 31)))) : (long long)(rng() % (uint64_t)(largest + 1));
        const double most = (double)(K * largest);
        long long dual = (long long)(rng() % (uint64_t)(1ll << (1 + rng() % 43)));
        if (rng() % 2 && K * w > 0) dual = K * w - (long long)(rng() % (uint64_t)(1 + (K * w >> (rng() % 43))));
        const long long value = K * w - dual;
        const long long away = (long long)(rng() % (uint64_t)(1ll << (1 + rng() % 40)));
        for (int side = 0; side < 3; ++side) {          // worth the cut, more, less
            const double cut = (double)(side == 0 ? value : side == 1 ? value - away : value + 1 + away);
            const bool is = (double)value >= cut, may = may_reach((float)K, (int)w, (float)(double)dual, cut_in_floats(cut, most));
            ++tried;
            if (is && !may) ++wrong;
            if (!is) { ++below; through += may; }
        }
        if (!may_reach((float)K, (int)w, (float)(double)dual, cut_in_floats(LIST_ALL, most)) || may_reach((float)K, (int)w, (float)(double)dual, cut_in_floats(LIST_NONE, most))) ++wrong;
    }
    // far below the cut is left out: by more than 2^-18 of the largest weight's worth and the cut
    for (int t = 0; t < 1000000; ++t) {
        const long long K = 2 + (long long)(rng() % 40000), largest = 1 + (long long)(rng() % (1ull << 24)), w = (long long)(rng() % (uint64_t)(largest + 1));
        const double most = (double)(K * largest), value = (double)(K * w), cut = value + 0x1p-18 * (2.0 * most + value) + 1.0;
        if (may_reach((float)K, (int)w, 0.0f, cut_in_floats(cut, most))) ++wrong;
    }
    printf("%lld cuts, %lld of %lld entries below one looked at exactly, %lld wrong\n", tried, through, below, wrong);
    return wrong != 0;
}
