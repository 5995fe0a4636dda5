// Runs csrc/half_list.h with arrays of 64 in a wavefront's place (test_half_list.py) and compares with plain loops.
//
//   half_list RULE      "exact": as the header has it; "rounded up": the second value from its float, rounded up
#include <math.h>
#include <stdint.h>
#include <stdio.h>
#include <string.h>
#include <algorithm>
#include <random>
#include "half_list.h"

struct Arrays {
    struct Values { double a[64]; };
    struct Keys { int a[64]; };
    static int bits(float f) { int i; memcpy(&i, &f, 4); return i; }

    Keys keys(const Values &v, double outside) const { Keys k; for (int l = 0; l < 64; ++l) k.a[l] = bits((float)std::max(v.a[l] - outside, 0.0)); return k; }
    double distance(int key) const { float f; memcpy(&f, &key, 4); return (double)f; }
    int largest(const Keys &k) const { return *std::max_element(k.a, k.a + 64); }
    unsigned long long equal(const Keys &k, int to) const { unsigned long long m = 0; for (int l = 0; l < 64; ++l) m |= (unsigned long long)(k.a[l] == to) << l; return m; }
    double largest_among(const Values &v, unsigned long long lanes) const { double x = -1e300; for (int l = 0; l < 64; ++l) if (lanes >> l & 1) x = std::max(x, v.a[l]); return x; }
    unsigned long long equal_among(const Values &v, double to, unsigned long long lanes) const { unsigned long long m = 0; for (int l = 0; l < 64; ++l) m |= (unsigned long long)(v.a[l] == to) << l; return m & lanes; }
    Keys without(const Keys &k, int lane) const { Keys o = k; o.a[lane] = 0; return o; }
    double at(const Values &v, int lane) const { return v.a[lane]; }
};

int main(int argc, char **argv)
{
    if (argc != 2) return 2;
    const bool rounded = !strcmp(argv[1], "rounded up");
    if (!rounded && strcmp(argv[1], "exact")) return 2;
    const Arrays wave;
    std::mt19937_64 random(5);
    long wrong_lane = 0, wrong_value = 0, cases = 0;
    for (int kind = 0; kind < 60; ++kind) {
        // spread around a value of 2^scale, some of it below `outside`
        const int scale = kind % 20 + 8 + kind / 20 * 13;
        for (int t = 0; t < 3000; ++t) {
            Arrays::Values v;
            const int64_t base = (int64_t)1 << std::min(scale, 50), spread = (int64_t)1 << (random() % std::min(scale, 50));
            const int tied = (int)(random() % 4);
            for (int l = 0; l < 64; ++l)
                v.a[l] = (double)(base + (int64_t)(random() % (uint64_t)(tied == 0 ? 3 : 2 * spread)) - (tied == 1 && l % 3 ? base : 0));
            if (tied == 2) for (int l = 0; l < 64; l += 5) v.a[l] = v.a[l / 5];
            if (t % 7 == 0) for (int l = 20; l < 64; ++l) v.a[l] = -2.147e18;        // infeasible entries
            double sorted[64];
            std::copy(v.a, v.a + 64, sorted);
            std::sort(sorted, sorted + 64);
            const double outsides[] = {0.0, sorted[63], sorted[62], sorted[62] - 1.0, sorted[60], std::max(sorted[0], 0.0), sorted[63] + 5.0, 1.0e300};
            const double outside = std::max(outsides[random() % 8], 0.0);
            const unsigned turn = (unsigned)(random() % 64);
            const Arrays::Keys key = wave.keys(v, outside);
            int top, next;
            const int best = best_lane(wave, v, key, turn, &top);
            double second = next_value(wave, v, key, best, outside, &next);
            if (rounded && next > 0) {
                float f;
                memcpy(&f, &next, 4);
                second = std::min(v.a[best], std::ceil(outside + (double)(f * (1.0f + 0x1p-22f))));
            }
            int expect = -1;                                // the first of the best at or after lane `turn`, round about
            for (int l = 0; l < 64 && expect < 0; ++l) if (v.a[(turn + l) % 64] == sorted[63]) expect = (int)((turn + l) % 64);
            ++cases;
            wrong_lane += best != expect || (top > 0) != (sorted[63] > outside);
            wrong_value += second != std::max(sorted[62], outside) || (next > 0) != (sorted[62] > outside);
        }
    }
    printf("%ld cases, %ld wrong lanes, %ld wrong values\n", cases, wrong_lane, wrong_value);
    return wrong_lane == 0 && wrong_value == 0 ? 0 : 1;
}
