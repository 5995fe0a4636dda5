// line_parts.h: how long whole lines take, against all wavefronts busy all the time; usage: line_parts [prefixes]
#include <cstdio>
#include <initializer_list>
#include <cstring>
#include "line_parts.h"

int main(int argc, char **argv)
{
    const bool prefixes = argc > 1 && !strcmp(argv[1], "prefixes");
    long long tried = 0, wrong = 0;
    double worst = 0.0;
    for (int waves : {8, 64, 240, 256, 2048})
        for (int slices = 1; slices <= 40; ++slices)
            for (int lines = 1; lines <= 6 * waves; lines += lines < 700 ? 1 : 13) {
                const int parts = parts_of_line(slices, lines, waves, prefixes);
                ++tried;
                if (parts < 1 || parts > slices) { ++wrong; continue; }
                // turns of the busiest wavefront, each as many slices as the longest part has
                const long long turns = ((long long)lines * parts + waves - 1) / waves * ((slices + parts - 1) / parts);
                const long long ideal = ((long long)lines * slices + waves - 1) / waves;
                const double off = (double)turns / (double)ideal;
                worst = off > worst ? off : worst;
                if (4 * turns > 5 * ideal) ++wrong;
            }
    printf("%lld tried, %.2f of the ideal at worst, %lld wrong\n", tried, worst, wrong);
    return wrong != 0;
}
