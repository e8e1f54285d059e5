// Prints the tile id that the library chooses for a dense FP8 layer on 256 compute units: one "id cout P taps steps" per input line.
#include "../../paper_2411_00288_amd/csrc/ss_conv_params.h"
#include <cstdio>

int main()
{
    int id, cout, P, taps, steps;
    while (std::scanf("%d %d %d %d %d", &id, &cout, &P, &taps, &steps) == 5) {
        ss::ConvParams p{};
        p.Cout = cout; p.P = P; p.Ks = steps;
        std::printf("%d\n", ss::choose_height(p, id, taps != 0, true, false, 256, true));
    }
    return 0;
}
