// Prints the tile id that the library chooses for a tall grid on 256 compute units: one "id cout P taps bytes sparse" per input line.
#include "../../paper_2411_00288_amd/csrc/ss_conv_params.h"
#include <cstdio>

int main()
{
    int id, cout, P, taps, bytes, sparse;
    while (std::scanf("%d %d %d %d %d %d", &id, &cout, &P, &taps, &bytes, &sparse) == 6) {
        ss::ConvParams p{};
        p.Cout = cout; p.P = P;
        std::printf("%d\n", ss::choose_height(p, id, taps != 0, bytes != 0, sparse != 0, 256));
    }
    return 0;
}
