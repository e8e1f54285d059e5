// Prints the tile of a channels-last layer with taps and K < 512 on 256 compute units: one "cout P bytes sparse f8" per input line.
#include "../../paper_2411_00288_amd/csrc/ss_conv_params.h"
#include <cstdio>

int main()
{
    int cout, P, bytes, sparse, f8;
    while (std::scanf("%d %d %d %d %d", &cout, &P, &bytes, &sparse, &f8) == 5) {
        ss::ConvParams p{};
        p.Cout = cout; p.P = P; p.K = 288;
        std::printf("%d\n", ss::choose_vec_short(p, bytes != 0, sparse != 0, f8 != 0, 256));
    }
    return 0;
}
