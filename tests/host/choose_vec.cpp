// Prints the tile id that the library chooses for a channels-last layer on 256 compute units: one "cout K P bytes sparse" per input line.
#include "../../paper_2411_00288_amd/csrc/ss_conv_params.h"
#include <cstdio>

int main()
{
    int cout, K, P, bytes, sparse;
    while (std::scanf("%d %d %d %d %d", &cout, &K, &P, &bytes, &sparse) == 5) {
        ss::ConvParams p{};
        p.Cout = cout; p.K = K; p.P = P;
        std::printf("%d\n", ss::choose_vec(p, bytes != 0, sparse != 0, 256));
    }
    return 0;
}
