// Prints the tile that a sparse 8-bit channels-last layer takes on 256 compute units, given the choice before: one "id cout P K" per input line (K in 2-byte units).
#include "../../paper_2411_00288_amd/csrc/ss_conv_params.h"
#include <cstdio>

int main()
{
    int id, cout, P, K;
    while (std::scanf("%d %d %d %d", &id, &cout, &P, &K) == 4) {
        ss::ConvParams p{};
        p.Cout = cout; p.P = P; p.K = K;
        std::printf("%d\n", ss::choose_vec8_sparse(p, id, 256));
    }
    return 0;
}
