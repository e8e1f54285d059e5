// Prints the kernel that an inverted bottleneck takes on 256 compute units, and whether the resident one could run it: one "P Cin Cmid Cout act sparse" per line.
#include "../../paper_2411_00288_amd/csrc/ss_conv_params.h"
#include <cstdio>

int main()
{
    int sparse;
    ss::MlpParams p{};
    while (std::scanf("%d %d %d %d %d %d", &p.P, &p.Cin, &p.Cmid, &p.Cout2, &p.act1, &sparse) == 6)
        std::printf("%d %d\n", ss::choose_mlp(p, sparse != 0, 256), ss::mlp_takes(p, sparse != 0, 42));
    return 0;
}
