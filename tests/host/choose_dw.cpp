// Prints the kernel that a depthwise layer takes on 256 compute units (ids of ss_debug_force_tile): one "N H W C k rows" per input line, rows: of padding above and below.
#include "../../paper_2411_00288_amd/csrc/ss_dwconv.h"
#include <cstdio>

int main()
{
    int N, H, W, C, k, p;
    while (std::scanf("%d %d %d %d %d %d", &N, &H, &W, &C, &k, &p) == 6)
        std::printf("%d\n", ss::choose_dw(ss::DwShape{N, H, W, C, k, k, p, H + 2 * p - k + 1, W + k / 2 * 2 - k + 1}, 256));
    return 0;
}
