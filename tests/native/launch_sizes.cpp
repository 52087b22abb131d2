// Prints launch sizes of csrc/launch_sizes.hpp for the numbers on stdin, one line per line read.
#include <inttypes.h>
#include <stdio.h>
#include <string.h>

#include "launch_sizes.hpp"

int main()
{
    char what[16];
    int64_t x;
    while (scanf("%15s %" SCNd64, what, &x) == 2) {
        if (!strcmp(what, "pairs")) {   // panels -> column tiles per block, blocks, threads per block
            const int64_t span = ul::panel_span(x);
            printf("%" PRId64 " %" PRId64 " %" PRId64 "\n", span, ul::panel_blocks(x, span), ul::kPairThreads);
        } else if (!strcmp(what, "grid")) {   // blocks of 256 threads -> the grid's dimensions
            const ul::Grid2 g = ul::grid2(x, 256);
            printf("%" PRIu32 " %" PRIu32 "\n", g.x, g.y);
        } else if (!strcmp(what, "halo")) {   // near, kept, n, components -> whether a halo is staged
            int64_t kept, n;
            int32_t dim;
            if (scanf("%" SCNd64 " %" SCNd64 " %" SCNd32, &kept, &n, &dim) != 3) return 1;
            printf("%d\n", ul::halo_pays(x, kept, n, dim) ? 1 : 0);
        } else if (!strcmp(what, "ranks")) {   // points, features, neighbours -> whether every pair is taken once
            int32_t d, k;
            if (scanf("%" SCNd32 " %" SCNd32, &d, &k) != 2) return 1;
            printf("%d\n", ul::pairs_pay(x, d, k) ? 1 : 0);
        } else {
            return 1;
        }
    }
    return 0;
}
