// Prints the launch shapes that the host-side rules of paper_2403_04206_amd/csrc/grawa_route.h give (no GPU toolchain).
//   split <n_cells>...   -> per line: n_cells grid_x grid_y threads
#include <cstdio>
#include <cstdlib>
#include <cstring>

#include "grawa_route.h"

int main(int argc, char **argv)
{
    if (argc < 2) return 2;
    if (!std::strcmp(argv[1], "split")) {
        for (int i = 2; i < argc; ++i) {
            const long long n = std::atoll(argv[i]);
            unsigned gx = 0, gy = 0;
            grawa_split_grid(n, &gx, &gy);
            std::printf("%lld %u %u %d\n", n, gx, gy, GRAWA_SPLIT_THREADS);
        }
        return 0;
    }
    return 2;
}
