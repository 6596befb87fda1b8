// Row pitch of the scatter adjoint's box for every box of at most argv[1] cells
// (plain C++, built with g++): prints the number of boxes, and exits with 1 at
// the first whose rows overlap or that no longer fits.
#include "plan_logic.h"

#include <cstdio>
#include <cstdlib>

int main(int, char** argv) {
    const int cells = std::atoi(argv[1]);
    int n = 0, padded = 0;
    for (int bw = 8; bw * 8 <= cells; ++bw)
        for (int bh = 8; bw * bh <= cells; ++bh, ++n) {
            const int p = dg::scatter_box_pitch(bw, bh, cells);
            if (p < bw || p * bh > cells) {
                std::printf("%d x %d: %d\n", bw, bh, p);
                return 1;
            }
            padded += p % 16 == 8;
        }
    std::printf("%d %d\n", n, padded);
    return 0;
}
