// Walks dealt shares of a tile list (plain C++, built with g++): prints the
// tiles visited for "begin stride end" as one line each.
#include "plan_logic.h"

#include <cstdio>
#include <cstdlib>

int main(int argc, char** argv) {
    for (int i = 1; i + 2 < argc; i += 3) {
        const int begin = std::atoi(argv[i]), stride = std::atoi(argv[i + 1]), end = std::atoi(argv[i + 2]);
        for (int t = begin; t < end; t = dg::next_dealt(t, stride, end)) std::printf("%d ", t);
        std::printf("\n");
    }
    return 0;
}
