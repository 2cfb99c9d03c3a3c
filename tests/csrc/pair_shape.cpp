// Prints the decomposition that a single grid's iterations run in pairs with, one
// line per "I J K row_align coefficient-bytes" line of its input: form (flat, row
// or none), points per lane, waves, tiles per row (flat: segments per plane).
#include <cstdio>

#include "pair.hpp"

using namespace ofl;

int main() {
    int I, J, K, row_align, eb;
    while (std::scanf("%d %d %d %d %d", &I, &J, &K, &row_align, &eb) == 5) {
        PairShape s;
        if (pair_choose(I, J, K, round_up(I, row_align > 0 ? row_align : kPitchAlign), eb, &s))
            std::printf("%s %d %d %d\n", s.flat ? "flat" : "row", s.vec, s.waves, s.nti);
        else
            std::printf("none 0 0 0\n");
    }
    return 0;
}
