// The choice between row tiles and flat segments for a grid's pair sweep over
// random and edge sizes: where it takes segments, they cover the interior, none
// starts past it, the partial sums fit the staging buffer, and nothing that
// pair_plan refuses is taken.
#include <cstdio>
#include <cstdlib>
#include <random>

#include "pair.hpp"

using namespace ofl;

static void check(bool ok, const char *what, int I, int J, int K, int pitch, const PairShape &s) {
    if (ok)
        return;
    std::printf("%s: %dx%dx%d pitch %d: nti %d nkc %d chunk %d\n", what, I, J, K, pitch, s.nti, s.nkc, s.chunk);
    std::exit(1);
}

int main() {
    std::mt19937 rng(9);
    long long flat = 0;
    for (int t = 0; t < 20000; ++t) {
        const int edge[] = {3, 4, 33, 64, 65, 66, 67, 129, 130, 150, 161, 257, 258, 301, 400, 512};
        auto size = [&](int hi) {
            return rng() % 3 == 0 ? edge[rng() % 16] : 3 + static_cast<int>(rng() % static_cast<unsigned>(hi));
        };
        const int I = size(600), J = size(300), K = size(300), eb = rng() % 2 ? 4 : 2;
        const int pitch = round_up(I, rng() % 2 ? 32 : 4);
        PairShape rows, s;
        const bool planned = pair_plan(I, J, K, pitch, eb, &rows);
        const bool taken = pair_choose(I, J, K, pitch, eb, &s);
        check(planned || !taken, "taken where refused", I, J, K, pitch, s);
        if (!taken || !s.flat)
            continue;
        ++flat;
        check(s.vec == 4 && s.waves == kPairBatchWaves && s.njt == 1, "shape", I, J, K, pitch, s);
        const long long own = pair_flat_own(pitch, s.waves), first = pair_flat_first(pitch);
        check(own > 0 && own % 8 == 0 && first % 8 == 0 && first <= pitch, "segments", I, J, K, pitch, s);
        check(first + s.nti * own >= (J - 1LL) * pitch, "the segments end short", I, J, K, pitch, s);
        check(first + (s.nti - 1LL) * own < (J - 1LL) * pitch, "a segment too many", I, J, K, pitch, s);
        check(s.nkc * s.chunk >= K - 2 && (s.nkc - 1) * s.chunk < K - 2, "planes", I, J, K, pitch, s);
        check(4LL * 8 * s.blocks() <= 4LL * I * J * K, "partials", I, J, K, pitch, s);
    }
    std::printf("flat choices ok: %lld\n", flat);
    return flat > 1000 ? 0 : 1;
}
