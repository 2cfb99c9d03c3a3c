// The pair sweep's decomposition over random and edge sizes: every tile, row
// block and chunk it names covers the interior, each starts inside it, the
// partial sums fit the staging buffer, and the offsets the kernel keeps in 32
// bits do.
#include <cstdio>
#include <cstdlib>
#include <random>

#include "pair.hpp"

using namespace ofl;

static void check(bool ok, const char *what, int I, int J, int K, int eb, const PairShape &s) {
    if (ok)
        return;
    std::printf("%s: %dx%dx%d, %d-byte coefficients: vec %d waves %d nti %d njt %d nkc %d chunk %d\n", what, I, J, K, eb,
                s.vec, s.waves, s.nti, s.njt, s.nkc, s.chunk);
    std::exit(1);
}

int main() {
    std::mt19937 rng(7);
    long long planned = 0;
    for (int t = 0; t < 20000; ++t) {
        const int edge[] = {3, 4, 64, 65, 66, 67, 128, 129, 130, 256, 257, 258, 505, 506, 753, 754};
        auto size = [&](int hi) {
            return rng() % 3 == 0 ? edge[rng() % 16] : 3 + static_cast<int>(rng() % static_cast<unsigned>(hi));
        };
        const int I = size(1200), J = size(400), K = size(400), eb = rng() % 2 ? 4 : 2;
        const int pitch = round_up(I, rng() % 2 ? 32 : 4);
        PairShape s;
        if (!pair_plan(I, J, K, pitch, eb, &s))
            continue;
        ++planned;
        const int span = kWave * s.vec, m = pair_margin(s.vec), stride = span - 2 * m;
        check(s.vec == 4 || s.waves == 8, "waves", I, J, K, eb, s);
        // the last tile reaches the row's last point, or ends just before it
        check((s.nti - 1) * stride + span >= I - 1, "the tiles end short", I, J, K, eb, s);
        check(s.nti == 1 || (s.nti - 2) * stride + span < I - 1, "a tile too many", I, J, K, eb, s);
        check(s.njt * (s.waves - 2) >= J - 2 && (s.njt - 1) * (s.waves - 2) < J - 2, "rows", I, J, K, eb, s);
        check(s.nkc * s.chunk >= K - 2 && (s.nkc - 1) * s.chunk < K - 2, "planes", I, J, K, eb, s);
        check(4LL * 8 * s.blocks() <= 4LL * I * J * K, "partials", I, J, K, eb, s);
        check(static_cast<long long>(pitch) * J * 4 <= 0x7fffffffLL, "offsets", I, J, K, eb, s);
    }
    if (pair_margin(1) < 2 || pair_margin(2) < 2 || pair_margin(4) < 2)
        return 1;
    PairShape s;
    if (pair_plan(1 << 16, 1 << 14, 3, 1 << 16, 4, &s))
        return 1;
    std::printf("pair plans ok: %lld\n", planned);
    return planned > 10000 ? 0 : 1;
}
