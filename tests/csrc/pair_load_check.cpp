// Row form of the pair sweep, over random and edge sizes: every load that holds an
// interior point's value starts at the point its lane takes it for, is aligned to
// its size, and stays inside the row. And the 4-points-per-lane forms are taken
// where that holds only.
#include <cstdio>
#include <cstdlib>
#include <random>

#include "pair.hpp"

using namespace ofl;

static void check(bool ok, const char *what, int I, int J, int K, int cpitch, int eb, const PairShape &s) {
    if (ok)
        return;
    std::printf("%s: %dx%dx%d, coefficient rows of %d x %d bytes, vec %d waves %d tiles %d\n", what, I, J, K, cpitch, eb,
                s.vec, s.waves, s.nti);
    std::exit(1);
}

int main() {
    std::mt19937 rng(11);
    long long rows = 0, wide = 0;
    for (int t = 0; t < 30000; ++t) {
        const int edge[] = {242, 250, 251, 252, 253, 256, 257, 258, 259, 260, 410, 411, 412, 442, 500, 505};
        const int I = rng() % 3 == 0 ? edge[rng() % 16] : 3 + static_cast<int>(rng() % 1000);
        const int J = 3 + static_cast<int>(rng() % 300), K = 3 + static_cast<int>(rng() % 300);
        const int aligns[] = {0, 4, 8, 16, 32};
        const int row_align = aligns[rng() % 5], eb = rng() % 2 ? 4 : 2;
        // the layout of make_layout (grid.cpp)
        const int pitch = round_up(I, row_align > 0 ? row_align : kPitchAlign);
        const int cpitch = row_align > 0 ? pitch : round_up(I - 1, kPitchAlign * 4 / eb);
        PairShape s;
        if (!pair_choose(I, J, K, pitch, eb, &s) || s.flat)
            continue;
        ++rows;
        check(pair_row_form(s.vec, eb, cpitch), "a row form the launch refuses", I, J, K, cpitch, eb, s);
        const int n = s.vec == 4 && eb == 2 ? 8 : s.vec;  // points per coefficient load
        wide += n == 8;
        for (int it = 0; it < s.nti; ++it) {
            const int ts = it * (kWave * s.vec - 2 * pair_margin(s.vec));
            for (int lane = 0; lane < kWave; ++lane) {
                const int i0 = ts + lane * s.vec, at = pair_row_at(i0, I, s.vec);
                check(at % s.vec == 0 && at + s.vec <= pitch, "a load of p", I, J, K, cpitch, eb, s);
                check(at == i0 || i0 > I - 1, "p moved", I, J, K, cpitch, eb, s);
                const int c0 = n == 8 ? ts + lane % 32 * 8 : at, c = pair_coef_at(c0, cpitch, n);
                check(c >= 0 && c + n <= cpitch, "a load of coefficients", I, J, K, cpitch, eb, s);
                check(c % n == 0 && cpitch % n == 0, "alignment", I, J, K, cpitch, eb, s);
                check(c == c0 || c0 > I - 2, "coefficients moved", I, J, K, cpitch, eb, s);
            }
        }
    }
    std::printf("row loads ok: %lld row shapes, %lld with 16-byte bfloat16 loads\n", rows, wide);
    return rows > 5000 && wide > 1000 ? 0 : 1;
}
