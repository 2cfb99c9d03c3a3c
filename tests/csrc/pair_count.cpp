// The pair sweep's launchers counting their calls, for the host-code build on the
// stand-in HIP runtime: the driver reads how often iterations went in pairs.
#include "pair.hpp"

namespace {
long g_grid = 0, g_batch = 0;
}

extern "C" long pair_launches(void) { return g_grid; }
extern "C" long pair_batch_launches(void) { return g_batch; }

namespace ofl {
void launch_pair(const GridView &, int, const PairShape &, float, double *, const double *, hipStream_t) { ++g_grid; }
void launch_pair_fold(const double *, const PairShape &, float, double *, hipStream_t) {}
void launch_pair_batch(const GridView *, const PairItem *, int, const int *, int, int, float, double *, const double *,
                       hipStream_t) {
    ++g_batch;
}
void launch_pair_batch_fold(const GridView *, const double *, int, const int *, int, float, hipStream_t) {}
}  // namespace ofl
