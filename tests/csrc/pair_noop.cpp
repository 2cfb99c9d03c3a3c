// The pair sweep's launchers doing nothing, beside the no-op launchers of the
// host-code build on the stand-in HIP runtime: with them present the host code
// runs iterations in pairs.
#include "pair.hpp"

namespace ofl {
void launch_pair(const GridView &, int, const PairShape &, float, double *, const double *, hipStream_t) {}
void launch_pair_fold(const double *, const PairShape &, float, double *, hipStream_t) {}
void launch_pair_batch(const GridView *, const PairItem *, int, const int *, int, int, float, double *, const double *,
                       hipStream_t) {}
void launch_pair_batch_fold(const GridView *, const double *, int, const int *, int, float, hipStream_t) {}
}  // namespace ofl
