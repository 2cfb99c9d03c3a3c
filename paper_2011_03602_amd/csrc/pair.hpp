// The pair sweep (pair.hip): two iterations in one pass over the coefficients,
// and the rule that decides where and in what decomposition it runs.
#pragma once

#include <algorithm>

#include "ofl_internal.hpp"

namespace ofl {

// Points at either end of a tile inside a row that it computes for its own
// second step only: two, in whole lanes.
__host__ __device__ inline constexpr int pair_margin(int vec) { return vec < 2 ? 2 : vec; }

// Row form: where a lane whose points start at i0 loads its vec points of p, and
// where it loads n coefficients for the points from i0. Loads that would pass the
// row's end move back; no load that holds an interior point's value may move,
// since its lane takes the values by position.
__host__ __device__ inline constexpr int pair_row_at(int i0, int I, int vec) {
    const int last = (I - 1) / vec * vec;
    return i0 < last ? i0 : last;
}
__host__ __device__ inline constexpr int pair_coef_at(int i0, int cpitch, int n) {
    return i0 < cpitch - n ? i0 : cpitch - n;
}
// bfloat16 coefficients at 4 points per lane travel in 16-byte loads of 8 points,
// the last of which would move back by 4 in a row of 4 points more than a multiple
// of 8 (and every other row would start 8 bytes off the load's size): such rows
// take flat segments, whose loads run across row ends, or fewer points per lane.
__host__ __device__ inline constexpr bool pair_row_form(int vec, int coef_elem, int cpitch) {
    return vec < 4 || coef_elem == 4 || cpitch % 8 == 0;
}

// Decomposition of one grid's pair sweep: tiles of 64*vec points along i (which
// overlap by two margins), waves-2 rows along j and `chunk` planes along k.
struct PairShape {
    int vec = 0, waves = 0;
    int nti = 0, njt = 0, nkc = 0, chunk = 0;
    bool flat = false;  // nti segments of a plane instead of tiles and rows (njt 1)
    int blocks() const { return nti * njt * nkc; }
};

inline int pair_itiles(int I, int vec) {
    const int span = kWave * vec, stride = span - 2 * pair_margin(vec);
    return I - 1 <= span ? 1 : 1 + (I - 1 - span + stride - 1) / stride;
}

// What a pair takes in `blocks` work-groups of a form, us. A launch is a few rounds
// of resident work-groups: one per CU at 4 points per lane, whose registers fill
// it, two below, where one alone is faster. A round costs chunk + 3 planes (two
// margin planes, and the fill of the pipeline), a plane a fixed part (its barrier
// and arithmetic) and its share of the memory rate, by the rows of 64 points it
// loads; what the last-level cache holds (arrays of up to 224 MiB) streams twice
// as fast. Fitted to 51 grids from 33x33x65 to 385x257x385 in both formats and
// 30 to 80 decompositions each: the choice by it takes 1.015 times the best
// measured one on average, 1.13 at worst.
struct PairForm {
    int vec, waves;
    double plane_us;
};
inline double pair_us(const PairForm &form, long long blocks, int chunk, double rows, double bytes, int coef_elem) {
    const long long slots = 256 * (form.vec == 4 ? 1 : 2);  // an MI355X has 256 CUs, and the fit is theirs
    const double per_row = (coef_elem == 4 ? 1.18e-4 : 0.61e-4) * (bytes < 224.0 * (1 << 20) ? 1.0 : 2.0);
    double us = 3.0 + 0.004 * static_cast<double>(blocks);
    for (long long left = blocks; left > 0; left -= slots) {
        const double alone = form.vec < 4 && left <= 256 ? 0.76 : 1.0;
        us += (chunk + 3) * (form.plane_us * alone + static_cast<double>(std::min(left, slots)) * rows * per_row);
    }
    return us;
}

// The best decomposition of a grid's pairs by rows; false where there is none.
// What it decides most is how full the last round is: at 257x257x513 in FP32, 7
// waves and 5 chunks make 255 work-groups of one round (361 us), 8 waves 258 of
// two (603 us) or 473 (387 us).
inline bool pair_plan(int I, int J, int K, int pitch, int coef_elem, PairShape *best, double *predicted_us = nullptr) {
    if (static_cast<long long>(pitch) * J > (1LL << 28))
        return false;  // offsets inside a plane are 32-bit byte counts
    const double points = static_cast<double>(I) * J * K;
    const double bytes = points * (12 * coef_elem + 8);
    constexpr PairForm kForms[] = {{4, 8, 1.66}, {4, 7, 1.54}, {2, 8, 1.40}, {1, 8, 0.86}};
    double best_us = 0.0;
    best->vec = 0;
    for (const auto &form : kForms) {
        if (form.vec == 1 && I - 1 > kWave)
            continue;  // tiles of 60 points split cache lines
        if (!pair_row_form(form.vec, coef_elem, pitch))
            continue;  // by pitch: compact coefficient rows have p's, the default ones whole lines under a pitch of 32 k
        PairShape s;
        s.vec = form.vec;
        s.waves = form.waves;
        s.nti = pair_itiles(I, s.vec);
        s.njt = (J - 2 + s.waves - 3) / (s.waves - 2);
        const long long tiles = static_cast<long long>(s.nti) * s.njt;
        // rows of 64 points that a work-group loads per plane (80 more points
        // for a tile boundary: the overlap and the lines it splits)
        const double rows = s.waves * (I + 80.0 * (s.nti - 1)) / s.nti / kWave;
        for (int nkc = 1; nkc <= std::min(K - 2, 1024) && tiles * nkc <= 8192; ++nkc) {
            const int chunk = (K - 2 + nkc - 1) / nkc;
            if (chunk == s.chunk)
                continue;
            s.chunk = chunk;
            s.nkc = (K - 2 + chunk - 1) / chunk;
            // the partial sums live in the grid's staging buffer
            if (32.0 * s.blocks() > 4.0 * points)
                continue;
            const double us = pair_us(form, s.blocks(), chunk, rows, bytes, coef_elem);
            if (best->vec == 0 || us < best_us) {
                best_us = us;
                *best = s;
            }
        }
    }
    if (predicted_us)
        *predicted_us = best_us;
    return best->vec != 0;
}

// Flat form, for a batch's grids and single ones (pair_choose): a work-group
// covers 256 * kPairBatchWaves consecutive points of a plane, whatever the row
// length, and owns those that lie a row and a point from either end (in whole
// 16-byte loads of bfloat16).
constexpr int kPairBatchWaves = 8;
__host__ __device__ inline constexpr int pair_flat_margin(int pitch) { return (pitch + 1 + 7) / 8 * 8; }
__host__ __device__ inline constexpr int pair_flat_own(int pitch, int waves) {
    return waves * kWave * 4 - 2 * pair_flat_margin(pitch);
}
// The first owned point of a plane's first work-group, and how many there are.
__host__ __device__ inline constexpr int pair_flat_first(int pitch) { return pitch / 8 * 8; }
inline int pair_flat_segments(int J, int pitch) {
    const int own = pair_flat_own(pitch, kPairBatchWaves);
    return ((J - 1) * pitch - pair_flat_first(pitch) + own - 1) / own;
}

// The decomposition a single grid's iterations run in pairs with: pair_plan's, or
// flat segments where they take less; false where the iterations run one by one.
// Flat wins where tiles of 64, 128 or 256 points leave many lanes idle or cut
// rows in pieces, us per pair: 150x150x150 FP32 44.9 -> 38.3, bfloat16 39.0 ->
// 30.1; 161x161x321 85.0 -> 79.5 and 71.2 -> 62.8; 301x99x143 49.3 -> 46.7 and
// 39.8 -> 36.4. Pairs are worth it while they take less than two single fused
// iterations at the copy rate (a slab of one row, whose margins are five sixths
// of the work, may not); 33x33x65 14.0 -> 3.1 us per iteration. Flat segments are
// compared for rows whose margins leave half of them, and for grids that have a row
// form: one without has none of few enough work-groups, or partial sums past its
// staging buffer (thin grids of a few points), which segments share.
inline bool pair_choose(int I, int J, int K, int pitch, int coef_elem, PairShape *best) {
    double us = 0.0;
    if (!pair_plan(I, J, K, pitch, coef_elem, best, &us))
        return false;
    const double points = static_cast<double>(I) * J * K;
    const double bytes = points * (12 * coef_elem + 8);
    const double single_us = 2.0 * (6.0 + bytes / I * pitch / 5.2e6);  // whole rows stream
    if (pair_flat_own(pitch, kPairBatchWaves) < 0.5 * 4 * kWave * kPairBatchWaves)
        return us <= single_us;
    constexpr PairForm kFlat = {4, kPairBatchWaves, 1.59};
    PairShape s;
    s.flat = true;
    s.vec = 4;
    s.waves = kPairBatchWaves;
    s.nti = pair_flat_segments(J, pitch);
    s.njt = 1;
    for (int nkc = 1; nkc <= std::min(K - 2, 1024) && static_cast<long long>(s.nti) * nkc <= 8192; ++nkc) {
        const int chunk = (K - 2 + nkc - 1) / nkc;
        if (chunk == s.chunk)
            continue;
        s.chunk = chunk;
        s.nkc = (K - 2 + chunk - 1) / chunk;
        if (32.0 * s.blocks() > 4.0 * points)
            continue;
        const double t = pair_us(kFlat, s.blocks(), chunk, 4.0 * kPairBatchWaves, bytes, coef_elem);
        if (t < us) {
            us = t;
            *best = s;
        }
    }
    return us <= single_us;
}

// A work-group's share of a batch: grid, first owned point, planes [m0, m1).
struct PairItem {
    int grid, first, m0, m1;
};

// parts: 2 * blocks() doubles, every one written; prev: the previous pair's
// parts (same shape), whose two residuals this launch turns into gosa, or null.
// Weak: the host code also links without the device code (it then runs every
// iteration by itself).
__attribute__((weak)) void launch_pair(const GridView &g, int bf16, const PairShape &s, float omega, double *parts,
                                       const double *prev, hipStream_t st);
// The last pair's two residuals into gosa.
__attribute__((weak)) void launch_pair_fold(const double *parts, const PairShape &s, float omega, double *gosa,
                                            hipStream_t st);

// The same for a batch: views of every grid, items grid by grid (grid b owns
// items range[b] .. range[b+1]-1), 2 * nitems partial sums.
__attribute__((weak)) void launch_pair_batch(const GridView *views, const PairItem *items, int nitems,
                                             const int *range, int ngrids, int bf16, float omega, double *parts,
                                             const double *prev, hipStream_t st);
__attribute__((weak)) void launch_pair_batch_fold(const GridView *views, const double *parts, int nitems,
                                                  const int *range, int ngrids, float omega, hipStream_t st);

}  // namespace ofl
