/* When iterations go in pairs, on the stand-in HIP runtime (hip_stand_in.cpp) with
 * launchers that count (pair_count.cpp): whatever was called before, a tile of the
 * caller's turns pairs off. A search measures tiles without them and leaves them on
 * unless it finds single iterations faster (the stand-in's times are all the same).
 * A search under a time limit runs what the run without one does, and stops.
 * Repeated runs replay their graphs. */
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include "ofl.h"

long pair_launches(void);
long pair_batch_launches(void);
long stand_in_alloc_calls(void);

#define CHECK(c)                                                                                       \
    do {                                                                                               \
        if (!(c)) {                                                                                    \
            fprintf(stderr, "FAIL %s:%d: %s (last error: %s)\n", __FILE__, __LINE__, #c,               \
                    ofl_last_error());                                                                 \
            return 1;                                                                                  \
        }                                                                                              \
    } while (0)

typedef struct {
    float *arr[14];
    ofl_grid *g;
} problem;

static int make(problem *pb, int I, int J, int K) {
    const size_t n = (size_t)I * J * K;
    ofl_grid_desc d;
    memset(&d, 0, sizeof d);
    for (int a = 0; a < 14; ++a) {
        pb->arr[a] = (float *)malloc(n * sizeof(float));
        for (size_t t = 0; t < n; ++t)
            pb->arr[a][t] = a == 3 ? 1.0f / 6.0f : (a < 3 || (a >= 7 && a <= 10) ? 1.0f : 0.25f);
        if (a < 12)
            d.coef[a] = pb->arr[a];
    }
    d.I = I;
    d.J = J;
    d.K = K;
    d.p = pb->arr[12];
    d.wrk2 = pb->arr[13];
    d.device = -1;
    return ofl_grid_create(&d, &pb->g);
}

static void drop(problem *pb) {
    ofl_grid_destroy(pb->g);
    for (int a = 0; a < 14; ++a)
        free(pb->arr[a]);
}

/* Pair launches of one run, which captures its graph again when something changed. */
static long grid_pairs(ofl_grid *g, int iters) {
    const long n = pair_launches();
    double x;
    return ofl_jacobi_run(g, iters, 0.8f, &x) == OFL_OK ? pair_launches() - n : -1;
}

static long batch_pairs(ofl_batch *b, int iters) {
    const long n = pair_batch_launches();
    double x[2];
    return ofl_batch_run(b, iters, 0.8f, x) == OFL_OK ? pair_batch_launches() - n : -1;
}

static int batch_tiles(void) {
    problem pb[2];
    CHECK(make(&pb[0], 37, 19, 17) == OFL_OK && make(&pb[1], 41, 23, 20) == OFL_OK);
    ofl_grid *grids[2] = {pb[0].g, pb[1].g};
    ofl_tile t;
    for (int run_first = 0; run_first < 2; ++run_first) {
        ofl_batch *b = NULL;
        CHECK(ofl_batch_create(grids, 2, NULL, &b) == OFL_OK);
        if (run_first)
            CHECK(batch_pairs(b, 7) == 3);
        CHECK(ofl_batch_get_tile(b, &t) == OFL_OK && ofl_batch_set_tile(b, &t) == OFL_OK);
        CHECK(batch_pairs(b, 7) == 0 && batch_pairs(b, 9) == 0);
        ofl_batch_destroy(b);
    }
    drop(&pb[0]);
    drop(&pb[1]);
    return 0;
}

static int grid_tiles(void) {
    problem pb;
    ofl_tile t;
    CHECK(make(&pb, 37, 19, 17) == OFL_OK);
    CHECK(grid_pairs(pb.g, 7) == 3);
    CHECK(ofl_get_tile(pb.g, &t) == OFL_OK && ofl_set_tile(pb.g, &t) == OFL_OK);
    CHECK(grid_pairs(pb.g, 7) == 0);
    drop(&pb);
    return 0;
}

/* Nothing runs on the stand-in, so results are wrong: a tolerance that lets them pass. */
static const ofl_ga_params kGa = {2, 1, 7, 0.9, 0.05, 1, 5, 1, 1e30};

static int tuned(void) {
    problem pb[2];
    ofl_tune_result r;
    ofl_tile t;
    CHECK(make(&pb[0], 37, 19, 17) == OFL_OK && make(&pb[1], 41, 23, 20) == OFL_OK);
    for (int profiling = 0; profiling < 2; ++profiling) {
        CHECK(ofl_set_profiling(pb[0].g, profiling) == OFL_OK);
        long n = pair_launches();
        CHECK(ofl_grid_tune(pb[0].g, &kGa, &r) == OFL_OK);
        CHECK(pair_launches() - n <= 2);  /* the comparison's graph of two pairs and nothing else */
        CHECK(ofl_set_profiling(pb[0].g, 0) == OFL_OK);
        CHECK(ofl_get_tile(pb[0].g, &t) == OFL_OK && memcmp(&t, &r.best, sizeof t) == 0);
        CHECK(grid_pairs(pb[0].g, 7) == 3);
        CHECK(ofl_set_tile(pb[0].g, &t) == OFL_OK && grid_pairs(pb[0].g, 7) == 0);
    }
    ofl_grid *grids[2] = {pb[0].g, pb[1].g};
    ofl_batch *b = NULL;
    CHECK(ofl_batch_create(grids, 2, NULL, &b) == OFL_OK);
    for (int set_first = 0; set_first < 2; ++set_first) {
        if (set_first)
            CHECK(ofl_batch_get_tile(b, &t) == OFL_OK && ofl_batch_set_tile(b, &t) == OFL_OK);
        long n = pair_batch_launches();
        CHECK(ofl_batch_tune(b, &kGa, &r) == OFL_OK);
        CHECK(pair_batch_launches() - n == 2);  /* the same */
        CHECK(ofl_batch_get_tile(b, &t) == OFL_OK && memcmp(&t, &r.best, sizeof t) == 0);
        CHECK(batch_pairs(b, 7) == 3);
    }
    /* a search that fails (nothing matches) leaves the batch as it was */
    ofl_ga_params strict = kGa;
    strict.tolerance = 1e-9;
    CHECK(ofl_batch_set_tile(b, &t) == OFL_OK);
    CHECK(ofl_batch_tune(b, &strict, &r) == OFL_ESTATE && batch_pairs(b, 7) == 0);
    ofl_batch_destroy(b);
    CHECK(ofl_grid_tune(pb[1].g, &strict, &r) == OFL_ESTATE && grid_pairs(pb[1].g, 7) == 3);
    drop(&pb[0]);
    drop(&pb[1]);
    return 0;
}

static int limited_search(void) {
    problem pb;
    ofl_loop_search_result r;
    CHECK(make(&pb, 37, 19, 17) == OFL_OK);
    const int wanted = 2 * 258 + 1 + 2 * 4;  /* two full graphs' worth of pairs and some */
    const long n = pair_launches();
    CHECK(ofl_grid_search_loops(pb.g, &kGa, wanted, 0.8f, OFL_XFER_HOISTED, 1e9, &r) == OFL_OK);
    CHECK(pair_launches() > n && r.timed_out == 0);
    /* every gene passes its limit at its first nest or its first pairs, but the
     * all-CPU one, which is measured without a limit first and is no candidate */
    CHECK(ofl_grid_search_loops(pb.g, &kGa, wanted, 0.8f, OFL_XFER_HOISTED, 1e-6, &r) == OFL_ESTATE);
    CHECK(ofl_set_offload_mask(pb.g, OFL_MASK_ALL_GPU, OFL_XFER_HOISTED) == OFL_OK && grid_pairs(pb.g, 7) == 3);
    drop(&pb);
    return 0;
}

/* Repeated runs replay their graphs: no capture, whatever the number of pairs. */
static int replays(void) {
    static const int iters[] = {8, 50, 100, 257, 258, 300, 303, 600, 1027};
    problem pb;
    CHECK(make(&pb, 37, 19, 17) == OFL_OK);
    for (size_t t = 0; t < sizeof iters / sizeof *iters; ++t) {
        CHECK(grid_pairs(pb.g, iters[t]) >= 0 && grid_pairs(pb.g, iters[t]) >= 0);
        const long calls = stand_in_alloc_calls();
        for (int r = 0; r < 4; ++r)
            CHECK(grid_pairs(pb.g, iters[t]) == 0);
        CHECK(stand_in_alloc_calls() == calls);
    }
    /* and so do two lengths in turn */
    for (int r = 0; r < 2; ++r)
        CHECK(grid_pairs(pb.g, 40) >= 0 && grid_pairs(pb.g, 60) >= 0);
    for (int r = 0; r < 4; ++r)
        CHECK(grid_pairs(pb.g, 40) == 0 && grid_pairs(pb.g, 60) == 0);
    drop(&pb);
    return 0;
}

int main(void) {
    if (batch_tiles() || grid_tiles() || tuned() || limited_search() || replays())
        return 1;
    printf("pair policy ok\n");
    return 0;
}
