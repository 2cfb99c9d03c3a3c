"""Tile searches measure the tiles they name in the iterations that such a tile runs,
and a tuned grid or batch is not slower than an untuned one."""

import sys
import time

import numpy as np
import pytest

import paper_2011_03602_amd as ofl
import synth
from helpers import OMEGA

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():  # collected on CPU hosts, skipped there
    pytestmark = [pytest.mark.gpu, pytest.mark.skip(reason="needs a GPU")]

PROBE = 60


def say(*args):
    print("[gpu]", *args, flush=True)
    sys.stdout.flush()


@pytest.fixture
def cache(tmp_path):
    path = str(tmp_path / "tune.txt")
    ofl.ofl_set_tune_cache(path)
    yield path
    ofl.ofl_set_tune_cache(None)


def best_ms(run, repeats=9):
    run()
    ms = []
    for _ in range(repeats):
        t0 = time.perf_counter()
        run()
        ms.append((time.perf_counter() - t0) * 1e3)
    return min(ms)  # the host's other work only adds


def make_batch():
    grids = [ofl.Grid(synth.make_problem(*s, seed=sum(s)), row_align=4) for s in ((45, 40, 37), (70, 33, 31))]
    for g in grids:
        ofl.ofl_data_enter(g.handle)
    return ofl.ofl_batch_create([g.handle for g in grids]), grids


def close(b, grids):
    ofl.ofl_batch_destroy(b)
    for g in grids:
        ofl.ofl_data_exit(g.handle)
        g.close()


def first_time(path):
    with open(path) as f:
        return float(f.readline().split()[4])


def test_batch_search_times_its_first_tile_as_that_tile_runs(cache):
    """The gene of the current tile is measured first. Pairs take a third of the time
    or less at these sizes; the file's time is the launches', a run's its host work
    and synchronisation too, which 60 iterations of 3 launches outweigh."""
    say("batch tune, first gene")
    b, grids = make_batch()
    n = len(grids)
    ofl.ofl_batch_run(b, 3, OMEGA, n)
    pairs = best_ms(lambda: ofl.ofl_batch_run(b, PROBE, OMEGA, n))
    tile = ofl.ofl_batch_get_tile(b)
    ofl.ofl_batch_tune(b, ofl.ga_params(population=2, generations=1, probe_iters=PROBE, repeats=3))
    measured = first_time(cache)
    ofl.ofl_batch_set_tile(b, tile)
    single = best_ms(lambda: ofl.ofl_batch_run(b, PROBE, OMEGA, n))
    close(b, grids)
    print(f"in pairs {pairs:.3f} ms, one by one {single:.3f} ms, the search {measured:.3f} ms")
    assert pairs < 0.6 * single
    assert measured > 0.7 * single


def test_grid_search_times_its_first_tile_as_that_tile_runs(cache):
    say("grid tune, first gene")
    g = ofl.Grid(synth.make_problem(45, 40, 37, seed=50))
    ofl.ofl_data_enter(g.handle)
    tile = ofl.ofl_get_tile(g.handle)
    ofl.ofl_grid_tune(g.handle, ofl.ga_params(population=2, generations=1, probe_iters=PROBE, repeats=3))
    measured = first_time(cache)
    ofl.ofl_set_tile(g.handle, tile)
    single = best_ms(lambda: ofl.ofl_jacobi_run(g.handle, PROBE, OMEGA))
    ofl.ofl_data_exit(g.handle)
    g.close()
    assert measured > 0.7 * single


def test_tuned_grid_is_not_slower():
    """And it gives the same iterate. (The limit lies between the timing's noise and
    single iterations, which take over twice the time of pairs here.)"""
    say("grid tune, then run")
    a = synth.make_problem(97, 61, 67, seed=51)
    g, h = ofl.Grid(a), ofl.Grid(a)
    for x in (g, h):
        ofl.ofl_data_enter(x.handle)
    r = ofl.ofl_grid_tune(h.handle, ofl.ga_params(population=4, generations=2, probe_iters=2, repeats=3))
    assert ofl.ofl_get_tile(h.handle).as_dict() == r.best.as_dict()
    x = ofl.ofl_jacobi_run(g.handle, 7, OMEGA)
    y = ofl.ofl_jacobi_run(h.handle, 7, OMEGA)
    ofl.ofl_update_host(g.handle)
    ofl.ofl_update_host(h.handle)
    assert np.array_equal(g.p, h.p) and abs(x - y) <= 1e-9 * abs(x)
    plain = best_ms(lambda: ofl.ofl_jacobi_run(g.handle, PROBE, OMEGA))
    tuned = best_ms(lambda: ofl.ofl_jacobi_run(h.handle, PROBE, OMEGA))
    for x in (g, h):
        ofl.ofl_data_exit(x.handle)
        x.close()
    assert tuned <= 1.6 * plain


def test_tuned_batch_is_not_slower():
    say("batch tune, then run")
    b, grids = make_batch()
    n = len(grids)
    plain = best_ms(lambda: ofl.ofl_batch_run(b, PROBE, OMEGA, n))
    r = ofl.ofl_batch_tune(b, ofl.ga_params(population=4, generations=2, probe_iters=10, repeats=3))
    assert ofl.ofl_batch_get_tile(b).as_dict() == r.best.as_dict()
    tuned = best_ms(lambda: ofl.ofl_batch_run(b, PROBE, OMEGA, n))
    close(b, grids)
    assert tuned <= 1.6 * plain
