"""Iterations in pairs (the pair sweep) against the same iterations nest by nest.

A run of three iterations or more with every nest on the GPU, hoisted transfers
and no tile of its own goes two iterations per launch; profiling keeps it nest
by nest. Both give every point the same operations in the same order and end on
the same single iteration, so p must be bitwise equal and gosa exactly equal."""

import sys

import numpy as np
import pytest

import oracle
import paper_2011_03602_amd as ofl
import synth
from helpers import OMEGA, TOL_GOSA_F32, TOL_P_F32, boundary_equal, p_rel_err

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():  # collected on CPU hosts, skipped there
    pytestmark = [pytest.mark.gpu, pytest.mark.skip(reason="needs a GPU")]

FUSE_ALL = ofl.OFL_FUSE_RESIDUAL | ofl.OFL_FUSE_COPYBACK_SWAP


def say(*args):
    print("[gpu]", *args, flush=True)
    sys.stdout.flush()


def run(a, fmt, iters_list, profiled, fusion=0, sum_mode=ofl.OFL_SUM_F64, row_align=0):
    g = ofl.Grid(a, coef_format=fmt, sum_mode=sum_mode, row_align=row_align)
    ofl.ofl_set_fusion(g.handle, fusion)
    ofl.ofl_set_profiling(g.handle, profiled)
    ofl.ofl_data_enter(g.handle)
    gosa = [ofl.ofl_jacobi_run(g.handle, n, OMEGA) for n in iters_list]
    ofl.ofl_data_exit(g.handle)
    assert list(ofl.ofl_get_stats(g.handle).gpu_nests) == [sum(iters_list)] * 3
    p = g.p.copy()
    g.close()
    return p, gosa


# Rows that end at, before and past a tile of 64, 128 and 256 points (the
# boundary column inside the tile, just past it, a second and third tile), rows
# and planes around a work-group's 5 or 6 rows and its chunk, the smallest grid.
SHAPES = [(3, 3, 3), (4, 9, 5), (64, 8, 7), (65, 7, 12), (66, 15, 6), (129, 14, 9), (130, 13, 8), (256, 8, 5),
          (257, 12, 21), (258, 9, 33), (505, 8, 6), (506, 9, 4), (770, 7, 5), (97, 41, 30)]


@pytest.mark.parametrize("fmt", [ofl.OFL_COEF_F32, ofl.OFL_COEF_BF16, ofl.OFL_COEF_BF16_OFFSET])
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)))
def test_pairs_equal_single_iterations(shape, fmt):
    say("pairs", shape, "format", fmt)
    a = synth.make_problem(*shape, seed=synth.grid_seed(sum(shape)))
    for row_align in (0, 4):
        iters = [3, 6, 4]  # none, then an odd and an even number of pairs behind a single iteration
        p1, g1 = run(a, fmt, iters, True, row_align=row_align)
        p2, g2 = run(a, fmt, iters, False, row_align=row_align)
        assert np.array_equal(p1, p2)
        assert g1 == g2
    if fmt == ofl.OFL_COEF_F32:
        p_o, g_o = oracle.jacobi(a, sum(iters), float(OMEGA))
        # a converged point's term is FP32 rounding: below (2 ulp of a value of at most 2)^2
        floor = p_o.size * (2 * 2.0 ** -22 / float(OMEGA)) ** 2
        assert p_rel_err(p2, p_o) <= TOL_P_F32 and abs(g2[-1] - g_o) <= TOL_GOSA_F32 * g_o + floor
    assert boundary_equal(p2, a["p"])


@pytest.mark.parametrize("fusion,sum_mode", [(ofl.OFL_FUSE_RESIDUAL, ofl.OFL_SUM_F64),
                                             (ofl.OFL_FUSE_COPYBACK_SWAP, ofl.OFL_SUM_KAHAN_F32),
                                             (FUSE_ALL, ofl.OFL_SUM_F64), (0, ofl.OFL_SUM_KAHAN_F32)])
def test_pairs_in_every_form(fusion, sum_mode):
    say("pairs, fusion", fusion, "sum", sum_mode)
    a = synth.make_problem(131, 37, 45, seed=5)
    for iters in ([5], [6, 3], [4, 4]):
        p1, g1 = run(a, ofl.OFL_COEF_F32, iters, True, fusion, sum_mode)
        p2, g2 = run(a, ofl.OFL_COEF_F32, iters, False, fusion, sum_mode)
        assert np.array_equal(p1, p2)
        assert g1 == g2


def test_pairs_replay_and_continue():
    """Pairs replayed from graphs, with the program's own work between the
    replays, long enough for several graphs, and a change of omega."""
    say("pairs, replays")
    a = synth.make_problem(41, 23, 37, seed=6)
    one, two = ofl.Grid(a), ofl.Grid(a)
    ofl.ofl_set_profiling(one.handle, True)
    for iters, om in [(8, OMEGA), (8, OMEGA), (8, OMEGA), (300, OMEGA), (8, np.float32(0.7)), (5, OMEGA), (8, OMEGA)]:
        x1 = ofl.ofl_jacobi_run(one.handle, iters, om)
        x2 = ofl.ofl_jacobi_run(two.handle, iters, om)
        torch.ones(1000, device="cuda").sum().item()
        assert x1 == x2
        assert np.array_equal(one.p, two.p)
    assert ofl.ofl_residual(one.handle) == ofl.ofl_residual(two.handle)
    one.close()
    two.close()


# Sizes at which single grids take flat segments: one and several per plane,
# chunks of one and of several planes, pitches on and off multiples of 8.
@pytest.mark.parametrize("shape", [(161, 40, 45), (150, 70, 65), (97, 40, 80), (301, 40, 46), (130, 67, 61)])
@pytest.mark.parametrize("fmt", [ofl.OFL_COEF_F32, ofl.OFL_COEF_BF16_OFFSET])
@pytest.mark.parametrize("row_align", [0, 4])
def test_flat_pairs_equal_single_iterations(shape, fmt, row_align):
    say("flat pairs", shape, "format", fmt, "row_align", row_align)
    a = synth.make_problem(*shape, seed=31)
    for iters in ([3], [6, 5]):
        p1, g1 = run(a, fmt, iters, True, row_align=row_align)
        p2, g2 = run(a, fmt, iters, False, row_align=row_align)
        assert np.array_equal(p1, p2)
        assert g1 == g2


# ------------------------------------------------------------------ batches


def run_batch(probs, aligns, fmt, iters_list, own_tile, fusion=0):
    """own_tile: the default tile set by the caller, which keeps single iterations."""
    grids = [ofl.Grid(a, coef_format=fmt, row_align=ra) for a, ra in zip(probs, aligns)]
    b = ofl.ofl_batch_create([g.handle for g in grids])
    ofl.ofl_batch_set_fusion(b, fusion)
    if own_tile:
        ofl.ofl_batch_set_tile(b, ofl.ofl_batch_get_tile(b))
    gosa = [ofl.ofl_batch_run(b, n, OMEGA, len(grids)) for n in iters_list]
    ofl.ofl_batch_destroy(b)
    out = [g.p.copy() for g in grids]
    for g in grids:
        g.close()
    return out, gosa


# Planes shorter than a work-group's 2048 points, of several work-groups, ending
# on and off their bounds; pitches on and off multiples of 8; one row; few planes.
BATCHES = [
    [(3, 3, 3), (5, 4, 6)],
    [(33, 33, 65), (34, 66, 9), (36, 60, 12), (62, 130, 5)],
    [(161, 40, 20), (97, 41, 31), (129, 33, 9)],
    [(300, 7, 6), (33, 3, 40), (41, 23, 37)],
]


@pytest.mark.parametrize("fusion", [0, FUSE_ALL])
@pytest.mark.parametrize("fmt", [ofl.OFL_COEF_F32, ofl.OFL_COEF_BF16_OFFSET])
@pytest.mark.parametrize("shapes", BATCHES, ids=str)
def test_batch_pairs_equal_single_iterations(shapes, fmt, fusion):
    say("batch pairs", shapes, "format", fmt, "fusion", fusion)
    probs = [synth.make_problem(*s, seed=synth.grid_seed(70 + t)) for t, s in enumerate(shapes)]
    for aligns in ([4] * len(probs), [0, 8, 4, 32][:len(probs)]):
        iters = [3, 6, 6, 5]
        p1, g1 = run_batch(probs, aligns, fmt, iters, True, fusion)
        p2, g2 = run_batch(probs, aligns, fmt, iters, False, fusion)
        for x, y in zip(p1, p2):
            assert np.array_equal(x, y)
        assert g1 == g2


def test_two_batches_share_a_grid():
    """Pairs exchange a grid's buffers: another batch that holds it follows."""
    say("batches sharing a grid")
    probs = [synth.make_problem(41, 23, 37, seed=8), synth.make_problem(33, 20, 12, seed=9)]
    ref = [ofl.Grid(a, row_align=4) for a in probs]
    grids = [ofl.Grid(a, row_align=4) for a in probs]
    one = ofl.ofl_batch_create([grids[0].handle, grids[1].handle])
    two = ofl.ofl_batch_create([grids[0].handle])
    done = 0
    for b, n in ((one, 4), (two, 4), (one, 7), (two, 3), (one, 3)):
        ofl.ofl_batch_run(b, n, OMEGA, 2 if b is one else 1)
        done += n
    for g, n in zip(ref, (done, 14)):
        ofl.ofl_set_profiling(g.handle, True)
        ofl.ofl_jacobi_run(g.handle, n, OMEGA)
    for g, r in zip(grids, ref):
        assert np.array_equal(g.p, r.p)
    ofl.ofl_batch_destroy(two)
    ofl.ofl_batch_destroy(one)
    for g in grids + ref:
        g.close()
