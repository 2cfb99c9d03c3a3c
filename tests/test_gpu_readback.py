"""Residuals on their way to the host: ofl_residual as one sweep with its sum
against the three nest kernels (a tile of the caller's own keeps those), and the
residuals that kernels leave in pinned host memory, for more grids than the
process's page of slots holds and for a batch."""

import numpy as np
import pytest

import oracle
import paper_2011_03602_amd as ofl
import synth
from helpers import OMEGA, TOL_GOSA_F32, rel_err

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():  # collected on CPU hosts, skipped there
    pytestmark = [pytest.mark.gpu, pytest.mark.skip(reason="needs a GPU")]


# One point; sums shorter and longer than a pass of the summing work-group
# (8192 partials), rows of every vector width.
@pytest.mark.parametrize("shape", [(3, 3, 3), (33, 33, 65), (66, 11, 9), (131, 37, 45), (258, 61, 70), (65, 129, 260)])
@pytest.mark.parametrize("fmt", [ofl.OFL_COEF_F32, ofl.OFL_COEF_BF16, ofl.OFL_COEF_BF16_OFFSET])
def test_residual_in_one_sweep(shape, fmt):
    print("[gpu] residual", shape, fmt, flush=True)
    a = synth.make_problem(*shape, seed=11)
    g, own = ofl.Grid(a, coef_format=fmt), ofl.Grid(a, coef_format=fmt)
    ofl.ofl_set_tile(own.handle, ofl.ofl_get_tile(own.handle))
    for profiled in (False, False, True, False):
        ofl.ofl_set_profiling(g.handle, profiled)
        r, want = ofl.ofl_residual(g.handle), ofl.ofl_residual(own.handle)
        # the same FP64 terms, none negative, in another order of additions
        assert rel_err(r, want) <= a["p"].size * 2.0 ** -53
    if fmt == ofl.OFL_COEF_F32:  # (the oracle's coefficients are not rounded to bfloat16)
        assert rel_err(r, oracle.residual(a)) <= TOL_GOSA_F32
    assert np.array_equal(g.p, a["p"])
    s = ofl.ofl_get_stats(g.handle)
    assert list(s.gpu_nests) == [4, 4, 0] and list(s.gpu_regions) == [4, 4, 0]
    # the sweep left wrk2 as an iteration's would: the run goes on from it
    assert ofl.ofl_jacobi_run(g.handle, 3, OMEGA) == ofl.ofl_jacobi_run(own.handle, 3, OMEGA)
    assert np.array_equal(g.p, own.p)
    g.close()
    own.close()


def test_batch_residuals_are_each_grids_own():
    shapes = [(33, 20, 17), (70, 11, 9), (40, 40, 40)]
    arrays = [synth.make_problem(*s, seed=20 + t) for t, s in enumerate(shapes)]
    grids, lone = [ofl.Grid(a) for a in arrays], [ofl.Grid(a) for a in arrays]
    b = ofl.ofl_batch_create([g.handle for g in grids])
    for step in range(3):
        print("[gpu] batch residuals", step, flush=True)
        got = ofl.ofl_batch_run(b, 4, OMEGA, len(grids))
        for g, one, x in zip(grids, lone, got):
            want = ofl.ofl_jacobi_run(one.handle, 4, OMEGA)
            assert np.array_equal(g.p, one.p)
            assert rel_err(x, want) <= g.p.size * 2.0 ** -53
    ofl.ofl_batch_destroy(b)
    for g in grids + lone:
        g.close()


def test_more_grids_than_slots():
    """The first 64 grids read through slots, the others copy; slots go back."""
    a = synth.make_problem(5, 6, 7, seed=3)
    for step in range(2):
        print("[gpu] slots", step, flush=True)
        grids = [ofl.Grid(a) for _ in range(70)]
        got = {ofl.ofl_jacobi_run(g.handle, 1 + t % 2, OMEGA) for t, g in enumerate(grids)}
        assert len(got) == 2
        assert len({ofl.ofl_residual(g.handle) for g in grids[::2]}) == 1
        for g in grids:
            g.close()
