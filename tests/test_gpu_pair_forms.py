"""Every form of the pair sweep against the same iterations nest by nest, bitwise,
at sizes for which the decomposition rule (asked on the host) takes that form."""

import os
import subprocess
import sys

import numpy as np
import pytest

import paper_2011_03602_amd as ofl
import synth
from helpers import OMEGA
from test_sanitizers import CSRC, ROCM, ROOT, TESTS_CSRC, needs_toolchain

torch = pytest.importorskip("torch")
pytestmark = [pytest.mark.gpu, needs_toolchain]

if not torch.cuda.is_available():  # collected on CPU hosts, skipped there
    pytestmark = [pytest.mark.gpu, pytest.mark.skip(reason="needs a GPU")]

F32, BF16, BF16_OFFSET = ofl.OFL_COEF_F32, ofl.OFL_COEF_BF16, ofl.OFL_COEF_BF16_OFFSET


@pytest.fixture(scope="module")
def shape_of(tmp_path_factory):
    """The rule's (form, points per lane, waves, tiles) for a grid."""
    exe = str(tmp_path_factory.mktemp("pair") / "shape")
    subprocess.run(["g++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", f"-I{ROCM}/include", f"-I{ROOT}/include",
                    f"-I{CSRC}", os.path.join(TESTS_CSRC, "pair_shape.cpp"), "-o", exe], check=True)

    def ask(shape, row_align, fmt):
        line = " ".join(map(str, (*shape, row_align, 4 if fmt == F32 else 2)))
        out = subprocess.run([exe], input=line, capture_output=True, text=True, check=True).stdout.split()
        return (out[0], *map(int, out[1:]))

    return ask


def run(a, fmt, row_align, iters_list, profiled):
    g = ofl.Grid(a, coef_format=fmt, row_align=row_align)
    ofl.ofl_set_profiling(g.handle, profiled)
    ofl.ofl_data_enter(g.handle)
    gosa = [ofl.ofl_jacobi_run(g.handle, n, OMEGA) for n in iters_list]
    ofl.ofl_data_exit(g.handle)
    p = g.p.copy()
    g.close()
    return p, gosa


def check(shape, fmt, row_align):
    print("[gpu] pair form", shape, "format", fmt, "row_align", row_align, flush=True)
    sys.stdout.flush()
    a = synth.make_problem(*shape, seed=synth.grid_seed(sum(shape)))
    for iters in ([3], [6, 5]):  # one pair; two of them behind a single iteration, then two
        p1, g1 = run(a, fmt, row_align, iters, True)
        p2, g2 = run(a, fmt, row_align, iters, False)
        assert np.array_equal(p1, p2)
        assert g1 == g2


# Rows of one to four tiles of 256 points, ending at, before and past a tile.
ROW4 = [
    ((257, 45, 33), BF16_OFFSET, 0, 7, 1), ((242, 117, 33), BF16, 0, 7, 1), ((257, 45, 61), BF16, 0, 8, 1),
    ((505, 29, 61), BF16_OFFSET, 0, 7, 2), ((442, 85, 33), BF16, 0, 8, 2), ((700, 45, 33), BF16, 0, 7, 3),
    ((750, 29, 33), BF16_OFFSET, 0, 8, 3),
    ((255, 45, 33), F32, 0, 7, 1), ((257, 85, 33), F32, 0, 8, 1), ((505, 45, 33), F32, 0, 7, 2),
    ((410, 61, 33), F32, 0, 8, 2), ((750, 33, 33), F32, 0, 7, 3), ((700, 29, 61), F32, 0, 8, 3),
    ((770, 29, 61), F32, 0, 8, 4),
    ((255, 29, 61), BF16, 4, 7, 1), ((257, 61, 145), F32, 4, 8, 1), ((505, 33, 61), F32, 4, 8, 2),
    ((750, 33, 33), F32, 4, 7, 3), ((750, 29, 33), BF16_OFFSET, 8, 8, 3),
    ((242, 117, 33), BF16, 8, 7, 1), ((442, 85, 33), BF16_OFFSET, 8, 8, 2), ((410, 61, 33), F32, 8, 8, 2),
]


@pytest.mark.parametrize("shape,fmt,row_align,waves,tiles", ROW4, ids=str)
def test_rows_at_four_points_per_lane(shape_of, shape, fmt, row_align, waves, tiles):
    assert shape_of(shape, row_align, fmt) == ("row", 4, waves, tiles)
    check(shape, fmt, row_align)


# bfloat16 rows of 4 points more than a multiple of 8, which 16-byte loads do not
# divide (I % 8 of 2, 3 and 4 have interior points past the last whole load).
@pytest.mark.parametrize("fmt", [BF16, BF16_OFFSET])
@pytest.mark.parametrize("shape", [(250, 33, 145), (442, 61, 61), (250, 117, 33), (251, 33, 129), (411, 65, 65),
                                   (252, 33, 129), (500, 61, 33)], ids=str)
def test_bfloat16_rows_that_loads_do_not_divide(shape_of, shape, fmt):
    form, vec, _, _ = shape_of(shape, 4, fmt)
    assert form == "flat" or (form == "row" and vec < 4)
    check(shape, fmt, 4)


# Flat segments of single grids, pitches on and off multiples of 8.
@pytest.mark.parametrize("shape,fmt,row_align", [((150, 70, 65), F32, 0), ((150, 150, 40), BF16, 0),
                                                 ((161, 161, 45), BF16_OFFSET, 4), ((301, 99, 60), F32, 4),
                                                 ((301, 99, 60), BF16, 0), ((150, 150, 65), BF16_OFFSET, 4)], ids=str)
def test_flat_segments(shape_of, shape, fmt, row_align):
    assert shape_of(shape, row_align, fmt)[0] == "flat"
    check(shape, fmt, row_align)
