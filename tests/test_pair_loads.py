"""Host side of the pair sweep's loads in row form: positions and alignment as a
property over many sizes, layouts and formats."""

import os
import subprocess
import tempfile

from test_sanitizers import CSRC, FLAGS, ROCM, ROOT, TESTS_CSRC, needs_toolchain


@needs_toolchain
def test_row_loads_hold_their_own_points():
    with tempfile.TemporaryDirectory() as d:
        exe = os.path.join(d, "loads")
        subprocess.run(["g++", "-std=c++17", *FLAGS, "-D__HIP_PLATFORM_AMD__", f"-I{ROCM}/include", f"-I{ROOT}/include",
                        f"-I{CSRC}", os.path.join(TESTS_CSRC, "pair_load_check.cpp"), "-o", exe], check=True)
        res = subprocess.run([exe], capture_output=True, text=True, timeout=300)
        assert res.returncode == 0 and "row loads ok" in res.stdout, res.stdout + res.stderr
