"""The threaded bfloat16 encoding of a grid's arrays (host code) against the
same encoding value by value, under the sanitizers."""

import os
import subprocess
import tempfile

import pytest

from test_sanitizers import CSRC, FLAGS, ROCM, ROOT, TESTS_CSRC, needs_toolchain


@needs_toolchain
@pytest.mark.parametrize("threads", [1, 5, 8])
def test_threaded_encoding_is_bitwise_the_serial_one(threads):
    with tempfile.TemporaryDirectory() as d:
        exe = os.path.join(d, "encode")
        subprocess.run(["g++", "-std=c++17", *FLAGS, "-D__HIP_PLATFORM_AMD__", f"-I{ROCM}/include", f"-I{ROOT}/include",
                        f"-I{CSRC}", os.path.join(TESTS_CSRC, "encode_check.cpp"), os.path.join(CSRC, "cpu_nests.cpp"),
                        "-o", exe, "-lpthread"], check=True)
        res = subprocess.run([exe], capture_output=True, text=True, timeout=300,
                             env=dict(os.environ, OFL_CPU_THREADS=str(threads)))
        assert res.returncode == 0 and "encoding ok" in res.stdout, res.stdout + res.stderr
