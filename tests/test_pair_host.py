"""Host side of the iterations in pairs: the decomposition rule as a property
over many sizes, and the device-error paths of a run that goes in pairs (on the
stand-in HIP runtime, every HIP call failing in turn)."""

import os
import subprocess
import tempfile

from test_sanitizers import CSRC, FLAGS, ROCM, ROOT, TESTS_CSRC, _build, needs_toolchain


@needs_toolchain
def test_pair_decomposition_covers_every_grid():
    with tempfile.TemporaryDirectory() as d:
        exe = os.path.join(d, "plan")
        subprocess.run(["g++", "-std=c++17", *FLAGS, "-D__HIP_PLATFORM_AMD__", f"-I{ROCM}/include", f"-I{ROOT}/include",
                        f"-I{CSRC}", os.path.join(TESTS_CSRC, "pair_plan_check.cpp"), "-o", exe], check=True)
        res = subprocess.run([exe], capture_output=True, text=True, timeout=300)
        assert res.returncode == 0 and "pair plans ok" in res.stdout, res.stdout + res.stderr


@needs_toolchain
def test_device_errors_are_sticky_and_leak_nothing_in_pairs():
    with tempfile.TemporaryDirectory() as d:
        exe = _build(d, ["hip_stand_in.cpp", "launch_noop.cpp", "pair_noop.cpp"], "fault_check", [])
        env = dict(os.environ, ASAN_OPTIONS="detect_leaks=1:abort_on_error=1", UBSAN_OPTIONS="print_stacktrace=1")
        res = subprocess.run([exe], capture_output=True, text=True, env=env, timeout=600)
        assert res.returncode == 0, res.stdout + res.stderr
        assert "device-error paths ok" in res.stdout


@needs_toolchain
def test_flat_segments_cover_every_grid_they_are_chosen_for():
    with tempfile.TemporaryDirectory() as d:
        exe = os.path.join(d, "flat")
        subprocess.run(["g++", "-std=c++17", *FLAGS, "-D__HIP_PLATFORM_AMD__", f"-I{ROCM}/include", f"-I{ROOT}/include",
                        f"-I{CSRC}", os.path.join(TESTS_CSRC, "pair_flat_check.cpp"), "-o", exe], check=True)
        res = subprocess.run([exe], capture_output=True, text=True, timeout=300)
        assert res.returncode == 0 and "flat choices ok" in res.stdout, res.stdout + res.stderr
