"""When iterations go in pairs, on the stand-in HIP runtime with counting
launchers (host code only)."""

import os
import subprocess
import tempfile

from test_sanitizers import _build, needs_toolchain


@needs_toolchain
def test_pairs_follow_the_calls_not_their_history():
    with tempfile.TemporaryDirectory() as d:
        exe = _build(d, ["hip_stand_in.cpp", "launch_noop.cpp", "pair_count.cpp"], "pair_policy_check", [])
        env = dict(os.environ, ASAN_OPTIONS="detect_leaks=1:abort_on_error=1", UBSAN_OPTIONS="print_stacktrace=1")
        res = subprocess.run([exe], capture_output=True, text=True, env=env, timeout=300)
        assert res.returncode == 0 and "pair policy ok" in res.stdout, res.stdout + res.stderr
