"""The rounds of the mesh kernel's trees (csrc/tokens.hpp) built for the host, a fiber per thread, and
run under different orders of a work-group's threads between two barriers: every thread passes
the same barriers, also when a departure count overflows while tokens walk, and the trees are the
serial algorithm's."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)


def test_threads_leave_the_rounds_together(tmp_path):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("g++ not available")
    # next to its stand-ins, so that the kernel's own includes are not taken
    for f in ("tests/token_rounds/pop.hpp", "tests/token_rounds/rounds.cpp", "paper_2510_20604_amd/csrc/tokens.hpp"):
        shutil.copy(os.path.join(ROOT, f), tmp_path)
    exe = tmp_path / "rounds"
    subprocess.run([gxx, "-std=c++17", "-O1", "-fno-strict-aliasing", "-Wno-unknown-pragmas", "rounds.cpp", "-o", str(exe)],
                   cwd=tmp_path, check=True, capture_output=True)
    res = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert res.returncode == 0, res.stdout
