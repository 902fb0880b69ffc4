"""The arrival lines of the whole-chunk operations (csrc/arrive.h) on the CPU:
tests/host/arrivals.cpp runs the protocol itself with its atomics in random
orders, within one call and across calls of one plan that overlap.  Built with
g++; no device code."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_lines_are_zero_after_calls_in_any_order(tmp_path):
    if shutil.which("g++") is None:
        pytest.skip("needs g++")
    exe = str(tmp_path / "arrivals")
    b = subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Wno-unknown-pragmas",
                        "-I", os.path.join(ROOT, "paper_2509_03047_amd", "csrc"),
                        os.path.join(ROOT, "tests", "host", "arrivals.cpp"), "-o", exe],
                       capture_output=True, text=True, timeout=300)
    assert b.returncode == 0, b.stderr[-3000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout + r.stderr
