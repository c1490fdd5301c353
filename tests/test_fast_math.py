"""Step code compiled for the host: the FP64 logarithm, exponential, sine and
cosine (ems_math.hpp) against long double, the range-table search around the
table size from which it reads groups of nodes, and the walk of the box
hierarchy against a test of every box."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.parametrize("name", ["fast_math_check", "range_walk_check", "world_walk_check"])
def test_host_check(tmp_path, name):
    exe = tmp_path / name
    subprocess.run(["g++", "-O2", "-ffp-contract=off", "-std=c++17", os.path.join(ROOT, "tests", name + ".cpp"), "-o",
                    str(exe)], check=True, capture_output=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout
