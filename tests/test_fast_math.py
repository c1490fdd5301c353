"""The FP64 logarithm, exponential, sine and cosine of the step code
(ems_math.hpp), compiled for the host, against long double."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_fast_math_against_long_double(tmp_path):
    exe = tmp_path / "fast_math_check"
    subprocess.run(["g++", "-O2", "-std=c++17", os.path.join(ROOT, "tests", "fast_math_check.cpp"), "-o", str(exe)],
                   check=True, capture_output=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout
