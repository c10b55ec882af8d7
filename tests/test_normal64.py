"""The samplers' double-precision functions (`csrc/normal64.hpp`), compiled for
the host from the same source (IEEE operations only, so the same bits as on the
GPU but for the hardware's reciprocal approximations, which are given errors of
2^-22 here), against long double over two million arguments: every word's
uniform at both ends and around every 64th of the range, and random ones.
Bounds, in units in the last place: the logarithm sums two rounded terms, of
which the table's may be twice the result (1/2 + 1/2 + 1/2, and the series'
leading terms); the root and the reciprocals end on a correction by an exact
residual; sine and cosine are the sum of two products with rounded table
entries (four half units of 1, counted in units of 1/8 where they are small).
No GPU."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_1803_07560_amd", "csrc")
BOUNDS = {"log_word": 2.0, "log": 2.0, "cos": 4.0, "sin": 4.0, "root": 0.51, "rroot": 1.0,
          "reciprocal": 1.0}


def test_errors_against_long_double(tmp_path):
    if shutil.which("g++") is None:
        pytest.skip("g++ not available")
    exe = str(tmp_path / "normal64_check")
    r = subprocess.run(["g++", "-O2", "-std=c++17", "-Wall", "-Werror", "-ffp-contract=off",
                        "-I", CSRC, os.path.join(HERE, "normal64_check.cpp"), "-o", exe],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    out = subprocess.run([exe], capture_output=True, text=True, timeout=120).stdout
    got = {n: (float(a), float(b)) for n, a, b in (line.split() for line in out.splitlines())}
    assert set(got) == set(BOUNDS)
    for name, (most, mean) in got.items():
        assert most <= BOUNDS[name], (name, most)
        assert mean <= 0.5, (name, mean)
