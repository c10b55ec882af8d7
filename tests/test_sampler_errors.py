"""The samplers' double-precision functions (`csrc/normal64.hpp`) are no further
off than the device library's, in whose place they stand: compiled for the host
from the same source and compared with long double over their whole ranges, in
units in the last place of the result however small it is.  The bounds are the
largest and mean errors of `log`, `sincospi`, `sqrt` with a division, and `pow`
on an MI355X over the same kinds of arguments (4 million words; the quotient's
largest is bounded by its two roundings, 1/2 of a root that may stand at the top
of its binade and 1/2).  No GPU."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_1803_07560_amd", "csrc")
LIBRARY = {"log": (0.635, 0.252), "cos": (0.874, 0.258), "sin": (0.873, 0.258),
           "over_root": (1.5, 0.347)}
POWER = {3: (3.71, 0.297), 4: (1.28, 0.266), 6: (2.0, 0.266), 8: (1.08, 0.257), 15: (0.94, 0.253),
         16: (0.96, 0.253), 20: (1.09, 0.253), 32: (0.72, 0.252)}
LIBRARY |= {f"{part}{d}": bound for d, bound in POWER.items() for part in ("inner", "shell")}


def test_no_further_off_than_the_library(tmp_path):
    if shutil.which("g++") is None:
        pytest.skip("g++ not available")
    exe = str(tmp_path / "sampler_errors_check")
    r = subprocess.run(["g++", "-O2", "-std=c++17", "-Wall", "-Werror", "-ffp-contract=off",
                        "-I", CSRC, os.path.join(HERE, "sampler_errors_check.cpp"), "-o", exe],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    out = subprocess.run([exe], capture_output=True, text=True, timeout=300).stdout
    got = {n: (float(a), float(b)) for n, a, b in (line.split() for line in out.splitlines())}
    assert set(got) == set(LIBRARY)
    for name, (most, mean) in got.items():
        assert most <= LIBRARY[name][0], (name, most)
        assert mean <= LIBRARY[name][1], (name, mean)
