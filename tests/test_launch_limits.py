"""Launches of several threads per subvolume, leaf or entry at the counts where
they would pass the 2^32 threads of a launch (2^22 subvolumes with 16 wavefronts,
2^26 fold entries, 2^27 leaves): fewer wavefronts, or slices that cover every entry
once (`csrc/launch_limits.h`, compiled for the host).  No GPU."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_1803_07560_amd", "csrc")


def test_launches_fit_and_cover(tmp_path):
    if shutil.which("g++") is None:
        pytest.skip("g++ not available")
    exe = str(tmp_path / "launch_limits_check")
    r = subprocess.run(["g++", "-O1", "-std=c++17", "-Wall", "-Werror", "-I", CSRC,
                        os.path.join(HERE, "launch_limits_check.cpp"), "-o", exe],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    out = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert out.returncode == 0, out.stdout
