"""Lists of work items (`list_items`, `ItemCount` in `csrc/runtime.h`): every sample
in one item, record slots in list order, whole items before rests, the rests by
falling length; chunks and counts at their edges; and a list of 10^6 ragged leaves
at the cost of a pass over it, not of a sort.  A C++ program linked with the
library; no GPU."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
PKG = os.path.join(ROOT, "paper_1803_07560_amd")


def test_lists(tmp_path):
    if shutil.which("g++") is None or not os.path.exists("/opt/rocm/include"):
        pytest.skip("g++ or the ROCm headers not available")
    if not os.path.exists(os.path.join(PKG, "libbfi.so")):
        pytest.skip("library not built")
    exe = str(tmp_path / "item_list_check")
    r = subprocess.run(["g++", "-O2", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I",
                        os.path.join(ROOT, "include"), "-I", os.path.join(PKG, "csrc"), "-isystem",
                        "/opt/rocm/include", os.path.join(HERE, "item_list_check.cpp"), "-o", exe,
                        "-L", PKG, "-lbfi", "-Wl,-rpath," + PKG, "-L/opt/rocm/lib", "-lamdhip64",
                        "-Wl,-rpath,/opt/rocm/lib", "-lrocprofiler-sdk-roctx"],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    out = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert out.returncode == 0, out.stdout
