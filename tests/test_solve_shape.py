"""The launch shape and workspace of the persistent solve for every size, form and device size that the entry
points accept (tests/shape_checks.cpp; host code only)."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CXX = os.environ.get("CXX", "g++")


@pytest.mark.skipif(shutil.which(CXX) is None, reason="no host C++ compiler")
def test_every_accepted_call_has_a_shape(tmp_path):
    exe = tmp_path / "shape_checks"
    r = subprocess.run([CXX, "-std=c++17", "-O1", "-Wall", "-D__HIP_PLATFORM_AMD__",
                        "-I/opt/rocm/include",
                        os.path.join(ROOT, "tests", "shape_checks.cpp"), "-o", str(exe)],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout + r.stderr
