"""The tagged exchanges of the inner solvers never wait for a word that has been rewritten:
tests/tag_walk.cpp walks every interleaving of two workgroups of two waves over three steps of
each form, with the slots that the kernel uses (scalar_slot, vector_slot).  No GPU."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CXX = os.environ.get("CXX", "g++")


@pytest.fixture(scope="module")
def walk(tmp_path_factory):
    if shutil.which(CXX) is None:
        pytest.skip("no host C++ compiler")
    exe = tmp_path_factory.mktemp("walk") / "tag_walk"
    r = subprocess.run([CXX, "-std=c++17", "-O2", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                        os.path.join(ROOT, "tests", "tag_walk.cpp"), "-o", str(exe)],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    return lambda *a: subprocess.run([str(exe), *map(str, a)], capture_output=True, text=True,
                                     timeout=300)


def test_the_slots_of_the_kernel_leave_no_stuck_wait(walk):
    r = walk()
    assert r.returncode == 0, r.stdout + r.stderr


@pytest.mark.parametrize("slots,form", [((2, 2), "streaming"), ((4, 1), "single reduction")])
def test_the_walk_finds_a_slot_too_few(walk, slots, form):
    """Scalars that alternate between two slots, or vectors in one, do get stuck."""
    r = walk(*slots)
    assert r.returncode == 1
    assert any(l.startswith(form) and not l.endswith(" 0 stuck") for l in r.stdout.splitlines())
