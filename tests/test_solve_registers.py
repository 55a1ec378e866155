"""Registers of the persistent solve's instances, as the compiler recorded them in the library:
up to 512 columns every form leaves room for two workgroups per CU (256 registers), which the
gradient pass needs to keep enough of A in flight; no form spills more than the widest streaming
one needs.  No GPU."""
import os
import re
import struct
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_1912_03514_amd", "libmihs.so")
READELF = "/opt/rocm/llvm/bin/llvm-readelf"
pytestmark = pytest.mark.skipif(not os.path.exists(LIB) or not os.path.exists(READELF),
                                reason="needs the built library and llvm-readelf")


def _device_objects(path):
    """The AMDGPU ELF images inside the library."""
    blob = open(path, "rb").read()
    for m in re.finditer(rb"\x7fELF\x02\x01\x01\x40", blob):  # 64-bit, OS ABI of the GPU runtime
        at = m.start()
        shoff, = struct.unpack_from("<Q", blob, at + 40)
        shentsize, shnum = struct.unpack_from("<HH", blob, at + 58)
        yield blob[at:at + shoff + shentsize * shnum]


def _kernels(tmp_path):
    out = {}
    for i, image in enumerate(_device_objects(LIB)):
        p = tmp_path / f"{i}.elf"
        p.write_bytes(image)
        notes = subprocess.run([READELF, "--notes", str(p)], capture_output=True, text=True,
                               check=True).stdout
        for block in notes.split("- .agpr_count:")[1:]:
            name = re.search(r"\.name:\s+(\S+)", block).group(1)
            out[name] = {k: int(re.search(rf"\.{k}:\s+(\d+)", block).group(1))
                         for k in ("vgpr_count", "private_segment_fixed_size")}
    return out


def test_two_workgroups_per_cu_and_bounded_spills(tmp_path):
    forms = {}
    for name, res in _kernels(tmp_path).items():
        m = re.match(r"_ZN4mihs12solve_kernelI(\w)(\w)(\w)Li(\d+)ELb(\d)ELb(\d)E", name)
        if m:
            forms[m.groups()] = res
    # four type pairs; both streaming forms at seven widths, and the Gram forms
    assert len(forms) >= 4 * 14
    for (ta, ts, _, ept, gram, res), r in forms.items():
        what = f"A {ta}, operator {ts}, {64 * int(ept)} columns, gram {gram}, resident {res}: {r}"
        if int(ept) <= 8:
            assert r["vgpr_count"] <= 256, what
        assert r["private_segment_fixed_size"] <= 600, what
