"""Alignment that the slot stores of the single-species kernels promise to the compiler (CPU: the generated IR).

Rows of a width that fills no whole 16 bytes start the last lane's columns at any column, so a vector store may be
taken as aligned to one value only."""
import os
import re
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_slot_stores_promise_the_alignment_of_a_value(tmp_path):
    from paper_1902_02064_amd.build import CSRC, FLAGS, HIPCC
    if not os.path.exists(HIPCC):
        pytest.skip("no HIP compiler")
    out = tmp_path / "flytile.ll"
    cmd = [HIPCC, *FLAGS, "-O1", "-x", "hip", "--cuda-device-only", "-S", "-emit-llvm",
           os.path.join(CSRC, "flytile.hip"), "-o", str(out)]
    subprocess.run(cmd, check=True, capture_output=True, cwd=ROOT, timeout=300)
    stores = re.findall(r"store <\d+ x (double|float)> .*addrspace\(1\).*align (\d+)", out.read_text())
    assert {t for t, _ in stores} == {"double", "float"}
    assert all(int(a) <= {"double": 8, "float": 4}[t] for t, a in stores)
