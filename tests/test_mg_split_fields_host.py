"""Fields of the 3D multigrid that are aligned as doubles and no more (a
contiguous slice at an odd offset): tests/host/mg_split_fields.cpp runs the
kernels that take them in pairs of cells on the CPU with g++'s alignment check.
Bar: no misaligned access assumed aligned, results bit for bit those on
16-byte aligned fields."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HOST = os.path.join(ROOT, "tests", "host")


def test_fields_aligned_as_doubles(tmp_path):
    if not shutil.which("g++"):
        pytest.skip("g++ not available")
    exe = str(tmp_path / "mg_split_fields")
    cmd = ["g++", "-O1", "-std=c++17", "-ffp-contract=off", "-w", "-fsanitize=alignment",
           "-fno-sanitize-recover=alignment", "-I", os.path.join(HOST, "cpu"), "-I", os.path.join(ROOT, "include"),
           "-I", os.path.join(ROOT, "paper_2004_03275_amd", "csrc"), os.path.join(HOST, "mg_split_fields.cpp"),
           "-o", exe]
    out = subprocess.run(cmd, capture_output=True, text=True, timeout=300)
    assert out.returncode == 0, out.stderr[-3000:]
    out = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert out.returncode == 0, (out.stdout[-2000:], out.stderr[-2000:])
    assert out.stdout.strip() == "wrong 0"
