"""The multigrid's kernels with barriers on the CPU (tests/host/mg_levels.cpp on
tests/host/cpu/hip/hip_runtime.h): the coarse tail of every size class and the
tiled 2D launches, each lane run to its next wait before the others.  Bar: the
same bits in every order of the waves, and nothing read from LDS before it is
written (NaN at the start)."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HOST = os.path.join(ROOT, "tests", "host")


def test_levels_do_not_depend_on_the_waves_order(tmp_path):
    if not shutil.which("g++"):
        pytest.skip("g++ not available")
    exe = str(tmp_path / "mg_levels")
    cmd = ["g++", "-O1", "-std=c++17", "-ffp-contract=off", "-fno-extern-tls-init", "-w", "-I",
           os.path.join(HOST, "cpu"), "-I", os.path.join(ROOT, "include"), "-I",
           os.path.join(ROOT, "paper_2004_03275_amd", "csrc"), os.path.join(HOST, "mg_levels.cpp"), "-o", exe]
    out = subprocess.run(cmd, capture_output=True, text=True, timeout=300)
    assert out.returncode == 0, out.stderr[-3000:]
    out = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert out.returncode == 0, (out.stdout[-3000:], out.stderr[-1000:])
    assert out.stdout.strip().endswith("wrong 0")
