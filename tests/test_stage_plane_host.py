"""The 2D stage kernel's own source on the CPU (tests/host/stage_plane_queue.cpp
on tests/host/cpu/hip/hip_runtime.h): each wave in turn runs from one barrier to
the next before any other moves, so a wait that is missing between the waves of
a workgroup (the queue's next leaf written over the one still to be read) gives
wrong leaves.  Bar: every schedule bit for bit the result of one workgroup per
leaf, a device-timed step's clock and Courant slots included."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2004_03275_amd", "csrc")
HOST = os.path.join(ROOT, "tests", "host")


def test_every_schedule_gives_the_same_leaves(tmp_path):
    if not shutil.which("g++"):
        pytest.skip("g++ not available")
    exe = str(tmp_path / "stage_plane_queue")
    cmd = ["g++", "-O1", "-std=c++17", "-ffp-contract=off", "-w", "-I", os.path.join(HOST, "cpu"), "-I",
           os.path.join(ROOT, "include"), "-I", CSRC, os.path.join(HOST, "stage_plane_queue.cpp"),
           os.path.join(CSRC, "forest.cpp"), "-pthread", "-o", exe]
    out = subprocess.run(cmd, capture_output=True, text=True, timeout=300)
    assert out.returncode == 0, out.stderr[-3000:]
    out = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert out.returncode == 0, (out.stdout[-3000:], out.stderr[-1000:])
    assert out.stdout.strip().endswith("wrong 0")
