"""The forest multigrid's kernels on the host, against its per-cell functions:
tests/host/fmg_kernels.cpp includes csrc/fmg.hip and runs the launches of a
V-cycle and of the residual check on the CPU (tests/host/cpu/hip/hip_runtime.h)
on a forest's block tree, built with the address and undefined-behaviour
checks.  Bar: bit for bit, the coarse-fine ghosts that a leaf keeps included;
arrays that nothing has written yet hold NaN."""
import os
import shutil
import subprocess

import pytest

import workloads as W

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HOST = os.path.join(ROOT, "tests", "host")


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    if not shutil.which("g++"):
        pytest.skip("g++ not available")
    exe = str(tmp_path_factory.mktemp("fmgkern") / "fmg_kernels")
    cmd = ["g++", "-O1", "-std=c++17", "-ffp-contract=off", "-w", "-fsanitize=address,undefined",
           "-fno-sanitize-recover=undefined", "-I", os.path.join(HOST, "cpu"), "-I", os.path.join(ROOT, "include"),
           "-I", os.path.join(ROOT, "paper_2004_03275_amd", "csrc"), os.path.join(HOST, "fmg_kernels.cpp"), "-o", exe]
    out = subprocess.run(cmd, capture_output=True, text=True, timeout=600)
    assert out.returncode == 0, out.stderr[-3000:]
    return exe


CASES = [
    # ndim, base, max_level, centre, radius
    (3, 1, 3, (0.2, 0.2, 0.2), 0.1),
    (3, 2, 2, (0.3, 0.35, 0.4), 0.1),
    (2, 4, 3, (0.27, 0.3), 0.15),
    (2, 2, 4, (0.5, 0.45), 0.2),
]


@pytest.mark.parametrize("bc", [0, 1])
@pytest.mark.parametrize("nd,base,max_level,centre,radius", CASES)
def test_kernels_equal_the_per_cell_functions(program, tmp_path, bc, nd, base, max_level, centre, radius):
    f = W.fmg_forest(W.fmg_scheme(base=base, max_level=max_level, bc=bc, ndim=nd), centre=centre, radius=radius)
    assert f.n >= 1
    s = f.scheme
    path = tmp_path / "forest.txt"
    with open(path, "w") as fh:
        fh.write(f"{f.n} {s.base_blocks[0]} {s.max_level} {bc} {nd}\n")
        for k in range(f.n):
            fh.write(f"{f.level[k]} {f.ijk[k, 0]} {f.ijk[k, 1]} {f.ijk[k, 2]}\n")
    out = subprocess.run([program, str(path)], capture_output=True, text=True, timeout=300)
    print(f.level_counts(), out.stdout.strip())
    assert out.returncode == 0, (out.stdout[-2000:], out.stderr[-3000:])
    assert "mismatches 0" in out.stdout
