"""CPU check of the tile passes (paper Sec. 3.1-3.2: patch systems with PMBC junctions):
every index their kernels form along an axis, and the two solves of the slopes, the moments
and the transposed slopes as the kernels evaluate them in FP32 against the patch systems in FP64 (tests/tile_check.cpp)."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

# N, M, halo, end mode: the workloads' axes, patches longer than a tile (64), remainders of
# one interval and up, halos wider than the patches, the other end rows
AXES = [(512, 64, 12, 0), (256, 64, 10, 0), (2048, 256, 12, 0), (1024, 128, 12, 0), (128, 64, 8, 0), (64, 64, 8, 0),
        (65, 64, 8, 0), (130, 64, 12, 0), (1100, 128, 10, 0), (183, 48, 8, 0), (50, 16, 6, 0), (40, 8, 6, 0),
        (48, 8, 20, 0), (37, 3, 2, 0), (63, 63, 5, 0), (100, 100, 4, 0), (5, 4, 2, 0), (96, 24, 8, 1), (130, 65, 12, 1),
        (48, 24, 10, 2), (96, 8, 20, 2), (300, 100, 9, 2), (71, 70, 20, 0), (128, 64, 10, 0), (141, 40, 8, 0), (300, 24, 10, 0), (130, 16, 12, 0),
        (130, 16, 12, 2), (160, 32, 12, 2), (210, 32, 9, 0), (100, 20, 9, 1), (40, 8, 8, 0), (71, 16, 7, 0), (96, 8, 7, 0)]


@pytest.fixture(scope="module")
def host_check(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("tile") / "tile_check")
    csrc = os.path.join(ROOT, "paper_2301_05127_amd", "csrc")
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I", csrc,
                           os.path.join(ROOT, "tests", "tile_check.cpp"), os.path.join(csrc, "tables.cpp"), "-o", exe])
    return exe


@pytest.mark.parametrize("across", [0, 1])
@pytest.mark.parametrize("op", [0, 1, 2])
@pytest.mark.parametrize("axis", AXES, ids=["N%d_M%d_h%d_e%d" % a for a in AXES])
def test_tile_tables_and_indices(host_check, axis, op, across):
    out = subprocess.run([host_check] + [str(v) for v in axis + (op, across)], capture_output=True, text=True)
    assert out.returncode == 0, out.stdout
    N, M, halo, end = axis
    if across and (op == 1 or not 8 <= M < 64 or N <= M):
        assert out.stdout.startswith("unsupported"), out.stdout
        return
    if out.stdout.startswith("unsupported"):
        # the transposed taps of a junction may reach the two pieces it separates only
        assert op == 2 and (end == 2 or halo >= min(M, N % M or M)), out.stdout
        return
    assert out.stdout.startswith("ok"), out.stdout
    # FP32 rounding of diagonally dominant systems (condition at most 3) on white noise
    tol = 5e-6 if op == 1 else 2e-6
    assert max(float(v) for v in out.stdout.split()[1:]) < tol, out.stdout
