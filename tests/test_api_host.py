"""CPU check of the host side of the C ABI (include/loss.h): the calls run against stand-ins
for the HIP runtime and the kernels (tests/api_check.cpp), which check every copy, every
receiver and every trace sample a launch is given against the sizes of the allocations."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def api_check(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("api") / "api_check")
    csrc = os.path.join(ROOT, "paper_2301_05127_amd", "csrc")
    subprocess.check_call(["g++", "-O1", "-w", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                           "-I", os.path.join(ROOT, "include"), "-I", csrc, os.path.join(ROOT, "tests", "api_check.cpp"),
                           os.path.join(csrc, "tables.cpp"), "-o", exe])

    def run(*args):
        out = subprocess.run([exe] + [str(a) for a in args], capture_output=True, text=True, timeout=100)
        assert out.returncode == 0 and out.stdout.endswith("ok\n"), (args, out.returncode, out.stdout, out.stderr)
        return out.stdout.splitlines()[:-1]
    return run


@pytest.mark.parametrize("physics", [0, 1])
def test_receivers_exchanged_before_the_adjoint(api_check, physics):
    """The adjoint's recompute records into the traces that exist then: the tiles' receiver
    tables go with them when loss_get_traces has laid them out anew."""
    api_check("exchanged_receivers", physics)


@pytest.mark.parametrize("physics", [0, 1])
def test_gradient_of_more_receivers_than_the_last(api_check, physics):
    """The device copy of the residuals is as large as the traces of the current receivers."""
    api_check("added_receivers", physics)


# physics, intervals, patches, halo, shots: tiles of a pass
TILES = [
    (0, (1024, 0, 1024), (16, 64, 64), 8, 8, 17 * 16 * 8),    # across junctions along x alone
    (0, (1024, 0, 1024), (64, 64, 16), 8, 8, 17 * 16 * 8),    # along the rows alone
    (0, (1024, 0, 1024), (16, 64, 16), 8, 8, 17 * 16 * 8),
    (0, (1024, 0, 1024), (64, 64, 64), 8, 8, 17 * 16 * 8),    # no patch shorter than a piece
    (1, (256, 256, 256), (16, 64, 64), 8, 1, 5 * 4 * 257),
]


@pytest.mark.parametrize("case", TILES, ids=["%s_%s" % ("x".join(map(str, c[1])), "x".join(map(str, c[2]))) for c in TILES])
def test_tiles_of_mixed_patches(api_check, case):
    """Pieces across junctions are counted, and taken, axis by axis."""
    physics, n, M, halo, shots, tiles = case
    out = api_check("route", physics, *n, *M, halo, shots)
    assert int(out[0].split()[1]) == tiles, out


# physics, intervals, patches, halo, shots: the faster schedule as measured (0 tiles, 1 line passes)
SCHEDULES = [
    (0, (300, 0, 300), (4, 1, 4), 8, 2, 1),
    (0, (400, 0, 400), (7, 1, 7), 8, 1, 1),
    (0, (200, 0, 200), (7, 1, 7), 8, 1, 0),
    (0, (64, 0, 64), (2, 1, 2), 8, 2, 1),
    (0, (64, 0, 64), (2, 1, 2), 8, 1, 0),
    (0, (700, 0, 700), (4, 1, 64), 8, 4, 1),
    (0, (400, 0, 400), (8, 1, 8), 8, 8, 0),
    (0, (2048, 0, 2048), (256, 1, 256), 12, 1, 0),
    (1, (64, 64, 64), (5, 5, 5), 8, 1, 1),
    (1, (48, 48, 48), (5, 5, 5), 8, 1, 0),
    (1, (128, 128, 128), (4, 64, 8), 8, 1, 1),
    (1, (128, 128, 128), (16, 16, 16), 8, 1, 0),
]


@pytest.mark.parametrize("case", SCHEDULES, ids=["%s_%s_S%d" % ("x".join(map(str, c[1])), "x".join(map(str, c[2])), c[4])
                                                 for c in SCHEDULES])
def test_schedule_of_small_tiles(api_check, case):
    physics, n, M, halo, shots, schedule = case
    out = api_check("route", physics, *n, *M, halo, shots)
    assert int(out[0].split()[0]) == schedule, out


# physics, intervals, patches, halo, end mode: whole calls direct; halos beyond the tile passes;
# transposes of periodic lines and of halos wider than the patches staged
HOST_DERIV = [(0, (60, 0, 50), (30, 1, 25), 8, 0), (0, (60, 0, 50), (30, 1, 25), 24, 0), (0, (60, 0, 48), (30, 1, 24), 8, 2),
              (1, (20, 18, 16), (10, 9, 8), 6, 0), (1, (20, 18, 16), (5, 6, 8), 9, 0)]


@pytest.mark.parametrize("case", HOST_DERIV, ids=["p%d_%s_h%de%d" % (c[0], "x".join(map(str, c[2])), c[3], c[4]) for c in HOST_DERIV])
def test_host_derivatives_upload_once(api_check, case):
    physics, n, M, halo, end = case
    api_check("host_deriv", physics, *n, *M, halo, end)


@pytest.mark.parametrize("case", [(0, (130, 0, 97), (64, 1, 16), 8, 3), (0, (63, 0, 64), (63, 1, 64), 6, 1),
                                  (1, (33, 20, 17), (16, 10, 16), 6, 2)], ids=["acoustic", "one_piece", "elastic"])
def test_receivers_by_tile(api_check, case):
    """Receivers go to the tile that updates their node, in the order given."""
    physics, n, M, halo, shots = case
    api_check("tile_receivers", physics, *n, *M, halo, shots)


# nodes along x and z, shots, GiB of the device: floats per row
PITCH = [(17, 40, 1, 288, 20), (5, 40, 1, 288, 8), (65, 65, 1, 288, 68), (129, 129, 4, 288, 132), (184, 40, 1, 288, 192),
         (257, 40, 1, 288, 272), (513, 40, 1, 288, 528), (1024, 40, 1, 288, 1024), (513, 2049, 50, 4, 516)]


@pytest.mark.parametrize("case", PITCH, ids=["x%d_S%d_%dGiB" % (c[0], c[2], c[3]) for c in PITCH])
def test_row_padding_is_small(api_check, case):
    """Rows are padded past 16 bytes where that costs little memory, of a row and of the device."""
    out = api_check("pitch", *case[:4])
    assert int(out[0]) == case[4], out


@pytest.mark.parametrize("physics", [0, 1])
def test_runs_without_room_for_the_tiles(api_check, physics):
    """The tables of the tiles, their receivers and their words are optional: three refusals
    that a run survives, on the line passes."""
    out = api_check("refusals", physics)
    assert int(out[0]) == 3, out


def test_gradient_operands_make_room(api_check):
    api_check("operands")
