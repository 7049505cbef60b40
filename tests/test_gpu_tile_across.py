"""Tile passes whose pieces reach across junctions along one axis only: patches shorter than a
piece along it, of a piece or longer along the other (Sec. 3.2), on enough tiles for the rule
to take such pieces, against the FP64 oracle and the line passes."""
import numpy as np
import pytest

from gpu_util import announce, require_gpu
from test_gpu_acoustic import _f32
from test_gpu_tile import _check, _src

pytestmark = pytest.mark.gpu

MIXED = [
    # intervals, patches, halo, end mode, layer, copies of the two shots (over 2500 tiles between junctions)
    ((205, 0, 200), (8, 1, 100), 8, 0, 0, 13),
    ((150, 0, 205), (75, 1, 8), 8, 2, 0, 17),
    ((197, 0, 130), (16, 1, 64), 12, 0, 10, 35),
]


@pytest.mark.parametrize("geom", MIXED, ids=["x".join(map(str, g[0])) + "e%dl%d" % g[3:5] for g in MIXED])
def test_acoustic_mixed_patches_match_oracle(orc, geom):
    require_gpu()
    from paper_2301_05127_amd import inputs
    n, M, halo, end, layer, copies = geom
    announce("acoustic mixed patches %s" % (geom,))
    g = inputs.grid(2, n, (10.0, 10.0, 10.0), M, halo, end)
    shape = inputs.field_shape(g)
    dt, nsteps = 1e-3, 40
    vp = 2500.0 * (1.0 + 0.1 * inputs.gaussian_random_field(shape, 10.0, 60.0, 9, -1.0, 1.0))
    cx, cz = 10.0 * (n[0] // 2), 10.0 * (n[2] // 2)
    rec = np.array([[i, 0, n[2] // 2 + 2] for i in range(2, n[0] - 1, 3)], np.int32)
    shots = [{"sources": [_src(0, (cx + 3.0, 0.0, cz - 2.0), 30.0, dt, nsteps)], "receivers": rec, "rec_comp": 0},
             {"sources": [_src(2, (cx, 0.0, cz), 30.0, dt, nsteps)], "receivers": rec, "rec_comp": 0}]
    w = _f32(dict(grid=g, physics=0, dt=dt, nsteps=nsteps, vp=vp, vs=None, rho=np.full(shape, 1000.0), shots=shots))
    _check(orc, w, layer, copies=copies)
