"""The transposed tile passes (x and row parts of D^T in one kernel, the z parts of three
bars in another) against the FP64 adjoint oracle at the sizes where they can go wrong: cut
patches, a last piece of one interval, rows that do not fill a wave, the other end rows, and
a grid whose transposed taps reach past the neighbouring piece (periodic: the line passes)."""
import numpy as np
import pytest

from gpu_util import announce, rel_l2, require_gpu
from test_gpu_adjoint_elastic import _f32, _gpu_grad, _obs, _oracle_grad

pytestmark = pytest.mark.gpu

# the bound of the repository's gradient tests: FP32 passes in both directions.  The acoustic
# runs are a few steps of a source as wide as the grid, with white residuals at receivers all
# over it: the gradient is a product of two wavefields, whose rounding counts relative to
# their maxima, so both have to fill the grid; and over tens of steps the natural end rows
# of grids this small grow rounding, whichever kernels run.
TOL = 1e-4

ACOUSTIC = [
    ((66, 0, 130), (66, 64, 128), 10, 0),    # cut patches
    ((65, 0, 64), (64, 64, 64), 6, 0),       # a last x piece of one interval
    ((70, 0, 65), (35, 64, 64), 6, 1),       # a last row piece of one interval; end stencil
    ((48, 0, 52), (24, 26, 26), 6, 2),       # periodic
    ((205, 0, 200), (8, 64, 8), 6, 0, 6),    # pieces across junctions
]
ELASTIC = [
    ((66, 18, 20), (66, 18, 20), 8, 0),      # cut x patch
    ((20, 66, 17), (20, 66, 16), 8, 0),      # cut rows; a last z piece of one interval
    ((17, 25, 22), (16, 12, 11), 5, 1),      # a last x piece and a last row piece of one interval
    ((56, 48, 36), (8, 8, 9), 6, 0),         # pieces across junctions
]


@pytest.mark.parametrize("geom", ACOUSTIC, ids=["x".join(map(str, g[0])) + "e%d" % g[3] for g in ACOUSTIC])
def test_acoustic_tile_gradient_matches_oracle(orc, geom):
    require_gpu()
    from paper_2301_05127_amd import inputs, loss
    n, M, halo, end = geom[:4]
    announce("acoustic tile gradient %s" % (geom,))
    g = inputs.grid(2, n, (10.0, 10.0, 10.0), M, halo, end)
    shape = inputs.field_shape(g)
    dt, nsteps, S = 1e-3, 12, (geom + (2,))[4]
    vp = _f32(inputs.gaussian_random_field(shape, 10.0, 80.0, 5, 2000.0, 2400.0))
    rho = np.full(shape, 1000.0)
    rec = np.array([[ix, 0, iz] for iz in range(0, n[2] + 1, 4) for ix in range(0, n[0] + 1, 5)], np.int32)
    shots = [{"sources": [{"kind": 0, "pos": (10.0 * (n[0] // 3) * (s % 2 + 1), 0.0, 10.0 * (n[2] // 2)), "spread": 300.0,
                           "wavelet": _f32(inputs.ricker(40.0, 0.004, dt, nsteps + 1, 0.5))}],
              "receivers": rec, "rec_comp": 0} for s in range(S)]
    res = np.random.default_rng(3).standard_normal((S, len(rec), nsteps))
    ref = sum(orc.acoustic_adjoint(g, dt, nsteps, vp, rho, sh["sources"], rec, res[s]) for s, sh in enumerate(shots))
    for sched in (0, 1):
        sim = loss.Simulation(g, 0, dt, nshots=S, trace_len=nsteps)
        sim.setup_workload(dict(grid=g, physics=0, dt=dt, nsteps=nsteps, vp=vp, vs=None, rho=rho, shots=shots))
        sim.set_shape([None, None, None, sched])
        sim.forward_ckpt(nsteps, 5)
        e = rel_l2(sim.adjoint(res.ravel(), loss.GRAD_K), ref)
        sim.close()
        print("schedule %d rel-L2 %.2e" % (sched, e))
        assert e < TOL, (sched, e)


@pytest.mark.parametrize("geom", ELASTIC, ids=["x".join(map(str, g[0])) + "e%d" % g[3] for g in ELASTIC])
def test_elastic_tile_gradient_matches_oracle(orc, geom):
    require_gpu()
    from paper_2301_05127_amd import inputs, loss
    n, M, halo, end = geom
    announce("elastic tile gradient %s" % (geom,))
    g = inputs.grid(3, n, (10.0, 10.0, 10.0), M, halo, end)
    shape = inputs.field_shape(g)
    vp = _f32(inputs.gaussian_random_field(shape, 10.0, 40.0, 61, 2800.0, 3300.0))
    vs = _f32(vp / np.sqrt(3.0))
    rho = _f32(inputs.gaussian_random_field(shape, 10.0, 40.0, 62, 2000.0, 2400.0))
    nsteps = 30

    def src(kind, shift):
        return {"kind": kind, "pos": tuple(5.0 * v for v in n), "spread": 15.0,
                "wavelet": _f32(inputs.ricker(50.0, 0.02, 1e-3, nsteps + 1, shift))}

    rec = np.array([[ix, n[1] // 2, n[2] // 2 + 3] for ix in range(3, n[0] - 2, 3)], np.int32)
    w = dict(grid=g, physics=1, dt=1e-3, nsteps=nsteps, vp=vp, vs=vs, rho=rho,
             shots=[{"sources": [src(1, 0.5)], "receivers": rec, "rec_comp": 2},
                    {"sources": [src(3, 0.0)], "receivers": rec, "rec_comp": 6}])
    obs = _obs(orc, w)
    gpu, _ = _gpu_grad(w, obs, loss.GRAD_LAME_RHO, 12)
    # the oracle's third output is dJ/db of b = 1/rho
    ref = _oracle_grad(orc, w, obs, with_b=True)
    e = [rel_l2(gpu[0], ref[0]), rel_l2(gpu[1], ref[1]), rel_l2(gpu[2], -ref[2] / rho ** 2)]
    print("rel-L2 lambda %.2e mu %.2e rho %.2e" % tuple(e))
    assert max(e) < TOL, e
