"""Tile passes whose pieces reach across junctions, on enough tiles for the rule to take such
pieces: along one axis only (patches shorter than a piece along it, of a piece or longer along
the other, Sec. 3.2), against the FP64 oracle and the line passes; and in the recompute of a
gradient through the absorbing layer (derivatives kept, memory variables and junctions inside
at once), against the oracle's layer adjoints."""
import numpy as np
import pytest

from gpu_util import announce, rel_l2, require_gpu
from test_gpu_acoustic import _f32 as _round_workload
from test_gpu_adjoint_elastic import _f32
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
    w = _round_workload(dict(grid=g, physics=0, dt=dt, nsteps=nsteps, vp=vp, vs=None, rho=np.full(shape, 1000.0), shots=shots))
    _check(orc, w, layer, copies=copies)


# the bound of the repository's gradient tests; white residuals at receivers all over the inner
# grid and a source as wide as it, so that both wavefields fill the grid
GRAD_TOL = 1e-4


def _gradient(w, layer, res, param, copies):
    from paper_2301_05127_amd import loss
    shots = w["shots"] * copies
    sim = loss.Simulation(w["grid"], w["physics"], w["dt"], nshots=len(shots), trace_len=w["nsteps"])
    sim.setup_workload(dict(w, shots=shots))
    sim.set_pml(layer["width"], layer["R"], layer["kmax"], layer["f0"])
    sim.forward_ckpt(w["nsteps"], 5)
    g = sim.adjoint(np.concatenate([r.ravel() for r in res * copies]), param)
    sim.close()
    return g / copies


def test_acoustic_layer_gradient_across_junctions(orc):
    require_gpu()
    from paper_2301_05127_amd import inputs, loss
    announce("acoustic layer gradient, pieces across junctions")
    n, width, dt, nsteps = (190, 0, 177), 9, 1e-3, 14
    g = inputs.grid(2, n, (10.0, 10.0, 10.0), (24, 1, 8), 7, 0)
    shape = inputs.field_shape(g)
    vp = _f32(inputs.gaussian_random_field(shape, 10.0, 80.0, 5, 2000.0, 2400.0))
    rho = np.full(shape, 1000.0)
    rec = np.array([[ix, 0, iz] for iz in range(12, n[2] - 10, 4) for ix in range(12, n[0] - 10, 5)], np.int32)
    shots = [{"sources": [{"kind": 0, "pos": (x, 0.0, 900.0), "spread": 300.0,
                           "wavelet": _f32(inputs.ricker(40.0, 0.004, dt, nsteps + 1, 0.5))}],
              "receivers": rec, "rec_comp": 0} for x in (600.0, 1300.0)]
    w = dict(grid=g, physics=0, dt=dt, nsteps=nsteps, vp=vp, vs=None, rho=rho, shots=shots)
    layer = dict(width=width, R=1e-6, kmax=1.5, f0=30.0, cmax=float(vp.max()))
    rng = np.random.default_rng(3)
    res = [rng.standard_normal((len(rec), nsteps)) for _ in shots]
    ref = sum(orc.acoustic_adjoint_pml(g, layer, dt, nsteps, vp, rho, sh["sources"], rec, r) for sh, r in zip(shots, res))
    e = rel_l2(_gradient(w, layer, res, loss.GRAD_K, 7), ref)
    print("rel-L2 %.2e" % e)
    assert np.abs(ref).max() > 0 and e < GRAD_TOL, e


def test_elastic_layer_gradient_across_junctions(orc):
    require_gpu()
    from paper_2301_05127_amd import inputs, loss
    announce("elastic layer gradient, pieces across junctions")
    n, width, dt, nsteps = (48, 41, 30), 5, 0.8e-3, 14
    g = inputs.grid(3, n, (10.0, 10.0, 10.0), (8, 8, 8), 6, 0)
    shape = inputs.field_shape(g)
    vp = _f32(inputs.gaussian_random_field(shape, 10.0, 60.0, 17, 2800.0, 3300.0))
    vs, rho = _f32(vp / np.sqrt(3.0)), _f32(inputs.gaussian_random_field(shape, 10.0, 40.0, 62, 2000.0, 2400.0))
    rec = np.array([[ix, iy, iz] for iz in range(7, 24, 4) for iy in range(7, 35, 5) for ix in range(7, 42, 5)], np.int32)

    def src(kind, shift):
        return {"kind": kind, "pos": tuple(5.0 * v for v in n), "spread": 60.0,
                "wavelet": _f32(inputs.ricker(50.0, 0.004, dt, nsteps + 1, shift))}

    shots = [{"sources": [src(1, 0.5)], "receivers": rec, "rec_comp": 2},
             {"sources": [src(3, 0.0)], "receivers": rec, "rec_comp": 6}]
    w = dict(grid=g, physics=1, dt=dt, nsteps=nsteps, vp=vp, vs=vs, rho=rho, shots=shots)
    layer = dict(width=width, R=1e-4, kmax=1.0, f0=50.0, cmax=float(vp.max()))
    rng = np.random.default_rng(4)
    res = [rng.standard_normal((len(rec), nsteps)) for _ in shots]
    ref = sum(np.array(orc.elastic_adjoint_pml(g, layer, dt, nsteps, vp, vs, rho, sh["sources"], rec, sh["rec_comp"], r,
                                               with_b=True)) for sh, r in zip(shots, res))
    ref[2] = -ref[2] / rho ** 2               # dJ/drho with lambda, mu fixed = -dJ/db / rho^2
    got = _gradient(w, layer, res, loss.GRAD_LAME_RHO, 2)
    e = [rel_l2(got[k], ref[k]) for k in range(3)]
    print("rel-L2 lambda %.2e mu %.2e rho %.2e" % tuple(e))
    assert all(np.abs(r).max() > 0 for r in ref) and max(e) < GRAD_TOL, e
