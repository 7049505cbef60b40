"""The tile passes (x and row derivatives of a sub-flow in one kernel, tile.hip) against
the FP64 oracle at the sizes where they can go wrong: patches longer than a tile (cut
inside, Sec. 3.2), last patches of one interval and of exactly a tile, rows that do not
fill a wave, halos wider than the patches, the other end rows, sources and receivers on
tile edges, the absorbing layer (Sec. 3.3), and the line passes on the same grid."""
import numpy as np
import pytest

from gpu_util import announce, rel_l2, require_gpu
from test_gpu_acoustic import _f32, _oracle

pytestmark = pytest.mark.gpu

# FP32 steps against FP64: the parity bound of the step tests (rounding of some tens of
# steps, each a few times 1e-7 of the field)
TOL = 1e-5

ACOUSTIC = [
    # intervals, patches, halo, end mode, layer
    ((128, 0, 128), (64, 64, 64), 8, 0, 0),      # last tile column cut so that node N has a lane
    ((130, 0, 257), (128, 64, 256), 12, 0, 0),   # cut patches; remainders of 2 and 1 intervals
    ((63, 0, 65), (63, 63, 64), 5, 0, 0),        # one tile column; a last row piece of one interval
    ((100, 0, 77), (100, 64, 77), 6, 0, 0),      # one patch per axis, cut
    ((96, 0, 96), (8, 8, 8), 20, 0, 0),          # halo 2.5 patches wide, the widest the window takes
    ((96, 0, 90), (70, 64, 24), 8, 1, 0),        # the paper's end stencil
    ((150, 0, 128), (75, 64, 64), 9, 2, 0),      # periodic
    ((150, 0, 131), (96, 64, 40), 8, 0, 12),     # layer over tile edges
]
# short patches and enough tiles: pieces across junctions
ACROSS = [
    # intervals, patches, halo, end mode, layer, copies of the shots
    ((205, 0, 200), (8, 8, 8), 12, 0, 0, 3),     # three junctions inside; taps wider than a patch
    ((193, 0, 210), (16, 16, 24), 5, 2, 0, 12),  # periodic; two inside and one
    ((190, 0, 177), (24, 24, 8), 7, 1, 9, 7),    # the end stencil; a last patch of one interval; layer
]


def _src(kind, pos, f0, dt, nsteps):
    from paper_2301_05127_amd import inputs
    return {"kind": kind, "pos": pos, "spread": 15.0,
            "wavelet": inputs.ricker(f0, 0.03, dt, nsteps + 1, 0.5 if kind < 2 else 0.0)}


def _check(orc, w, layer, schedules=(0, 1), copies=1):
    from paper_2301_05127_amd import loss
    w["shots"] = w["shots"] * copies
    S = len(w["shots"])
    ac = w["physics"] == 0
    refs = []
    for s in range(S):
        first = next(k for k in range(S) if w["shots"][k] is w["shots"][s])
        if first < s:                    # the same shot again
            refs.append(refs[first])
        elif layer:
            sh = w["shots"][s]
            lay = dict(width=layer, R=1e-6, kmax=1.5, f0=30.0, cmax=float(np.max(w["vp"])))
            kw = dict(sources=sh["sources"], receivers=sh["receivers"])
            if ac:
                refs.append(orc.run_pml(w["grid"], lay, w["dt"], w["nsteps"], w["vp"], w["rho"], **kw))
            else:
                refs.append(orc.run_pml_elastic(w["grid"], lay, w["dt"], w["nsteps"], w["vp"], w["vs"], w["rho"],
                                                rec_comp=sh["rec_comp"], **kw))
        else:
            refs.append(_oracle(orc, w, s))
    for sched in schedules:
        sim = loss.Simulation(w["grid"], w["physics"], w["dt"], nshots=S, trace_len=w["nsteps"])
        sim.setup_workload(w)
        if layer:
            sim.set_pml(layer, 1e-6, 1.5, 30.0)
        sim.set_shape([None, None, None, sched])
        sim.step(w["nsteps"] - 5)
        sim.step(5)
        for s in range(S):
            rf, rt = refs[s]
            errs = [rel_l2(sim.get_field(f, shot=s), rf[f]) for f in range(3 if ac else 9)]
            errs.append(rel_l2(sim.get_traces(s), rt))
            assert max(errs) < TOL, (sched, s, errs)
        sim.close()


def _ids(geoms):
    return ["x".join(map(str, g[0])) + "h%de%dl%d" % g[2:5] for g in geoms]


@pytest.mark.parametrize("geom", ACOUSTIC + ACROSS, ids=_ids(ACOUSTIC + ACROSS))
def test_acoustic_tiles_match_oracle(orc, geom):
    require_gpu()
    from paper_2301_05127_amd import inputs
    n, M, halo, end, layer = geom[:5]
    announce("acoustic tiles %s" % (geom,))
    g = inputs.grid(2, n, (10.0, 10.0, 10.0), M, halo, end)
    shape = inputs.field_shape(g)
    dt, nsteps = 1e-3, 40
    vp = 2500.0 * (1.0 + 0.1 * inputs.gaussian_random_field(shape, 10.0, 60.0, 9, -1.0, 1.0))
    # a pressure and a force source; receivers along a row and around a tile corner
    cx, cz = 10.0 * (n[0] // 2), 10.0 * (n[2] // 2)
    rec = [[i, 0, n[2] // 2 + 2] for i in range(2, n[0] - 1, 3)] + [[n[0] // 2, 0, k] for k in range(1, n[2], 4)]
    shots = [{"sources": [_src(0, (cx + 3.0, 0.0, cz - 2.0), 30.0, dt, nsteps),
                          _src(4, (cx - 40.0, 0.0, cz + 30.0), 25.0, dt, nsteps)],
              "receivers": np.array(rec, np.int32), "rec_comp": 0},
             {"sources": [_src(2, (cx, 0.0, cz), 30.0, dt, nsteps)], "receivers": np.array(rec, np.int32),
              "rec_comp": 0}]
    w = _f32(dict(grid=g, physics=0, dt=dt, nsteps=nsteps, vp=vp, vs=None, rho=np.full(shape, 1000.0), shots=shots))
    _check(orc, w, layer, copies=(geom + (1,))[5])


ELASTIC = [
    ((97, 70, 40), (96, 66, 40), 8, 0, 0),       # cut patches, last patch of one interval
    ((64, 64, 130), (64, 64, 128), 12, 0, 0),
    ((48, 41, 44), (20, 12, 9), 6, 0, 10),       # layer, rows that do not fill a wave
]
ELASTIC_ACROSS = [
    ((48, 41, 30), (8, 8, 8), 6, 0, 0, 2),
    ((50, 40, 35), (8, 20, 12), 6, 0, 8, 2),
]


@pytest.mark.parametrize("geom", ELASTIC + ELASTIC_ACROSS, ids=_ids(ELASTIC + ELASTIC_ACROSS))
def test_elastic_tiles_match_oracle(orc, geom):
    require_gpu()
    from paper_2301_05127_amd import inputs
    n, M, halo, end, layer = geom[:5]
    announce("elastic tiles %s" % (geom,))
    g = inputs.grid(3, n, (10.0, 10.0, 10.0), M, halo, end)
    shape = inputs.field_shape(g)
    dt, nsteps = 0.8e-3, 24
    vp = 3000.0 * (1.0 + 0.05 * inputs.gaussian_random_field(shape, 10.0, 60.0, 17, -1.0, 1.0))
    c = tuple(10.0 * (v // 2) + 3.0 for v in n)
    rec = np.array([[n[0] // 2 + 2, n[1] // 2 - 3, k] for k in range(n[2] // 4, 3 * n[2] // 4, 2)], np.int32)
    shots = [{"sources": [_src(1, c, 40.0, dt, nsteps)], "receivers": rec, "rec_comp": 2},
             {"sources": [_src(3, c, 40.0, dt, nsteps)], "receivers": rec, "rec_comp": 7}]
    w = _f32(dict(grid=g, physics=1, dt=dt, nsteps=nsteps, vp=vp, vs=vp / np.sqrt(3.0), rho=310.0 * vp ** 0.25,
                  shots=shots))
    _check(orc, w, layer, copies=(geom + (1,))[5])
