"""loss_deriv on device arrays (one launch from and to the caller's dense fields,
tile_axis.hip) against the FP64 oracle: lines that end on a tile edge, one node past it and
in a last patch of one interval, columns that do not fill a wave, batches larger than the
simulation's, the transposed operator on grids it is and is not tiled on, and calls in
place, which stage the fields instead.  Paper Sec. 3.1-3.2."""
import ctypes

import numpy as np
import pytest

from gpu_util import announce, rel_l2, require_gpu

pytestmark = pytest.mark.gpu

CASES = [
    # ndim, intervals, patches, halo, end mode, batch
    (2, (64, 0, 63), (64, 64, 63), 8, 0, 3),
    (2, (65, 0, 129), (64, 64, 128), 12, 0, 2),
    (2, (300, 0, 20), (150, 64, 5), 4, 0, 5),
    (2, (96, 0, 96), (8, 8, 8), 20, 0, 1),       # transposed taps reach past the next patch: staged
    (2, (130, 0, 64), (65, 64, 32), 12, 1, 2),
    (2, (96, 0, 72), (48, 48, 24), 10, 2, 2),    # periodic: the transposed operator is staged
    (2, (131, 0, 97), (16, 64, 8), 6, 0, 3),     # pieces across junctions
    (3, (33, 70, 66), (32, 35, 66), 6, 0, 2),
    (3, (66, 9, 17), (22, 9, 16), 8, 0, 4),
]


@pytest.mark.parametrize("case", CASES, ids=["x".join(map(str, c[1])) + "h%de%d" % (c[3], c[4]) for c in CASES])
def test_device_deriv_matches_oracle(orc, case):
    require_gpu()
    import torch
    from paper_2301_05127_amd import inputs, loss
    ndim, n, M, halo, mode, batch = case
    hs = (10.0, 7.0, 5.0)
    g = inputs.grid(ndim, n, hs, M, halo, mode)
    announce("device deriv %s" % (case,))
    sim = loss.Simulation(g, loss.ACOUSTIC if ndim == 2 else loss.ELASTIC, 1e-4, nshots=1)
    u = inputs.random_field((batch,) + sim.shape, seed=sum(n)).astype(np.float32)
    du = torch.from_numpy(u).cuda()
    torch.cuda.synchronize()
    for axis in ([0, 2] if ndim == 2 else [0, 1, 2]):
        D = orc.line_deriv_matrix(n[axis], hs[axis], M[axis], halo, mode)
        dim = (1 - axis // 2 if ndim == 2 else 2 - axis) + 1
        for order in (1, 2, -1):
            got = sim.deriv(axis, order, du).cpu().numpy()
            if order == -1:
                ref = np.moveaxis(np.tensordot(np.moveaxis(u.astype(np.float64), dim, -1), D, axes=([-1], [0])), -1, dim)
            else:
                ref = np.stack([orc.field_deriv(g, axis, order, u[b].astype(np.float64)) for b in range(batch)])
            # FP32 solve of a diagonally dominant system, condition <= 3
            tol = 5e-6 if order == 2 else 2e-6
            assert rel_l2(got, ref) < tol, (axis, order)
            inplace = du.clone()
            torch.cuda.synchronize()
            p = ctypes.c_void_p(inplace.data_ptr())
            assert loss.lib().loss_deriv(sim._h, axis, order, p, p, batch, loss.MEM_DEVICE) == 0
            sim.sync()
            assert rel_l2(inplace.cpu().numpy(), ref) < tol, (axis, order, "in place")
    sim.close()
