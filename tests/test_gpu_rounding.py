"""Rounding of loss_deriv's slopes and transposed slopes (tile_axis.hip, the solves of the tile
passes): no further from FP64 than the patch systems (paper Sec. 3.1-3.2) eliminated row by row
in FP32 with fused multiply-adds, the form of a pass along one axis, on the same fields."""
import numpy as np
import pytest

from gpu_util import announce, rel_l2, require_gpu

pytestmark = pytest.mark.gpu

F = np.float32


def _fma(a, b, c):
    """a b + c rounded once (the FP64 sum of an exact product is exact to far below FP32)."""
    return (np.float64(a) * np.float64(b) + np.float64(c)).astype(F)


def _patches(n, m):
    return [(s, min(s + m, n)) for s in range(0, n, m)]


def _slopes(D, n, m, h, u):
    """Slopes of the lines u[node, column]: [1 4 1] rows, junction rows from their taps, natural
    end rows (2 1); the factors in FP64, rounded once."""
    s3, w = F(3.0 / h), np.zeros_like(u)
    for s, e in _patches(n, m):
        k = e - s + 1
        sub, d, sup = np.ones(k), np.full(k, 4.0), np.ones(k)
        r = np.empty((k, u.shape[1]), F)
        r[1:-1] = s3 * (u[s + 2:e + 1] - u[s:e - 1])
        for i, j in ((0, s), (k - 1, e)):
            if j in (0, n):
                d[i] = 2.0
                a, b = (0, 1) if j == 0 else (n - 1, n)
                r[i] = s3 * (u[b] - u[a])
            else:
                d[i], sub[i], sup[i] = 1.0, 0.0, 0.0
                r[i] = 0
                for t in np.flatnonzero(D[j]):
                    r[i] = _fma(F(D[j, t]), u[t], r[i])
        for i in range(1, k):
            f = sub[i] / d[i - 1]
            d[i] -= f * sup[i - 1]
            r[i] = _fma(F(-f), r[i - 1], r[i])
        r[k - 1] = r[k - 1] * F(1.0 / d[k - 1])
        for i in range(k - 2, -1, -1):
            r[i] = _fma(F(-sup[i]), r[i + 1], r[i]) * F(1.0 / d[i])
        w[s:e + 1] = r
    return w


def _transposed(D, n, m, h, z):
    """G^T T^-T of the same systems: interior rows closed per patch, the junctions' from their
    neighbours, then the columns of G."""
    s3, y, out = F(3.0 / h), np.zeros_like(z), np.zeros_like(z)
    for s, e in _patches(n, m):
        lo, hi = s if s == 0 else s + 1, e if e == n else e - 1
        d = np.full(hi - lo + 1, 4.0)
        if s == 0:
            d[0] = 2.0
        if e == n:
            d[-1] = 2.0
        r = z[lo:hi + 1].copy()
        for i in range(1, len(d)):
            f = 1.0 / d[i - 1]
            d[i] -= f
            r[i] = _fma(F(-f), r[i - 1], r[i])
        r[-1] = r[-1] * F(1.0 / d[-1])
        for i in range(len(d) - 2, -1, -1):
            r[i] = (r[i] - r[i + 1]) * F(1.0 / d[i])
        y[lo:hi + 1] = r
    junctions = [s for s, _ in _patches(n, m)[1:]]
    for j in junctions:
        y[j] = (z[j] - y[j - 1]) - y[j + 1]
    g = y.copy()
    g[junctions] = 0
    out[1:-1] = _fma(s3, g[:-2], -(s3 * g[2:]))
    out[0] = -_fma(s3, g[0], s3 * g[1])
    out[-1] = _fma(s3, g[-1], s3 * g[-2])
    for j in junctions:
        for t in np.flatnonzero(D[j]):
            out[t] = _fma(F(D[j, t]), y[j], out[t])
    return out


# intervals, patch, halo: whole patches, remainders, patches longer than a piece (cut in it)
LINES = [(256, 64, 10), (203, 40, 8), (300, 32, 9), (512, 128, 12)]


@pytest.mark.parametrize("axis", [0, 2])
@pytest.mark.parametrize("line", LINES, ids=["N%d_M%d_h%d" % v for v in LINES])
def test_rounding_no_larger_than_row_by_row(orc, line, axis):
    require_gpu()
    import torch
    from paper_2301_05127_amd import inputs, loss
    n, m, halo = line
    h, other = 10.0, 191
    announce("rounding %s axis %d" % (line, axis))
    ivl = (n, 0, other) if axis == 0 else (other, 0, n)
    g = inputs.grid(2, ivl, (h,) * 3, (m if axis == 0 else other, 1, m if axis == 2 else other), halo, 0)
    sim = loss.Simulation(g, loss.ACOUSTIC, 1e-4, nshots=1)
    D = orc.line_deriv_matrix(n, h, m, halo, 0)
    for name in ("white", "smooth"):
        if name == "white":
            u = inputs.random_field(sim.shape, seed=n + m).astype(F)
        else:
            u = inputs.gaussian_random_field(sim.shape, h, 60.0, n + m, -1.0, 1.0).astype(F)
        du = torch.from_numpy(u[None]).cuda()
        torch.cuda.synchronize()
        lines = u if axis == 2 else np.ascontiguousarray(u.T)
        for order in (1, -1):
            got = sim.deriv(axis, order, du).cpu().numpy()[0]
            got = got if axis == 2 else got.T
            ref = (D if order == 1 else D.T) @ lines.astype(np.float64)
            plain = rel_l2((_slopes if order == 1 else _transposed)(D, n, m, h, lines), ref)
            err = rel_l2(got, ref)
            print("%s order %d: %.3e, row by row %.3e" % (name, order, err, plain))
            assert err <= plain, (name, order)
    sim.close()
