"""CPU emulation (FP32 operations of the kernel) of the culled scans' tile tests:
a tile that holds a point within a query's bound passes the query's box test,
and the coarser test of a group of queries passes every tile that some query of
the group passes."""
import numpy as np
import pytest

F = np.float32
EPS22, SHRINK = F(2.0 ** -22), F(1.0) - F(2.0 ** -19)


def gap2(lo, hi, ylo, yhi, axes):
    s = np.zeros(np.broadcast(lo[..., 0], ylo[..., 0]).shape, F)
    for a in axes:
        g = np.maximum(np.maximum(lo[..., a] - yhi[..., a], ylo[..., a] - hi[..., a]), F(0))
        s = (g.astype(np.float64) * g + s).astype(F)      # a fused multiply-add
    return s


@pytest.mark.parametrize("shift,scale", [(0.0, 1.0), (40.0, 1.0), (0.0, 1e3), (0.0, 1e-4)])
def test_group_test_passes_what_the_tile_test_passes(shift, scale):
    rng = np.random.default_rng(7)
    n, rows, m = 4096, 32, 64
    x = np.concatenate([rng.uniform(-0.6, 0.6, (n, 6)), rng.normal(0, 0.005, (n, 6))], 1)
    x = (x[np.argsort(x[:, 0])] + shift) * scale
    box = x.reshape(-1, rows, 12)
    lo = np.nextafter(box.min(1).astype(F), F(-np.inf))
    hi = np.nextafter(box.max(1).astype(F), F(np.inf))
    root_lo, root_hi = lo.min(0), hi.max(0)
    q = x[rng.integers(0, n, m)] + rng.normal(0, 0.02, (m, 12)) * scale
    d = np.sqrt(((q[:, None] - x[None]) ** 2).sum(2))
    reach = (np.linalg.norm(q, axis=1) + np.linalg.norm(x, axis=1).max()).astype(F)
    slack = EPS22 * reach + F(1e-30)
    y = q.astype(F)
    for factor in (1.0, 1.3, 4.0):
        U = np.nextafter((d.min(1) * factor).astype(F), F(np.inf))
        s12 = gap2(lo[None], hi[None], y[:, None], y[:, None], range(12))
        passes = np.sqrt(s12) * SHRINK - slack[:, None] <= U[:, None]
        holds = (d.reshape(m, -1, rows) <= U[:, None, None].astype(np.float64)).any(2)
        assert np.all(passes[holds])
        # a query's six-axis radius, and a group of 16 by its bounding box
        t = (U + slack) * F(1 + 2.0 ** -18)
        e2 = gap2(root_lo[None], root_hi[None], y, y, range(6, 12))
        r2 = t * t * F(1 + 2.0 ** -16) - e2 * F(1 - 2.0 ** -16) + F(1e-37)
        s6 = gap2(lo[None], hi[None], y[:, None], y[:, None], range(6))
        assert np.all((s6 <= r2[:, None])[passes])
        for g in range(0, m, 16):
            k = slice(g, g + 16)
            sg = gap2(lo, hi, y[k].min(0)[None], y[k].max(0)[None], range(6))
            assert np.all((sg <= r2[k].max())[passes[k].any(0)])
