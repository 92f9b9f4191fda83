"""Off-grid values at the edges of the interpolation kernel's grouping: every
K, point counts around a wave, nodes, leaf edges and corners of the root,
against the Chebyshev expansion of the leaf evaluated in numpy.  Tolerance:
both are stable evaluations of one degree K-1 interpolant of values of size
one, so they differ by a few K^2 roundings: 1e-12."""
import numpy as np
import pytest

from paper_2211_14537_amd import vfx
from paper_2211_14537_amd.tree import _coef_matrix, cheb_nodes

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("K", [4, 8, 12, 16])
@pytest.mark.parametrize("npts", [1, 3, 63, 64, 65, 1000])
def test_points_of_a_small_tree(gpu_device, K, npts):
    import torch
    print(f"case K={K} npts={npts}", flush=True)
    leaves = [(2, x, y) for x in range(4) for y in range(4) if not (x < 2 and y < 2)] + [(1, 0, 0)]
    lev, ix, iy = (np.array(a) for a in zip(*leaves))
    ctx = vfx.Context(K, 20)
    plan = vfx.Plan(ctx, lev, ix, iy, np.ones(lev.size))
    rng = np.random.default_rng(100 * K + npts)
    V = rng.standard_normal((lev.size, K, K))
    x, y = rng.uniform(-1, 1, (2, npts))
    h = 2.0 / 2.0 ** lev
    cx, cy = -1 + (ix + 0.5) * h, -1 + (iy + 0.5) * h
    t = cheb_nodes(K)
    special = [(cx[0] + 0.5 * h[0] * t[1], cy[0] + 0.5 * h[0] * t[K - 1]), (0.0, 0.0), (-1.0, -1.0), (1.0, 1.0),
               (0.5, cy[3] + 0.5 * h[3] * t[0])]
    for i, (a, b) in enumerate(special[:npts // 2]):
        x[2 * i], y[2 * i] = a, b
    C = _coef_matrix(K)
    want = np.empty(npts)
    for i in range(npts):
        # the upper / right leaf of a shared edge; the last one on the root's
        q = [min(max(int(np.floor((v + 1) * 2)), 0), 3) for v in (x[i], y[i])]
        j = leaves.index((1, 0, 0) if max(q) < 2 else (2, q[0], q[1]))
        T = [np.cos(np.arange(K) * np.arccos(np.clip(2 * (v - c) / h[j], -1, 1))) for v, c in ((x[i], cx[j]), (y[i], cy[j]))]
        want[i] = T[0] @ C @ V[j] @ C.T @ T[1]
    out = torch.empty(npts, dtype=torch.float64, device=gpu_device)
    to = lambda a: torch.tensor(np.ascontiguousarray(a), device=gpu_device)  # noqa: E731
    plan.interp(to(V.reshape(lev.size, -1)), to(x), to(y), out)
    torch.cuda.synchronize()
    err = np.abs(out.cpu().numpy() - want).max()
    print(f"    max error {err:.2e}", flush=True)
    assert err <= 1e-12 * np.abs(V).max()
