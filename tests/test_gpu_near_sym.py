"""FP64 near field from exterior moments on the GPU, at the edges of its
tiles: trees of one leaf to a few hundred, every K, and batch sizes that take
each size of work item.  V against the oracle's direct quadrature: 1e-12 on
trees whose V is all near field (the gate of the degenerate FP64 trees in
test_gpu_mixed.py), 1e-10 otherwise (the method's FP64 gate).  A right-hand
side of a batch has the same products in the same order whatever the item
size, so it is compared bitwise."""
import numpy as np
import pytest

import gpu_cases as G
from oracle import geometry, volume
from paper_2211_14537_amd import vfx

pytestmark = pytest.mark.gpu


def uniform(depth):
    n = 1 << depth
    ix, iy = (a.ravel() for a in np.meshgrid(np.arange(n), np.arange(n), indexing="ij"))
    return np.full(ix.size, depth), ix, iy


@pytest.mark.parametrize("K,depth", [(4, 0), (4, 2), (8, 0), (8, 1), (12, 1), (12, 2), (16, 0), (16, 2)])
def test_small_uniform_trees(gpu_device, K, depth):
    import torch
    level, ix, iy = uniform(depth)
    p = 40 if depth > 1 else 20
    G.say(f"case K={K} depth={depth} p={p}")
    ctx = vfx.Context(K, p)
    plan = vfx.Plan(ctx, level, ix, iy, np.ones(level.size))
    f = np.random.default_rng(K + depth).standard_normal((level.size, K * K))
    fl = torch.tensor(f, device=gpu_device)
    fe, V = torch.empty_like(fl), torch.full_like(fl, float("nan"))
    plan.execute(fl, torch.empty((0, ctx.n_stencil), dtype=torch.float64, device=gpu_device), fe, V)
    torch.cuda.synchronize()
    ot = geometry.Tree(level, ix, iy, (0.0, 0.0, 2.0))
    X, Y = ot.leaf_nodes(K)
    sel = np.random.default_rng(1).choice(X.size, min(64, X.size), replace=False)
    v = volume.potential(ot, f, K, X.ravel()[sel], Y.ravel()[sel])
    err = float(np.abs(V.cpu().numpy().ravel()[sel] - v).max() / np.abs(v).max())
    G.say(f"    V rel Linf {err:.2e}")
    assert err <= (1e-12 if depth < 2 else 1e-10)


@pytest.mark.parametrize("name", ["starfish_small", "disk_adaptive_small"])
def test_item_sizes_bitwise(gpu_device, name):
    import torch
    case = G.setup(name, all_regular=True)
    plan, n = case["plan"], case["K"] ** 2
    L = case["f_leaf"].shape[0]
    rng = np.random.default_rng(3)
    f = rng.standard_normal((7, L, n))
    F = torch.tensor(f, device=gpu_device)
    empty = torch.empty((0, case["ctx"].n_stencil), dtype=torch.float64, device=gpu_device)
    one = []
    for r in range(7):
        fe, V = torch.empty_like(F[r]), torch.empty_like(F[r])
        plan.execute(F[r].contiguous(), empty, fe, V)
        one.append(V)
    for nrhs in (2, 7):
        G.say(f"case {name} nrhs={nrhs}")
        fe, V = torch.empty_like(F[:nrhs]), torch.empty_like(F[:nrhs])
        plan.execute_batch(nrhs, F[:nrhs].contiguous(), empty, fe, V)
        torch.cuda.synchronize()
        for r in range(nrhs):
            assert torch.equal(V[r], one[r])
    sel, x, y = G.sample_targets(case, 64, leaves=(0, L - 1))
    v = volume.potential(case["otree"], f[6], case["K"], x, y)
    err = float(np.abs(one[6].cpu().numpy().ravel()[sel] - v).max() / np.abs(v).max())
    G.say(f"    V rel Linf {err:.2e}")
    assert err <= 1e-10
