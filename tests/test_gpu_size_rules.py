"""Kernels chosen by size, at the edges of each choice: groups of right-hand
sides in the batched extension (the order of every sum is independent of the
group, so a right-hand side has the bits of a batch of 8), column heights of
the GPU factorisation with the compile-time and the general form of the
extension (against the oracle's float64 extension within twice its
conditioning-aware bound, as in test_gpu_parity.py), and the work-group sizes
of the extension with the split M2L (fewer than 8 right-hand sides reproduce
single executes bitwise, as in test_gpu_batch.py)."""
import numpy as np
import pytest

import gpu_cases as G
from oracle import extension, geometry
from paper_2211_14537_amd import tree as T
from paper_2211_14537_amd import vfx
from workloads import get_config

pytestmark = pytest.mark.gpu


def inputs(case, nrhs, seed):
    rng = np.random.default_rng(seed)
    a = rng.uniform(0.5, 2.0, nrhs)[:, None, None]
    return (a * case["f_leaf"] + 0.1 * rng.standard_normal((nrhs,) + case["f_leaf"].shape),
            a * case["f_cut"] + 0.1 * rng.standard_normal((nrhs,) + case["f_cut"].shape))


def worst_over_bound(case, f_leaf, f_cut, fe, Kbar=12):
    tr = case["tree"]
    ref, info = extension.extend(case["otree"], tr["kind"], f_leaf, f_cut, tr["mask"].astype(bool), case["K"],
                                 Kbar=Kbar, precision="fp64")
    worst = 0.0
    for i, rec in info.items():
        row = list(tr["cut_ids"]).index(i)
        tol = 2.0 * extension.extension_tolerance(rec, ref[rec["targets"]], f_cut[row][tr["mask"][row] != 0])
        worst = max(worst, float(np.abs(fe[rec["targets"]] - ref[rec["targets"]]).max()) / tol)
    return worst


def batch(case, fl, fc, device):
    import torch
    FL, FC = torch.tensor(fl, device=device), torch.tensor(fc, device=device)
    FE, V = torch.full_like(FL, float("nan")), torch.full_like(FL, float("nan"))
    case["plan"].execute_batch(len(fl), FL, FC, FE, V)
    torch.cuda.synchronize()
    return FE, V


@pytest.mark.parametrize("nrhs", [9, 16, 17, 32, 33, 65])
def test_groups_of_right_hand_sides(gpu_device, nrhs):
    import torch
    G.say(f"case disk_adaptive_small nrhs={nrhs}")
    case = G.setup("disk_adaptive_small", p=20)
    fl, fc = inputs(case, nrhs, nrhs)
    FE, _ = batch(case, fl, fc, gpu_device)
    for r0 in (0, nrhs - 8):
        fe, _ = batch(case, fl[r0:r0 + 8], fc[r0:r0 + 8], gpu_device)
        assert torch.equal(FE[r0:r0 + 8], fe)


@pytest.mark.parametrize("K,Kbar", [(12, 12), (16, 16)])
def test_column_heights(gpu_device, K, Kbar):
    import torch
    G.say(f"case starfish_small K={K} Kbar={Kbar}")
    cfg = get_config("starfish_small")
    cfg["K"] = K
    ctx = vfx.Context(K, 20, Kbar=Kbar, root=cfg["root"])
    tr = T.build_tree(cfg, ctx.stencil_points())
    if Kbar == 16:  # one leaf with every stencil point inside: the tallest columns
        tr["mask"][0] = 1
    fl, fc = T.sample_inputs(cfg, tr, ctx.stencil_points())
    most = int(tr["mask"].sum(axis=1).max())
    assert 288 < most <= 480 if K == 12 else most > 480
    case = dict(K=K, tree=tr, f_leaf=fl, f_cut=fc, otree=geometry.Tree(tr["level"], tr["ix"], tr["iy"], cfg["root"]))
    plan = vfx.Plan(ctx, tr["level"], tr["ix"], tr["iy"], tr["kind"], tr["mask"], defer_factor=True)
    plan.factor_gpu()
    d = torch.tensor(fl, device=gpu_device)
    fe, V = torch.full_like(d, float("nan")), torch.empty_like(d)
    plan.execute(d, torch.tensor(fc, device=gpu_device), fe, V)
    torch.cuda.synchronize()
    w = worst_over_bound(case, fl, fc, fe.cpu().numpy(), Kbar)
    G.say(f"    {most} interior points at most: worst error/bound {w:.3f}")
    assert w <= 1.0


@pytest.mark.parametrize("name,p,nrhs", [("starfish_small", 24, 2), ("starfish_small", 24, 5),
                                         ("starfish_small", 20, 6), ("starfish_small", 24, 7),
                                         ("disk_adaptive_small", 30, 3), ("disk_adaptive_small", 40, 3)])
def test_work_group_sizes_bitwise(gpu_device, name, p, nrhs):
    import torch
    G.say(f"case {name} p={p} nrhs={nrhs}")
    case = G.setup(name, p=p)
    fl, fc = inputs(case, nrhs, 5)
    FE, V = batch(case, fl, fc, gpu_device)
    for r in (0, nrhs - 1):
        d = torch.tensor(fl[r], device=gpu_device)
        fe, v = torch.empty_like(d), torch.empty_like(d)
        case["plan"].execute(d, torch.tensor(fc[r], device=gpu_device), fe, v)
        torch.cuda.synchronize()
        assert torch.equal(FE[r], fe) and torch.equal(V[r], v)


@pytest.mark.parametrize("nrhs", [2, 3])
def test_extension_work_groups_bitwise(gpu_device, nrhs):
    """182 cut leaves: 1024 threads for one right-hand side, 512 for two, 256
    for three."""
    import torch
    cfg = get_config("starfish_small")
    cfg["K"] = 4
    ctx = vfx.Context(4, 20, root=cfg["root"])
    tr = T.build_tree(cfg, ctx.stencil_points())
    assert len(tr["cut_ids"]) <= 256 < 2 * len(tr["cut_ids"]) <= 512 < 3 * len(tr["cut_ids"])
    fl, fc = T.sample_inputs(cfg, tr, ctx.stencil_points())
    plan = vfx.Plan(ctx, tr["level"], tr["ix"], tr["iy"], tr["kind"], tr["mask"])
    case = dict(f_leaf=fl, f_cut=fc, plan=plan)
    G.say(f"case starfish_small K=4 nrhs={nrhs}")
    fl, fc = inputs(case, nrhs, 6)
    FE, V = batch(case, fl, fc, gpu_device)
    for r in range(nrhs):
        d = torch.tensor(fl[r], device=gpu_device)
        fe, v = torch.empty_like(d), torch.empty_like(d)
        plan.execute(d, torch.tensor(fc[r], device=gpu_device), fe, v)
        torch.cuda.synchronize()
        assert torch.equal(FE[r], fe) and torch.equal(V[r], v)
