"""Performance cases: the work a program built on vfx has the GPU do.

Every case goes through the public binding (``paper_2211_14537_amd.vfx``).  The geometry of a case (its
quad-tree, the plan's lists and operators) is fixed by the case; the seed draws the data: the amplitudes of the
Gaussian bumps the tree was refined for, the points, the samples and labels of the classifier.

Paths:
  execute   one extension + volume FMM of given data on a prepared plan
  batch     the same for several right-hand sides at once
  geometry  a new domain: plan, least-squares operators on the GPU, first execute
  graph     executes of several small plans captured in one HIP graph and replayed
  points    after a solve: V at off-grid points and the net charge of f^e
  train     one minibatch step of the refinement classifier (gradient + Adam)
  classify  FP16 decisions of the classifier for the boxes of one refinement sweep
"""
import math
from functools import lru_cache

import numpy as np
import torch

from paper_2211_14537_amd import tree as T
from paper_2211_14537_amd import vfx
from workloads.configs import _seeded_gaussians
from workloads.domains import EXTERIOR, REGULAR, Disk, SquareMinusWedge, Starfish

ROOT = (0.0, 0.0, 2.0)
KBAR, DEG, NG = 12, 10, 66
NPAR = 8385  # parameters of the classifier: W1 64x64, b1, W2 64x64, b2, w3, b3
# "box": data given on every leaf of a tree refined as for the disk
DOMAINS = {"box": lambda: Disk(0.6), "disk": lambda: Disk(0.6), "starfish": lambda: Starfish(0.5, 0.15, 5),
           "wedge": lambda: SquareMinusWedge(0.6, math.pi / 6)}
WIDTHS = {"box": (0.02, 0.1), "disk": (0.02, 0.1), "starfish": (0.01, 0.1), "wedge": (0.005, 0.1)}


def listed():
    return [
        # the smallest call: a uniform tree of 64 leaves, all latency
        dict(name="disk-uniform", path="execute", domain="disk", K=8, p=20, uniform=3, bumps=1),
        # K = 8 at the size of the paper's interior example (a few thousand leaves, hundreds of them cut)
        dict(name="disk-k8", path="execute", domain="disk", K=8, p=20, tol=1e-10, depth=8, cut=7, min_level=5, bumps=5),
        # an ordinary solve: a million nodes, the boundary resolved at level 8
        dict(name="starfish", path="execute", domain="starfish", K=16, p=24, tol=1e-13, depth=9, cut=8, bumps=1),
        # the largest single solve: 3.65 million nodes, a domain with corners
        dict(name="wedge", path="execute", domain="wedge", K=16, p=24, tol=1e-12, depth=10, cut=9, min_level=7,
             bumps=3),
        # the same with the near field on the int8 matrix cores
        dict(name="wedge-int8", path="execute", domain="wedge", K=16, p=24, tol=1e-12, depth=10, cut=9, min_level=7,
             bumps=3, near=2),
        # many right-hand sides on one tree (time steps, parameter studies)
        dict(name="starfish-batch", path="batch", domain="starfish", K=16, p=24, tol=1e-12, depth=8, cut=8, bumps=4,
             nrhs=32),
        # a few right-hand sides known in the whole box (no cut leaves), the grid size between the usual ones
        dict(name="box-k12-batch", path="batch", domain="box", K=12, p=30, tol=1e-9, depth=6, cut=5, bumps=2, nrhs=5),
        # a domain that moves: everything a new tree needs, then its first solve
        dict(name="new-geometry", path="geometry", domain="starfish", K=16, p=24, tol=1e-13, depth=9, cut=8, bumps=1),
        # many small trees, one launch
        dict(name="small-trees", path="graph", domain="starfish", K=16, p=24, bumps=7, trees=10),
        # V at the points of a plot and on the boundary, and the charge of the exterior problem
        dict(name="off-grid", path="points", domain="starfish", K=16, p=24, tol=1e-13, depth=9, cut=8, bumps=1,
             points=200000),
        # learned refinement: a training step at the trainer's batch, and one sweep's decisions
        dict(name="train-step", path="train", batch=1024),
        dict(name="classify", path="classify", batch=12000),
    ]


def draw(rng):
    kind = rng.choice(["execute"] * 5 + ["batch"] * 2 + ["geometry", "graph", "points", "points", "train", "classify"])
    logint = lambda a, b: int(round(math.exp(rng.uniform(math.log(a), math.log(b)))))  # noqa: E731
    if kind == "train":
        return dict(path="train", batch=logint(33, 16384))
    if kind == "classify":
        return dict(path="classify", batch=logint(5, 300000))
    domain = rng.choice(["box", "disk", "starfish", "wedge"])
    K = rng.choice([8, 8, 12, 16, 16, 16, 16])
    p = rng.choice([20, 20, 30, 17]) if K < 16 else rng.choice([24, 24, 24, 40, 30, 27])
    case = dict(path=kind, domain=domain, K=K, p=p, bumps=rng.randrange(1, 1000))
    if kind in ("geometry", "graph") and domain == "box":
        case["domain"] = "disk"
    if kind == "graph":
        return dict(case, K=16, trees=rng.randrange(2, 11))
    top = 8 if kind in ("execute", "points") else 7
    if rng.random() < 0.25:
        case.update(uniform=rng.randrange(2, 6 if K == 16 else 7))
    else:
        cut = rng.randrange(3, top + 1)
        case.update(tol=10.0 ** -rng.uniform(6, 12 if K == 16 else 9), depth=cut + rng.randrange(0, 2), cut=cut)
    if K == 16 and kind == "execute" and rng.random() < 0.3:
        case.update(near=rng.choice([1, 2]))
    if kind == "batch":
        case.update(nrhs=rng.randrange(2, 25))
    if kind == "points":
        case.update(points=logint(100, 400000))
    return case


# ---- geometry and data -----------------------------------------------------------------------------------


@lru_cache(maxsize=None)
def context(K, p):
    return vfx.Context(K, p, Kbar=KBAR, deg=DEG, root=ROOT)


@lru_cache(maxsize=None)
def geometry(domain, K, p, bumps, uniform, tol, depth, cut, min_level):
    """The tree of a case with its stencil masks, and the bumps it was refined for."""
    dom = DOMAINS[domain]()
    fun = _seeded_gaussians(dom, 4, *WIDTHS[domain], seed=bumps)
    spec = (dict(kind="uniform", depth=uniform) if uniform
            else dict(kind="adaptive", tol=tol, max_depth=depth, min_cut_level=cut, min_level=min_level))
    tree = T.build_tree(dict(root=ROOT, K=K, domain=dom, fun=fun, tree=spec), context(K, p).stencil_points())
    if domain == "box":
        tree.update(kind=np.full_like(tree["kind"], REGULAR), cut_ids=tree["cut_ids"][:0], mask=tree["mask"][:0])
    return tree, fun


def geometry_of(case):
    return geometry(case["domain"], case["K"], case["p"], case["bumps"], case.get("uniform", 0), case.get("tol", 0.0),
                    case.get("depth", 0), case.get("cut", 0), case.get("min_level", 0))


def small_trees(case):
    """The trees of a graph case: 160 to about 1500 leaves, each with its own bumps."""
    return [dict(case, path="execute", bumps=case["bumps"] + i, tol=10.0 ** -(6 + i % 4), depth=4 + i % 4,
                 cut=4 + i % 3) for i in range(case["trees"])]


def new_plan(case, defer=True):
    tree, _ = geometry_of(case)
    return vfx.Plan(context(case["K"], case["p"]), tree["level"], tree["ix"], tree["iy"], tree["kind"], tree["mask"],
                    defer_factor=defer)


def device():
    return torch.device("cuda:0" if torch.cuda.is_available() else "cpu")


def sample(case, seed):
    """f on the leaf grids and at the cut leaves' stencil points (zero outside the domain), nrhs x rows x points:
    the tree's bumps with amplitudes drawn from the seed."""
    tree, fun = geometry_of(case)
    K, nrhs, dev = case["K"], case.get("nrhs", 1), device()
    rng = np.random.default_rng([seed, case["bumps"]])
    size = (nrhs, fun.w.size)
    amp = torch.tensor(rng.uniform(0.5, 1.5, size) * rng.choice([-1.0, 1.0], size), device=dev)
    grid = lambda a: torch.tensor(np.ascontiguousarray(a), device=dev)  # noqa: E731
    cx, cy, h = grid(tree["cx"]), grid(tree["cy"]), grid(tree["h"])
    t = grid(T.cheb_nodes(K))
    n = cx.numel()
    X = (cx[:, None, None] + 0.5 * h[:, None, None] * t[None, :, None]).expand(n, K, K).reshape(n, K * K)
    Y = (cy[:, None, None] + 0.5 * h[:, None, None] * t[None, None, :]).expand(n, K, K).reshape(n, K * K)
    S = grid(context(K, case["p"]).stencil_points())
    cut = grid(tree["cut_ids"])
    CX = cx[cut][:, None] + 1.5 * h[cut][:, None] * S[None, :, 0]
    CY = cy[cut][:, None] + 1.5 * h[cut][:, None] * S[None, :, 1]

    def f(x, y):
        out = torch.zeros((nrhs,) + tuple(x.shape), dtype=torch.float64, device=dev)
        for k, ((bx, by), w) in enumerate(zip(fun.c, fun.w)):
            r2 = (x - bx) ** 2 + (y - by) ** 2
            g = (4.0 * r2 / (w * w) - 4.0 / w) * torch.exp(-r2 / w)
            for r in range(nrhs):
                out[r].add_(g * amp[r, k])
        return out

    return f(X, Y), torch.where(grid(tree["mask"]) != 0, f(CX, CY), 0.0)


def points_of(case, seed):
    """Off-grid points: half of them uniform in the root box, half on the circle r = 0.5."""
    rng = np.random.default_rng([seed, 7])
    m = case["points"]
    q = m // 2
    th = rng.uniform(0, 2 * math.pi, m - q)
    x = np.concatenate([rng.uniform(-1, 1, q), 0.5 * np.cos(th)])
    y = np.concatenate([rng.uniform(-1, 1, q), 0.5 * np.sin(th)])
    return torch.tensor(x, device=device()), torch.tensor(y, device=device())


def classifier(case, seed):
    """Parameters and moments of a classifier in mid-training, features in [-1, 1] and labels."""
    rng = np.random.default_rng([seed, 11])
    D = 64
    th = np.concatenate([rng.normal(0, math.sqrt(2 / D), D * D), rng.normal(0, 0.1, D),
                         rng.normal(0, math.sqrt(2 / D), D * D), rng.normal(0, 0.1, D),
                         rng.normal(0, math.sqrt(1 / D), D), rng.normal(0, 0.1, 1)])
    B = case["batch"]
    decay = np.linspace(0.2, -0.9, 16)[None, None, :]
    x = np.clip(decay + rng.normal(0, 0.35, (B, 4, 16)), -1, 1).reshape(B, D)
    y = (rng.random(B) < 0.5)
    m = rng.normal(0, 1e-3, NPAR)
    v = rng.uniform(0.5, 2.0, NPAR) * 1e-6
    return [torch.tensor(a.astype(np.float32), device=device()) for a in (th, x, y, m, v)]


# ---- one pass --------------------------------------------------------------------------------------------


def prepare(case, seed):
    path = case["path"]
    if path == "train":
        th, x, y, m, v = classifier(case, seed)
        work = torch.empty(vfx.mlp_grad_work(case["batch"]), dtype=torch.float32, device=device())
        return dict(path=path, theta=th, x=x, y=y, m=m, v=v, grad=torch.empty_like(th), work=work)
    if path == "classify":
        th, x, _, _, _ = classifier(case, seed)
        return dict(path=path, theta=th.half(), x=x.half(), logits=torch.empty(case["batch"], device=device()))
    if path == "graph":
        parts = [prepare(c, seed + i) for i, c in enumerate(small_trees(case))]
        for s in parts:
            run(s)
        torch.cuda.synchronize()
        stream, graph = torch.cuda.Stream(), vfx.Graph()
        graph.begin(stream)
        for s in parts:
            s["plan"].execute(s["f_leaf"], s["f_cut"], s["fe"], s["V"], stream=stream)
        graph.end(stream)
        return dict(path=path, parts=parts, graph=graph, stream=stream)
    f_leaf, f_cut = sample(case, seed)
    if path != "batch":
        f_leaf, f_cut = f_leaf[0].contiguous(), f_cut[0].contiguous()
    s = dict(path=path, case=dict(case), f_leaf=f_leaf, f_cut=f_cut, fe=torch.empty_like(f_leaf),
             V=torch.empty_like(f_leaf))
    if path == "geometry":
        geometry_of(case)
        return s
    s["plan"] = new_plan(case)
    s["plan"].factor_gpu()
    if case.get("near"):
        s["plan"].set_precision(case["near"])
        s["plan"].factor_gpu()
    if path == "batch":
        s["nrhs"] = case["nrhs"]
    if path == "points":
        s["px"], s["py"] = points_of(case, seed)
        s["out"] = torch.empty_like(s["px"])
        s["charge"] = torch.empty(1, dtype=torch.float64, device=device())
    return s


def run(s):
    path = s["path"]
    if path == "execute":
        s["plan"].execute(s["f_leaf"], s["f_cut"], s["fe"], s["V"])
        return {"fe": s["fe"], "V": s["V"]}
    if path == "batch":
        s["plan"].execute_batch(s["nrhs"], s["f_leaf"], s["f_cut"], s["fe"], s["V"])
        return {"fe": s["fe"], "V": s["V"]}
    if path == "geometry":
        plan = new_plan(s["case"])
        plan.factor_gpu()
        plan.execute(s["f_leaf"], s["f_cut"], s["fe"], s["V"])
        return {"fe": s["fe"], "V": s["V"]}
    if path == "graph":
        s["graph"].launch(torch.cuda.current_stream())
        return [{"fe": q["fe"], "V": q["V"]} for q in s["parts"]]
    if path == "points":  # leaf data in hand (here the samples of f) stand for V and f^e
        s["plan"].interp(s["f_leaf"], s["px"], s["py"], s["out"])
        s["plan"].net_charge(s["f_leaf"], s["charge"])
        return {"out": s["out"], "charge": s["charge"]}
    if path == "train":
        vfx.mlp_grad(s["theta"], s["x"], s["y"], s["grad"], s["work"])
        vfx.mlp_adam(s["theta"], s["grad"], s["m"], s["v"], 200, lr=3e-3)
        return {"grad": s["grad"], "theta": s["theta"], "m": s["m"], "v": s["v"]}
    vfx.mlp_infer_f16(s["theta"], s["x"], s["logits"])
    return s["logits"]


def work(case):
    path, D = case["path"], 64
    if path == "train":
        B = case["batch"]
        return {"bytes": 4.0 * (B * (D + 1) + 7 * NPAR), "flops": 3.0 * 2 * B * (2 * D * D + D)}
    if path == "classify":
        B = case["batch"]
        return {"bytes": 2.0 * (B * D + NPAR) + 4.0 * B, "flops": 2.0 * B * (2 * D * D + D)}
    if path == "graph":
        parts = [work(c) for c in small_trees(case)]
        return {k: sum(w[k] for w in parts) for k in ("bytes", "flops")}
    tree, _ = geometry_of(case)
    K, P, L, nrhs = case["K"], case["p"] + 1, tree["level"].size, case.get("nrhs", 1)
    n = K * K
    if path == "points":
        return {"bytes": 8.0 * (2 * L * n + 3 * case["points"]), "flops": 2.0 * (case["points"] * (n + K) + 2 * L * n)}
    st = new_plan(case).stats()
    interior = int(tree["mask"].sum())
    regular = int((tree["kind"] == REGULAR).sum())
    nbytes = 8.0 * (nrhs * (regular * n + interior + 2 * L * n) + NG * interior)
    ext = 2.0 * (NG * interior + st["n_cut"] * (NG * KBAR**2 + 2 * KBAR**3)
                 + st["n_ext_targets"] * (KBAR * KBAR * K // 2 + KBAR * n))
    near = 4.0 * n * min(n // 2, 3 * K) * st["n_list1"]
    far = 4.0 * P * (P * st["n_list2"] + n * (st["n_list3"] + st["n_list4"] + 2 * L))
    flops = nrhs * (ext + near + far)
    if path == "geometry":  # a QR and the explicit pseudo-inverse of every cut leaf
        flops += 4.0 * NG * NG * interior
    return {"bytes": nbytes, "flops": flops}


# ---- 64-bit values, from the definitions alone -----------------------------------------------------------


def cheb_values(x, n):
    """T_0 .. T_(n-1) at x, along a new last axis."""
    return torch.cos(torch.arange(n, dtype=torch.float64, device=x.device) * torch.arccos(x.clamp(-1, 1))[..., None])


def node_to_coef(K):
    a = np.arange(K)
    C = (2.0 / K) * np.cos(np.outer(a, np.arccos(-np.cos((2 * a + 1) * np.pi / (2 * K)))))
    C[0] *= 0.5
    return C


def exact_extension(case, f_leaf, f_cut):
    """f^e by the least-squares fit of every cut leaf (total degree 10 on the interior stencil points, minimum-norm
    in the values on the support nodes), on the leaves of its extension list."""
    tree, _ = geometry_of(case)
    K = case["K"]
    S = np.asarray(context(K, case["p"]).stencil_points())
    basis = [(m, k) for m in range(DEG + 1) for k in range(DEG + 1 - m)]
    Tx, Ty = (np.cos(np.arange(DEG + 1) * np.arccos(np.clip(S[:, d], -1, 1))[:, None]) for d in (0, 1))
    P = np.stack([Tx[:, m] * Ty[:, k] for m, k in basis], axis=1)
    A = np.linalg.solve(P[-NG:].T, P.T).T
    Cb, t = node_to_coef(KBAR), T.cheb_nodes(K)
    m, k = np.meshgrid(np.arange(KBAR), np.arange(KBAR), indexing="ij")
    low = (m + k) < KBAR
    kind, cx, cy, h, lev = (tree[q] for q in ("kind", "cx", "cy", "h", "level"))
    cuts = tree["cut_ids"]
    # owner of an exterior leaf: the closest cut centre among the extension squares that overlap it, the later one
    # on a tie (distances in whole units of the finest half side)
    unit = 2.0 / 2.0 ** int(lev.max()) / 2.0
    ix, iy = np.rint((cx + 1.0) / unit).astype(np.int64), np.rint((cy + 1.0) / unit).astype(np.int64)
    owner = np.full(lev.size, -1)
    ext = np.nonzero(kind == EXTERIOR)[0]
    best = np.full(lev.size, np.iinfo(np.int64).max)
    for i in cuts:
        dx, dy = np.abs(cx[ext] - cx[i]), np.abs(cy[ext] - cy[i])
        reach = 1.5 * h[i] + 0.5 * h[ext]
        j = ext[(dx < reach - 1e-12) & (dy < reach - 1e-12)]
        d2 = (ix[j] - ix[i]) ** 2 + (iy[j] - iy[i]) ** 2
        near = d2 <= best[j]
        best[j[near]], owner[j[near]] = d2[near], i
    fl, fc = f_leaf.cpu().numpy(), f_cut.cpu().numpy()
    fe = np.where((kind == REGULAR)[None, :, None], fl, 0.0)
    for r, i in enumerate(cuts):
        mask = tree["mask"][r] != 0
        fg = fc[:, r][:, mask] @ np.linalg.pinv(A[mask], rcond=1e-13).T
        bar = slice(K * K, K * K + KBAR * KBAR)
        g = np.where(mask[bar], fc[:, r, bar], fg @ A[bar].T).reshape(-1, KBAR, KBAR)
        c = np.einsum("ai,lij,bj->lab", Cb, g, Cb) * low
        for j in [i] + list(np.nonzero(owner == i)[0]):
            E = [np.cos(np.arange(KBAR) * np.arccos(np.clip(o + 0.5 * h[j] * t / (1.5 * h[i]), -1, 1))[:, None])
                 for o in ((cx[j] - cx[i]) / (1.5 * h[i]), (cy[j] - cy[i]) / (1.5 * h[i]))]
            fe[:, j] = np.einsum("am,lmk,bk->lab", E[0], c, E[1]).reshape(-1, K * K)
    return torch.tensor(fe, device=f_leaf.device)


def graded(x, levels=34, ratio=0.3, q=16):
    """Quadrature on [-1, 1] graded towards the point of it that is nearest to x: (nodes, weights) per entry of x."""
    g, w = np.polynomial.legendre.leggauss(q)
    edge = np.concatenate([ratio ** np.arange(levels), [0.0]])
    lo, hi = edge[1:], edge[:-1]
    u = torch.tensor((0.5 * (lo + hi)[:, None] + 0.5 * (hi - lo)[:, None] * g).ravel(), device=x.device)
    v = torch.tensor((0.5 * (hi - lo)[:, None] * w).ravel(), device=x.device)
    c = x.clamp(-1, 1)[:, None]
    return torch.cat([c + (1 - c) * u, c - (1 + c) * u], 1), torch.cat([(1 - c) * v, (1 + c) * v], 1)


def exact_potential(case, fe):
    """V at every leaf node by direct quadrature: pairs of leaves that touch by rules graded towards the target (one
    table per relative position), the others by a 24 x 24 Gauss rule on the source leaf."""
    tree, _ = geometry_of(case)
    K, dev = case["K"], fe.device
    n, L = K * K, fe.shape[1]
    C = torch.tensor(node_to_coef(K), device=dev)
    coef = torch.einsum("ai,rlij,bj->rlab", C, fe.reshape(-1, L, K, K), C).reshape(-1, L, n)
    t = torch.tensor(T.cheb_nodes(K), device=dev)
    cx, cy, h = (torch.tensor(tree[q], device=dev) for q in ("cx", "cy", "h"))
    V = torch.zeros_like(fe)
    # touching pairs by relative position (in target sides) and size
    gap = 0.5 * (h[:, None] + h[None, :]) * (1 + 1e-9)
    near = ((cx[:, None] - cx[None, :]).abs() <= gap) & ((cy[:, None] - cy[None, :]).abs() <= gap)
    tg, sr = near.nonzero(as_tuple=True)
    key = torch.stack([(cx[sr] - cx[tg]) / h[tg], (cy[sr] - cy[tg]) / h[tg], h[sr] / h[tg]], 1)
    kinds, which = torch.unique((key * 16).round().long(), dim=0, return_inverse=True)
    for c in range(kinds.shape[0]):
        ox, oy, sz = (kinds[c].double() / 16).tolist()
        x, wx = graded((0.5 * t - ox) / (0.5 * sz))
        y, wy = graded((0.5 * t - oy) / (0.5 * sz))
        ex, ey = cheb_values(x, K) * wx[..., None], cheb_values(y, K) * wy[..., None]
        table = torch.empty((K, K, K, K), dtype=torch.float64, device=dev)
        for a in range(K):
            dx = (0.5 * sz * x[a] - (0.5 * t[a] - ox)) ** 2
            for b in range(K):
                dy = (0.5 * sz * y[b] - (0.5 * t[b] - oy)) ** 2
                table[a, b] = ex[a].T.contiguous() @ (0.5 * torch.log(dx[:, None] + dy[None, :] + 1e-300) @ ey[b])
        sel = which == c
        i, j = tg[sel], sr[sel]
        area = (0.5 * h[j]) ** 2
        mean = coef[:, j] @ torch.outer(C.new_tensor([0.0 if k % 2 else 2.0 / (1 - k * k) for k in range(K)]),
                                        C.new_tensor([0.0 if k % 2 else 2.0 / (1 - k * k) for k in range(K)])).ravel()
        V.index_add_(1, i, (coef[:, j] @ table.reshape(n, n).T.contiguous() + (mean * torch.log(h[i]))[..., None])
                     * area[None, :, None])
    # the others: every source leaf resampled on a Gauss grid
    g, w = (torch.tensor(q, device=dev) for q in np.polynomial.legendre.leggauss(24))
    E = cheb_values(g, K)
    val = torch.einsum("am,rlmk,bk->rlab", E, coef.reshape(-1, L, K, K), E) * torch.outer(w, w)
    val = val.reshape(-1, L, 576) * (0.25 * h * h)[:, None]
    gx = (cx[:, None] + 0.5 * h[:, None] * g.repeat_interleave(24)).contiguous()
    gy = (cy[:, None] + 0.5 * h[:, None] * g.repeat(24)).contiguous()
    for i in range(L):
        X = (cx[i] + 0.5 * h[i] * t).repeat_interleave(K)
        Y = (cy[i] + 0.5 * h[i] * t).repeat(K)
        far = (~near[i]).nonzero()[:, 0]
        for s in far.split(max(1, 60_000_000 // (n * 576))):
            lg = torch.log((X[:, None] - gx[s].ravel()) ** 2 + (Y[:, None] - gy[s].ravel()) ** 2)
            V[:, i] += 0.5 * (val[:, s].reshape(val.shape[0], -1) @ lg.T.contiguous())
    return V / (2 * math.pi)


def exact_points(case, seed):
    f_leaf, _ = sample(case, seed)
    tree, _ = geometry_of(case)
    K, dev = case["K"], f_leaf.device
    px, py = points_of(case, seed)
    cx, cy, h, lev = (torch.tensor(tree[q], device=dev) for q in ("cx", "cy", "h", "level"))
    top = int(lev.max())
    cells = torch.full((1 << top, 1 << top), -1, dtype=torch.long, device=dev)
    for i, (l, x, y) in enumerate(zip(tree["level"].tolist(), tree["ix"].tolist(), tree["iy"].tolist())):
        s = 1 << (top - l)
        cells[x * s:(x + 1) * s, y * s:(y + 1) * s] = i
    at = [((q + 1) * 0.5 * (1 << top)).floor().long().clamp(0, (1 << top) - 1) for q in (px, py)]
    leaf = cells[at[0], at[1]]
    C = torch.tensor(node_to_coef(K), device=dev)
    coef = torch.einsum("ai,lij,bj->lab", C, f_leaf[0].reshape(-1, K, K), C)
    out = torch.empty_like(px)
    for s in torch.arange(px.numel(), device=dev).split(1 << 18):
        i = leaf[s]
        a, b = cheb_values(2 * (px[s] - cx[i]) / h[i], K), cheb_values(2 * (py[s] - cy[i]) / h[i], K)
        out[s] = (a * (coef[i] * b[:, None, :]).sum(2)).sum(1)
    mean = C.new_tensor([0.0 if k % 2 else 1.0 / (1 - k * k) for k in range(K)])
    charge = ((coef * torch.outer(mean, mean)).sum((1, 2)) * h * h).sum()
    return {"out": out, "charge": charge[None]}


def exact_classifier(case, seed):
    th, x, y, m, v = classifier(case, seed)
    half = case["path"] == "classify"
    th, x = (q.half().double() if half else q.double() for q in (th, x))
    th.requires_grad_(not half)
    D, rest = 64, th
    W1, b1, W2, b2, w3, b3 = torch.split(rest, [D * D, D, D * D, D, D, 1])
    gelu = lambda z: 0.5 * z * (1 + torch.erf(z / math.sqrt(2)))  # noqa: E731
    z = gelu(gelu(x @ W1.reshape(D, D).T + b1) @ W2.reshape(D, D).T + b2) @ w3 + b3
    if half:
        return z
    loss = (z.clamp(min=0) - z * y.double() + torch.log1p(torch.exp(-z.abs()))).mean()
    (g,) = torch.autograd.grad(loss, th)
    m1, v1 = 0.9 * m.double() + 0.1 * g, 0.999 * v.double() + 0.001 * g * g
    new = th.detach() - 3e-3 * (m1 / (1 - 0.9**200)) / ((v1 / (1 - 0.999**200)).sqrt() + 1e-8)
    return {"grad": g, "theta": new, "m": m1, "v": v1}


def exact(case, seed):
    path = case["path"]
    if path in ("train", "classify"):
        return exact_classifier(case, seed)
    if path == "points":
        return exact_points(case, seed)
    if path == "graph":
        return [exact(c, seed + i) for i, c in enumerate(small_trees(case))]
    f_leaf, f_cut = sample(case, seed)
    L, n = f_leaf.shape[1:]
    fe = exact_extension(case, f_leaf, f_cut)
    direct = float(L) * L * n * 576  # log evaluations of the direct sum
    V = exact_potential(case, fe) if direct <= 4e10 else None
    if path != "batch":
        fe, V = fe[0], V[0] if V is not None else None
    return {"fe": fe, "V": V}
