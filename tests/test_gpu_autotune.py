"""The autotuner reports a choice only where there is one: dense_mtb, which no
kernel depends on, is always 4 (a choice by timing noise would give 8 in half
of the calls), and at K < 16, where no kernel depends on the work-group cap,
the plan keeps the cap it has."""
import pytest

import gpu_cases as G

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("name,p", [("starfish_small", 24), ("disk_adaptive_small", 20)])
def test_choice(gpu_device, name, p):
    import torch
    G.say(f"case {name}")
    case = G.setup(name, p=p)
    fl = torch.tensor(case["f_leaf"], device=gpu_device)
    fc = torch.tensor(case["f_cut"], device=gpu_device)
    fe, V = torch.empty_like(fl), torch.empty_like(fl)
    case["plan"].execute(fl, fc, fe, V)
    torch.cuda.synchronize()
    want = V.clone()
    case["plan"].set_launch(300, 8)
    for _ in range(8):
        V.fill_(float("nan"))
        ch = case["plan"].autotune(1, fl, fc, fe, V, reps=1)
        torch.cuda.synchronize()
        G.say(f"    {ch}")
        assert ch["dense_mtb"] == 4 and torch.equal(V, want)
        assert ch["near_wgs"] in ((256, 512, 768, 1024) if case["K"] == 16 else (300,))
