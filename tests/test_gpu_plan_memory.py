"""Device memory of plans: everything a plan allocated - the batched
extension's buffers among it - is free again once the plan is closed or its
precision is set.  Nothing of torch's is allocated between the two readings of
the free memory, so they may differ by less than one of the plan's buffers of
batched products (n_cut x nrhs x N_G doubles, several times the granularity of
device allocations)."""
import numpy as np
import pytest

import gpu_cases as G
from paper_2211_14537_amd import vfx

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("how", ["close", "precision"])
def test_batch_buffers_return(gpu_device, how):
    import torch
    nrhs, rounds = 256, 4
    G.say(f"case starfish_small nrhs={nrhs} {how}")
    case = G.setup("starfish_small", p=24)
    tr, ctx = case["tree"], case["ctx"]
    FL = torch.tensor(np.repeat(case["f_leaf"][None], nrhs, 0), device=gpu_device)
    FC = torch.tensor(np.repeat(case["f_cut"][None], nrhs, 0), device=gpu_device)
    FE, V = torch.empty_like(FL), torch.empty_like(FL)

    def once(plan):
        if plan is None or how == "close":
            plan = vfx.Plan(ctx, tr["level"], tr["ix"], tr["iy"], tr["kind"], tr["mask"])
        plan.execute_batch(nrhs, FL, FC, FE, V)
        torch.cuda.synchronize()
        if how == "close":
            plan.close()
        else:
            plan.set_precision(0)
        torch.cuda.synchronize()
        return plan

    plan = once(None)  # the context's tables and the runtime's own memory
    free0 = torch.cuda.mem_get_info()[0]
    for _ in range(rounds):
        plan = once(plan)
    lost = free0 - torch.cuda.mem_get_info()[0]
    buffer = 8 * case["plan"].n_cut * nrhs * ctx.n_support
    G.say(f"    {lost / 2 ** 20:.1f} MiB fewer free after {rounds} rounds (one buffer {buffer / 2 ** 20:.1f} MiB)")
    assert buffer > 4 * 2 ** 20 and lost < buffer
