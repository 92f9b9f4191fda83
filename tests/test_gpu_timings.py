"""Per-phase times.  A tree that runs on one stream has disjoint phases, so
they add up to at most the total (but for the resolution of the event times,
10 ns a time, two times an interval); and P2L is timed where it runs, also with
the near field in mixed precision: the same kernel on the same entries takes
the same time, which the events of an empty interval (a few us) do not."""
import numpy as np
import pytest

import gpu_cases as G

pytestmark = pytest.mark.gpu


def phases(case, nrhs, device, reps=10):
    import torch
    FL = torch.tensor(np.repeat(case["f_leaf"][None], nrhs, 0), device=device)
    FC = torch.tensor(np.repeat(case["f_cut"][None], nrhs, 0), device=device)
    FE, V = torch.empty_like(FL), torch.empty_like(FL)
    for _ in range(3):
        case["plan"].execute_batch(nrhs, FL, FC, FE, V)
    case["plan"].set_timing(True)
    for _ in range(reps):
        case["plan"].execute_batch(nrhs, FL, FC, FE, V)
    t = case["plan"].timings()
    case["plan"].set_timing(False)
    assert t.pop("count") == reps
    G.say("    " + " ".join(f"{k} {1e3 * v:.1f}" for k, v in t.items()))
    return t


@pytest.mark.parametrize("name,mode", [("starfish_small", 0), ("starfish_small", 2), ("disk_adaptive_small", 0)])
def test_phases_of_one_stream_are_disjoint(gpu_device, name, mode):
    G.say(f"case {name} mode={mode}")
    case = G.setup(name, p=24 if name == "starfish_small" else 20)
    assert case["plan"].n_leaves < 1000  # everything on the caller's stream
    if mode:
        case["plan"].set_precision(mode)
    t = phases(case, 1, gpu_device)
    total = t.pop("total")
    assert 0.0 < sum(t.values()) <= total + 2 * 1e-5 * len(t)
    assert t["fe_init"] == 0.0 and t["p2m_up"] > 0.0 and t["m2l"] > 0.0 and t["far"] > 0.0


@pytest.mark.parametrize("mode", [1, 2])
def test_p2l_is_timed_where_it_runs(gpu_device, mode):
    G.say(f"case starfish_small mode={mode}")
    case = G.setup("starfish_small", p=24)
    assert case["plan"].stats()["n_list4"] > 0
    ref = phases(case, 256, gpu_device)["p2l"]
    case["plan"].set_precision(mode)
    got = phases(case, 256, gpu_device)["p2l"]
    G.say(f"    P2L {1e3 * ref:.1f} us with FP64 pairs, {1e3 * got:.1f} us with mixed pairs")
    assert ref >= 0.04 and got >= 0.3 * ref
