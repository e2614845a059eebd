"""Captured loops of networks with cells larger than LDS, alone and beside scheduled
groups: the first step leaves the factors in the device scratch and the later
ones keep them (the state goes back to the user's array once a launch), and the
result equals single steps bit for bit in every right-hand-side form."""
import numpy as np
import pytest

from workloads import cable_values, grow_random_forest

pytestmark = pytest.mark.gpu

NETWORKS = {
    "large": ([20000, 9000], {}),                              # streamed groups alone
    "mixed": ([50, 20000, 500, 7000], {}),                     # beside scheduled groups
    "packed": ([1500, 400, 900] * 12, dict(max_group_unknowns=16000, group_width=512)),  # several cells in a group
}


def kernels(run):
    """Names of the kernels that a call launched, with their number."""
    import torch
    from collections import Counter
    from torch.profiler import ProfilerActivity, profile
    with profile(activities=[ProfilerActivity.CUDA]) as pr:
        run()
        torch.cuda.synchronize()
    return Counter(e.name.split("<")[0].split("(")[0].split("::")[-1] for e in pr.events() if "k_" in e.name)


@pytest.mark.parametrize("name", list(NETWORKS))
@pytest.mark.parametrize("form", ["cv", "current", "noise"])
@pytest.mark.parametrize("steps", [1, 2, 3])
def test_loop_keeps_the_factors(name, form, steps):
    import torch
    from paper_1810_12742_amd import Plan
    sizes, opts = NETWORKS[name]
    f = grow_random_forest(np.random.default_rng(101), len(sizes), target_size=np.array(sizes))
    s = cable_values(f, np.random.default_rng(102), a_kind="cable", dt=0.025)
    p = Plan(f.parent, f.cell_offsets, **opts)
    assert p.info["kernel"] == 1 and p.info["workspace_groups"] > 0
    d, u, c, v0 = (torch.from_numpy(a).cuda() for a in (s.diag, s.upper, s.c, s.rhs))
    i = torch.from_numpy(0.1 * np.random.default_rng(103).standard_normal(f.n)).cuda()
    kw = dict(cv={}, current=dict(i_inj=i), noise=dict(noise_sigma=0.1, noise_seed=3))[form]
    v, want = v0.clone(), v0.clone()
    loop = p.timeloop(d, u, c, v, steps, first_step=4, **kw)
    for rep in range(3):
        for k in range(steps):
            p.timestep(d, u, c, want, want, step=4 + k, **kw)
        launched = kernels(loop.launch)
        assert launched["k_stream_store"] == 1 and launched["k_stream_sweep"] == steps, launched
        assert torch.equal(v, want), rep
    loop.close()
    p.close()
