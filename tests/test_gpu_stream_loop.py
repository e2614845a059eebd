"""Captured loops of networks with cells larger than LDS, alone and beside scheduled
groups: the first step leaves the factors in the device scratch and the later
ones keep them (the state goes back to the user's array once a launch), and the
result equals single steps bit for bit in every right-hand-side form."""
import ctypes

import numpy as np
import pytest

from workloads import cable_values, grow_random_forest

pytestmark = pytest.mark.gpu

NETWORKS = {
    "large": ([20000, 9000], {}),                              # streamed groups alone
    "mixed": ([50, 20000, 500, 7000], {}),                     # beside scheduled groups
    "packed": ([1500, 400, 900] * 12, dict(max_group_unknowns=16000, group_width=512)),  # several cells in a group
}


def graph_nodes(loop):
    """Kernels of a captured loop: the nodes of its graph, the first member of the
    handle's struct."""
    from paper_1810_12742_amd.hines import load
    lib = load()  # looked up through the library, so in the runtime that it uses
    lib.hipGraphGetNodes.argtypes = [ctypes.c_void_p, ctypes.c_void_p, ctypes.POINTER(ctypes.c_size_t)]
    graph = ctypes.cast(loop._h, ctypes.POINTER(ctypes.c_void_p))[0]
    count = ctypes.c_size_t(0)
    assert lib.hipGraphGetNodes(graph, None, ctypes.byref(count)) == 0
    return count.value


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
    # a stage and a sweep a step, one store; the scheduled groups' launches beside them
    assert graph_nodes(loop) == 2 * steps + 1 + (p.info["nclasses"] - 1)
    for rep in range(3):
        for k in range(steps):
            p.timestep(d, u, c, want, want, step=4 + k, **kw)
        loop.launch()
        assert torch.equal(v, want), rep
    loop.close()
    p.close()
