"""Noise loops of cell-lane plans on both sides of the rule that has the draws made
beside the steps (up to 1,200 waves) or inside them: what the loop allocates (50
bytes per walk slot, two steps' draws, against 34), and the result against
the eager steps, bit for bit."""
import numpy as np
import pytest

from workloads import cable_values, full_binary_forest

pytestmark = pytest.mark.gpu


# cells of 75 compartments, two lanes each: 32 to a wave
@pytest.mark.parametrize("cells,beside", [(32 * 1024, True), (32 * 1025, True), (32 * 1200, True), (32 * 1201, False)])
def test_draws_beside_up_to_1200_waves(cells, beside):
    import torch
    from paper_1810_12742_amd import Plan
    f = full_binary_forest(cells)
    s = cable_values(f, np.random.default_rng(91), a_kind="cable", dt=0.025)
    p = Plan(f.parent, f.cell_offsets, cell_lanes=1)
    assert p.table("cell_waves").size // 3 == cells // 32
    d, u, c, v0 = (torch.from_numpy(a).cuda() for a in (s.diag, s.upper, s.c, s.rhs))
    v, want = v0.clone(), v0.clone()
    torch.cuda.synchronize()
    free = torch.cuda.mem_get_info()[0]
    loop = p.timeloop(d, u, c, v, 3, noise_sigma=0.1, noise_seed=3)
    taken = (free - torch.cuda.mem_get_info()[0]) / p.layout_size
    assert (taken > 49) == beside and taken > 33
    for rep in range(2):
        for k in range(3):
            p.timestep(d, u, c, want, want, noise_sigma=0.1, noise_seed=3, step=k)
        loop.launch()
        assert torch.equal(v, want), rep
    loop.close()
    p.close()
