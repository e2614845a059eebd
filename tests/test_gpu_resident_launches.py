"""GPU parity of the LDS-resident plan when groups of several LDS classes share a
launch (few groups in a class) and when they do not, against the FP64 oracle
within the 1e-12 of every FP64 solve."""
import numpy as np
import pytest

import oracle
from workloads import cable_values, grow_random_forest

pytestmark = pytest.mark.gpu


# the smallest class beside the largest; one class; classes of more than one round of
# the device (cells of 1,000 do not pair at the default packing) beside small ones
@pytest.mark.parametrize("sizes,launches", [([30] * 3 + [5000], 1), ([2500] * 300, 1),
                                            ([1000] * 1600 + [5000] * 3 + [2500] * 4, None)])
@pytest.mark.parametrize("reroot", [False, True])
def test_merged_classes(sizes, launches, reroot):
    import torch
    from paper_1810_12742_amd import Plan
    f = grow_random_forest(np.random.default_rng(61), len(sizes), target_size=np.array(sizes))
    s = cable_values(f, np.random.default_rng(62), a_kind="cable", dt=0.025)
    p = Plan(f.parent, f.cell_offsets, resident=True, rebalance_root=reroot)
    assert p.info["kernel"] == 4
    if launches:
        assert p.info["nclasses"] == launches
    d, u, b = (torch.from_numpy(a).cuda() for a in (s.diag, s.upper, s.rhs))
    x = p.solve(d, u, b).cpu().numpy()
    xo = oracle.solve(f, s.diag, s.upper, s.rhs)
    err = np.maximum.reduceat(np.abs(x - xo), f.cell_offsets[:-1])
    assert np.max(err / np.maximum.reduceat(np.abs(xo), f.cell_offsets[:-1])) <= 1e-12
    p.close()
