"""GPU parity of the flow kernel's bins (groups of different sizes sharing one
workgroup) and of its two-batch staging, against the FP64 oracle.  Tolerance:
1e-12 per cell, the bound of every FP64 solve here; the sums of one step have a
handful of terms and the recurrence is diagonally dominant, so the error stays
within a small multiple of 2^-53 times the tree's depth (below 500)."""
import numpy as np
import pytest

import oracle
from workloads import cable_values, grow_random_forest

pytestmark = pytest.mark.gpu

TOL = 1e-12


def solve_and_check(sizes, **opts):
    import torch
    from paper_1810_12742_amd import Plan
    sizes = np.asarray(sizes, dtype=np.int64)
    f = grow_random_forest(np.random.default_rng(21), len(sizes), target_size=sizes)
    s = cable_values(f, np.random.default_rng(22), a_kind="cable", dt=0.025)
    p = Plan(f.parent, f.cell_offsets, f.branch_offsets, **opts)
    assert p.info["kernel"] == 1
    dev = torch.device("cuda")
    d, u, b, c = (torch.from_numpy(a).to(dev) for a in (s.diag, s.upper, s.rhs, s.c))
    x = p.solve(d, u, b).cpu().numpy()
    I = torch.from_numpy(0.1 * s.rhs).to(dev)
    v = p.timestep(d, u, c, b, i_inj=I).cpu().numpy()
    z = p.timestep(d, u, c, b, noise_sigma=0.1, noise_seed=3, step=7).cpu().numpy()
    w = p.timestep(d, u, c, b).cpu().numpy()
    noise = oracle.noise(3, 7, np.arange(f.n, dtype=np.int64), 0.1)
    for got, rhs in ((x, s.rhs), (v, s.c * s.rhs + 0.1 * s.rhs), (z, s.c * s.rhs + noise), (w, s.c * s.rhs)):
        xo = oracle.solve(f, s.diag, s.upper, rhs)
        err = np.maximum.reduceat(np.abs(got - xo), f.cell_offsets[:-1])
        ref = np.maximum.reduceat(np.abs(xo), f.cell_offsets[:-1])
        assert np.max(err / ref) <= TOL
    p.close()


# one cell each: the staging batches hold 384, 448 and 640 compartments (by right-hand
# side), two in flight, the rest one after the other
@pytest.mark.parametrize("n", [1, 63, 384, 385, 448, 640, 641, 768, 896, 897, 1280, 1281, 1921, 5000])
def test_one_cell_at_the_staging_batch_edges(n):
    solve_and_check([n])


# groups of one cell each (1,000 compartments do not pair under the default cap):
# one group per workgroup up to 256, bins of 1 to 8 above; mixed sizes in one bin;
# groups that are not one user range (cells sorted by size)
@pytest.mark.parametrize("cells,opts", [(256, {}), (257, {}), (1023, {}), (1024, {}), (2500, {}),
                                        (700, dict(cell_order=1))])
def test_bins_of_mixed_groups(cells, opts):
    rng = np.random.default_rng(cells)
    solve_and_check(rng.choice([40, 300, 1000, 2500, 4500], size=cells, p=[0.2, 0.2, 0.4, 0.15, 0.05]), **opts)
