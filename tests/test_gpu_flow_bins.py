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


# a group to a workgroup of four waves: a batch holds 16, 11 or 10 elements a thread by
# right-hand side (4,096, 2,816, 2,560 compartments), two batches in flight
@pytest.mark.parametrize("n", [1, 63, 64, 255, 256, 257, 2560, 2561, 2816, 2817, 4096, 4097, 5000, 5500])
def test_one_cell_at_the_staging_batch_edges(n):
    solve_and_check([n])


# groups of one cell each (1,000 compartments do not pair under the default cap):
# one group per workgroup (of four or two waves) up to 1,023, bins of 2 to 8 above, there
# with batches of 1,024, 704 and 640 compartments; mixed sizes in one bin;
# groups that are not one user range (cells sorted by size)
@pytest.mark.parametrize("cells,opts", [(256, {}), (257, {}), (512, {}), (513, {}), (1023, {}), (1024, {}), (2500, {}),
                                        (700, dict(cell_order=1))])
def test_bins_of_mixed_groups(cells, opts):
    rng = np.random.default_rng(cells)
    solve_and_check(rng.choice([40, 300, 1000, 2500, 4500], size=cells, p=[0.2, 0.2, 0.4, 0.15, 0.05]), **opts)


def comb_cell(n):
    """A chain with a leaf on every compartment: each leaf is a path of its own,
    padded to a whole chunk, so the step schedule's image does not fit LDS."""
    parent = np.empty(n, dtype=np.int32)
    parent[0::2] = np.arange(-2, n - 2, 2)
    parent[0] = -1
    parent[1::2] = np.arange(0, n - 1, 2)
    return parent


# 1e-12 where one FP64 elimination gives the result, 1e-11 (the refinement's
# bound after three sweeps) where the FP32 sweeps run
@pytest.mark.parametrize("comb", [0, 2000])
@pytest.mark.parametrize("sweeps", [1, 3])
def test_refined_solve_of_scheduled_and_level_groups(comb, sweeps):
    import torch
    from paper_1810_12742_amd import Plan
    from workloads import Forest
    f = grow_random_forest(np.random.default_rng(5), 40, target_size=np.full(40, 700))
    parent, offs = f.parent, f.cell_offsets
    if comb:
        q = comb_cell(comb)
        parent = np.concatenate([parent, np.where(q < 0, -1, q + f.n).astype(np.int32)])
        offs = np.append(offs, offs[-1] + comb)
    f = Forest(parent, offs, np.arange(len(parent) + 1, dtype=np.int64))
    s = cable_values(f, np.random.default_rng(6), a_kind="cable", dt=0.025)
    d32, u32 = s.diag.astype(np.float32), s.upper.astype(np.float32)
    xo = oracle.solve(f, d32.astype(np.float64), u32.astype(np.float64), s.rhs)
    p = Plan(parent, offs)
    assert p.info["kernel"] == 1 and p.info["nclasses"] == (2 if comb else 1)
    dev = torch.device("cuda")
    D, U, B = (torch.from_numpy(a).to(dev) for a in (d32, u32, s.rhs))
    for out in (None, B):  # the second in place
        x = p.solve_mixed(D, U, B, out=out, sweeps=sweeps).cpu().numpy()
        err = np.maximum.reduceat(np.abs(x - xo), offs[:-1]) / np.maximum.reduceat(np.abs(xo), offs[:-1])
        assert np.max(err[:40]) <= TOL
        if comb and sweeps == 3:
            assert err[40] <= 1e-11
    p.close()


# Captured loops against the same steps one by one, bit for bit, and against the
# oracle's loop.  Sizes around the elements that a group's threads keep in registers
# (24 or, with a current, 18 each, in one to four waves), several cells in a group, groups
# that are not one user range, loops of more than one launch (256 steps).
@pytest.mark.parametrize("form", ["cv", "current", "noise"])
@pytest.mark.parametrize("sizes,steps,opts", [
    ([4608], 3, {}), ([4609], 2, {}), ([5500], 2, {}), ([1, 64, 256, 257], 3, {}),
    ([2304, 2305] * 270, 2, {}), ([1152, 1153, 1536, 1537, 2100] * 220, 2, {}),
    ([1] * 130 + [40] * 30, 5, {}), ([30, 900, 31, 1700, 60] * 60, 3, dict(cell_order=1)),
    ([25, 300], 256, {}), ([25, 300], 257, {}), ([300], 1, {})])
def test_captured_loop_equals_single_steps(form, sizes, steps, opts):
    import torch
    from paper_1810_12742_amd import Plan
    sizes = np.asarray(sizes, dtype=np.int64)
    f = grow_random_forest(np.random.default_rng(31), len(sizes), target_size=sizes)
    s = cable_values(f, np.random.default_rng(32), a_kind="cable", dt=0.025)
    p = Plan(f.parent, f.cell_offsets, f.branch_offsets, **opts)
    assert p.info["kernel"] == 1
    dev = torch.device("cuda")
    d, u, c, v0 = (torch.from_numpy(a).to(dev) for a in (s.diag, s.upper, s.c, s.rhs))
    I = 0.1 * np.random.default_rng(33).standard_normal(f.n)
    kw = dict(cv={}, current=dict(i_inj=torch.from_numpy(I).to(dev)), noise=dict(noise_sigma=0.1, noise_seed=3))[form]
    want = v0.clone()
    for k in range(2 * steps):
        # the second launch replays the steps of the first
        p.timestep(d, u, c, want, want, step=4 + k % steps, **kw)
        if k == steps - 1:
            first = want.cpu().numpy()
    v = v0.clone()
    loop = p.timeloop(d, u, c, v, steps, first_step=4, **kw)
    loop.launch()
    assert np.array_equal(v.cpu().numpy(), first)
    _ = (d * 2).sum().item()
    loop.launch()
    assert np.array_equal(v.cpu().numpy(), want.cpu().numpy())
    loop.close()
    ref = s.rhs
    for k in range(steps):
        rhs = s.c * ref
        if form == "current":
            rhs = rhs + I
        elif form == "noise":
            rhs = rhs + oracle.noise(3, 4 + k, np.arange(f.n, dtype=np.int64), 0.1)
        ref = oracle.solve(f, s.diag, s.upper, rhs)
    err = np.maximum.reduceat(np.abs(first - ref), f.cell_offsets[:-1])
    assert np.max(err / np.maximum.reduceat(np.abs(ref), f.cell_offsets[:-1])) <= TOL
    p.close()
