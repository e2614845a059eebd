"""GPU parity of the streamed groups (cells whose image exceeds LDS) against the
FP64 oracle, in every right-hand-side form, alone, beside scheduled groups and
in a captured loop.  Tolerance: 1e-12 per cell, the bound of every FP64 solve
here.  The schedule's tables are replayed by the setup of every plan."""
import numpy as np
import pytest

import oracle
from workloads import Forest, cable_values, grow_random_forest

pytestmark = pytest.mark.gpu

TOL = 1e-12


def chain(n):
    return Forest(np.arange(-1, n - 1, dtype=np.int32), np.array([0, n]), np.array([0, n]))


def comb(n, every):
    """A chain with a leaf on every ``every``-th compartment."""
    m = n * every // (every + 1)
    par = list(range(-1, m - 1)) + [k for k in range(0, m, every)]
    par = np.array(par[:n], dtype=np.int32)
    return Forest(par, np.array([0, len(par)]), np.arange(len(par) + 1, dtype=np.int64))


def grown(sizes):
    return grow_random_forest(np.random.default_rng(51), len(sizes), target_size=np.array(sizes))


# cells of 20,000 compartments; the largest that the groups take; a cable (one lane,
# 1,000 steps); a comb (contributions in every chunk); many lanes' worth of short
# branches; large cells between small ones
@pytest.mark.parametrize("case", ["c3", "largest", "cable", "comb", "mixed"])
def test_streamed_cells(case):
    import torch
    from paper_1810_12742_amd import Plan
    f = {"c3": lambda: grown([20000] * 3), "largest": lambda: grown([32700]), "cable": lambda: chain(8000),
         "comb": lambda: comb(9000, 4), "mixed": lambda: grown([50, 20000, 500, 7000, 5000, 50, 12345] * 4)}[case]()
    s = cable_values(f, np.random.default_rng(52), a_kind="cable", dt=0.025)
    p = Plan(f.parent, f.cell_offsets)
    large = int((np.diff(f.cell_offsets) > 6000).sum())
    assert p.info["kernel"] == 1 and p.info["workspace_groups"] == large > 0
    dev = torch.device("cuda")
    d, u, b, c = (torch.from_numpy(a).to(dev) for a in (s.diag, s.upper, s.rhs, s.c))
    I = torch.from_numpy(0.1 * s.rhs).to(dev)
    noise = oracle.noise(3, 7, np.arange(f.n, dtype=np.int64), 0.1)

    def check(got, rhs):
        xo = oracle.solve(f, s.diag, s.upper, rhs)
        err = np.maximum.reduceat(np.abs(got - xo), f.cell_offsets[:-1])
        assert np.max(err / np.maximum.reduceat(np.abs(xo), f.cell_offsets[:-1])) <= TOL
    check(p.solve(d, u, b).cpu().numpy(), s.rhs)
    check(p.timestep(d, u, c, b).cpu().numpy(), s.c * s.rhs)
    check(p.timestep(d, u, c, b, i_inj=I).cpu().numpy(), s.c * s.rhs + 0.1 * s.rhs)
    check(p.timestep(d, u, c, b, noise_sigma=0.1, noise_seed=3, step=7).cpu().numpy(), s.c * s.rhs + noise)
    x = b.clone()
    p.solve(d, u, x, out=x)  # in place
    check(x.cpu().numpy(), s.rhs)
    v, want = b.clone(), b.clone()
    loop = p.timeloop(d, u, c, v, 3, i_inj=I)
    for rep in range(2):
        for _ in range(3):
            p.timestep(d, u, c, want, want, i_inj=I)
        loop.launch()
        assert torch.equal(v, want), rep
    loop.close()
    p.close()
