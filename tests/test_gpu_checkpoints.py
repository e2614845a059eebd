"""Traces and gradients do not depend on the distance of the checkpoints: one state
apart, more than the steps, or given with a minus sign (bit for bit: the recomputed
states are the forward run's); a distance of 0 is refused."""
import numpy as np
import pytest

from workloads import cable_values, grow_random_forest

pytestmark = pytest.mark.gpu


def test_distances():
    import torch
    from paper_1810_12742_amd import Plan
    from paper_1810_12742_amd.adjoint import soma_traces
    f = grow_random_forest(np.random.default_rng(121), 12, target_size=np.full(12, 150))
    s = cable_values(f, np.random.default_rng(122), a_kind="cable", dt=0.025)
    p = Plan(f.parent, f.cell_offsets)
    i = 0.1 * np.random.default_rng(123).standard_normal(f.n)

    def fit(every, steps=23):
        a, c, I = (torch.from_numpy(v).cuda().requires_grad_(True) for v in (s.a, s.c, i))
        torch.full((steps, f.ncells), float("nan"), dtype=torch.float64, device="cuda")  # what torch.empty may hold next
        tr = soma_traces(p, a, c, I, steps, every)
        return [tr.detach(), *torch.autograd.grad((tr ** 2).sum(), (a, c, I))]
    want = fit(10)
    assert all(bool(torch.isfinite(w).all()) for w in want) and float(want[0].abs().max()) > 0
    for every in (-10, 1, -1, 23, 100, -100):
        got = fit(every)
        assert torch.equal(got[0], want[0])
        for g, w in zip(got[1:], want[1:]):
            # where a block of adjoints ends its right-hand sides are rounded once more
            assert float((g - w).abs().max()) <= 1e-12 * float(w.abs().max())
    assert all(torch.equal(g, w) for g, w in zip(fit(-10), want))
    assert fit(10, 0)[0].shape == (0, f.ncells)
    with pytest.raises(ValueError):
        fit(0)
    p.close()
