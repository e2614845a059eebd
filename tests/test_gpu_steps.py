"""GPU: several steps of the time loop and of its adjoint in one call against
the single-step calls in turn.  The states and traces are the same bit for bit
(the loop repeats the products of one step); the adjoints agree to 1e-13 of the
largest value: the right-hand side at a root may be rounded once instead of
twice, 2^-53 per step over at most 20 steps.  Shapes: cells around the elements
a thread keeps in registers (18 with a current), many cells in a group (the first
root of a thread is kept, the rest looked up), groups that are not one user range, cells too large
for LDS, and plans of cell lanes (both fall back to single steps)."""
import numpy as np
import pytest

from workloads import cable_values, grow_random_forest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("sizes,steps,opts", [
    ([1], 3, {}), ([4608], 4, {}), ([4609, 700], 3, {}), ([1152, 1153, 2600] * 350, 2, {}),
    ([1] * 63 + [5] * 270, 5, {}), ([30, 900, 31, 1700, 60] * 60, 3, dict(cell_order=1)),
    ([20, 50], 257, {}), ([8000, 300], 3, {}), ([300] * 40, 4, dict(cell_lanes=2)), ([300], 1, {})])
@pytest.mark.parametrize("current", [True, False])
def test_steps_equal_single_calls(sizes, steps, opts, current):
    import torch
    from paper_1810_12742_amd import Plan
    sizes = np.asarray(sizes, dtype=np.int64)
    f = grow_random_forest(np.random.default_rng(41), len(sizes), target_size=sizes)
    s = cable_values(f, np.random.default_rng(42), a_kind="cable", dt=0.025)
    p = Plan(f.parent, f.cell_offsets, f.branch_offsets, **opts)
    dev = torch.device("cuda")
    rng = np.random.default_rng(43)
    d, u, c, v0 = (torch.from_numpy(a).to(dev) for a in (s.diag, s.upper, s.c, s.rhs))
    kw = dict(i_inj=torch.from_numpy(0.1 * rng.standard_normal(f.n)).to(dev)) if current else {}
    want, wtr, v = [], [], v0
    for k in range(steps):
        v = p.timestep(d, u, c, v, **kw)
        want.append(v)
        wtr.append(p.gather_roots(v))
    states = torch.full((steps, f.n), float("nan"), dtype=torch.float64, device=dev)
    traces = torch.full((steps, f.ncells), float("nan"), dtype=torch.float64, device=dev)
    last = torch.empty_like(v0)
    p.run_steps(d, u, c, v0, steps, states=states, v_out=last, traces=traces, **kw)
    assert torch.equal(states, torch.stack(want)) and torch.equal(traces, torch.stack(wtr))
    assert torch.equal(last, want[-1])
    inplace = v0.clone()
    p.run_steps(d, u, c, inplace, steps, v_out=inplace, traces=traces, **kw)
    assert torch.equal(inplace, want[-1]) and torch.equal(traces, torch.stack(wtr))

    steps = min(steps, 20)
    G = torch.from_numpy(rng.standard_normal((steps, f.ncells))).to(dev)
    for lam_in in (None, torch.from_numpy(rng.standard_normal(f.n)).to(dev)):
        lams = torch.full((steps, f.n), float("nan"), dtype=torch.float64, device=dev)
        p.adjoint_steps(d, u, c, lam_in, G, lams)
        lam, ref = lam_in, []
        for k in range(steps - 1, -1, -1):
            lam = p.solve(d, u, p.adjoint_rhs(c, lam, G[k]))
            ref.insert(0, lam)
        ref = torch.stack(ref)
        assert float((lams - ref).abs().max()) <= 1e-13 * float(ref.abs().max())
    st = torch.stack(want[:steps])
    g1 = [torch.from_numpy(rng.standard_normal(f.n)).to(dev) for _ in range(3)]
    g2 = [g.clone() for g in g1]
    for k in range(steps - 1, -1, -1):
        p.adjoint_accumulate(lams[k], st[k], st[k - 1] if k else v0, *g1)
    p.adjoint_accumulate_steps(lams, st, v0, *g2)
    assert all(torch.equal(a, b) for a, b in zip(g1, g2))
    p.close()
