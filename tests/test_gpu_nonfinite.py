"""Infinite and NaN values stay in their cell: a lane of the scheduled groups
eliminates paths of several cells in turn, and nothing of one may reach the next.
The other cells' results equal those of the same call on finite inputs bit for
bit, and the bad cells' roots are not finite (nothing is lost on the way)."""
import numpy as np
import pytest

from workloads import cable_values, grow_random_forest

pytestmark = pytest.mark.gpu

# groups of many small cells, a workgroup each; groups of more branches; bins of
# groups, a wave each; groups of several cells that exceed LDS
NETWORKS = {
    "packed": ([40, 75, 300, 8, 120] * 60, {}),
    "wide": ([500, 60, 900] * 40, dict(max_group_unknowns=4000, group_width=256)),
    "bins": ([700, 500, 300] * 1100, {}),
    "streamed": ([1500, 400, 900] * 20, dict(max_group_unknowns=16000, group_width=512)),
}


def systems(name):
    sizes, opts = NETWORKS[name]
    f = grow_random_forest(np.random.default_rng(71), len(sizes), target_size=np.array(sizes))
    s = cable_values(f, np.random.default_rng(72), a_kind="cable", dt=0.025)
    good = dict(d=s.diag, u=s.upper, b=s.rhs, c=s.c)
    bad = {k: a.copy() for k, a in good.items()}
    lo, hi = f.cell_offsets[:-1], f.cell_offsets[1:]
    cells = np.arange(2, f.ncells, 7)
    for k, cell in enumerate(cells):
        mid, tip, root = (lo[cell] + hi[cell]) // 2, hi[cell] - 1, lo[cell]
        if k % 5 == 0:
            bad["b"][tip] = np.nan
        elif k % 5 == 1:
            bad["b"][root] = np.inf
        elif k % 5 == 2:
            bad["d"][mid] = np.nan
        elif k % 5 == 3:
            bad["u"][tip] = -np.inf
        else:
            bad["d"][root] = np.nan
    return f, opts, good, bad, cells


CALLS = ["solve", "mixed1", "mixed3", "step", "current", "noise", "loop", "loop_current", "loop_noise", "run_steps",
         "adjoint_steps"]


# the refined solve is refused for groups that exceed LDS
@pytest.mark.parametrize("name,call", [(n, c) for n in NETWORKS for c in CALLS
                                       if n != "streamed" or not c.startswith("mixed")])
def test_other_cells_are_not_reached(name, call):
    import torch
    from paper_1810_12742_amd import Plan
    f, opts, good, bad, cells = systems(name)
    p = Plan(f.parent, f.cell_offsets, **opts)
    assert p.info["kernel"] == 1
    assert (p.info["workspace_groups"] > 0) == (name == "streamed")
    assert p.info["ngroups"] < f.ncells
    I = 0.1 * good["b"]

    def result(m):
        d, u, b, c, i = (torch.from_numpy(a).cuda() for a in (m["d"], m["u"], m["b"], m["c"], I))
        kw = dict(i_inj=i) if "current" in call else dict(noise_sigma=0.1, noise_seed=3) if "noise" in call else {}
        if call == "solve":
            return p.solve(d, u, b)
        if call.startswith("mixed"):
            return p.solve_mixed(d.float(), u.float(), b, sweeps=int(call[-1]))
        if call in ("step", "current", "noise"):
            return p.timestep(d, u, c, b, **kw)
        if call.startswith("loop"):
            v = b.clone()
            loop = p.timeloop(d, u, c, v, 3, **kw)
            for _ in range(2):
                loop.launch()
            torch.cuda.synchronize()
            loop.close()
            return v
        if call == "run_steps":
            rows = torch.empty(3, f.n, dtype=torch.float64, device="cuda")
            p.run_steps(d, u, c, b, 3, states=rows)
            return rows[-1]
        rows = torch.empty(3, f.n, dtype=torch.float64, device="cuda")
        p.adjoint_steps(d, u, c, b, torch.zeros(3, f.ncells, dtype=torch.float64, device="cuda"), rows)
        return rows[0]
    want, got = result(good).cpu().numpy(), result(bad).cpu().numpy()
    assert np.all(np.isfinite(want))
    hit = np.zeros(f.ncells, dtype=bool)
    hit[cells] = True
    assert not np.any(np.isfinite(got[f.cell_offsets[:-1][hit]]))
    ok = np.repeat(~hit, np.diff(f.cell_offsets))
    assert np.array_equal(got[ok], want[ok])
    p.close()
