"""What hines_run_steps and hines_adjoint_steps accept of overlapping arrays, the same
on plans that run the steps inside LDS and on plans that run them one by one:
v_out on v_in, and whole rows of the output after its first; every other overlap
is refused."""
import numpy as np
import pytest

from workloads import cable_values, grow_random_forest

pytestmark = pytest.mark.gpu

STEPS = 4


@pytest.fixture(scope="module", params=[{}, dict(cell_lanes=1), dict(level_sync=True)], ids=["lds", "lanes", "level"])
def setting(request):
    import torch
    from paper_1810_12742_amd import Plan
    f = grow_random_forest(np.random.default_rng(81), 30, target_size=np.full(30, 200))
    s = cable_values(f, np.random.default_rng(82), a_kind="cable", dt=0.025)
    p = Plan(f.parent, f.cell_offsets, **request.param)
    dev = torch.device("cuda")
    d, u, c, v = (torch.from_numpy(a).to(dev) for a in (s.diag, s.upper, s.c, s.rhs))
    yield f, p, d, u, c, v
    p.close()


def rows(n, m=STEPS):
    import torch
    return torch.full((m, n), float("nan"), dtype=torch.float64, device="cuda")


def test_run_steps(setting):
    import torch
    f, p, d, u, c, v = setting
    want, tr = rows(f.n), rows(f.ncells)
    p.run_steps(d, u, c, v, STEPS, states=want, traces=tr)
    # the last state is a row of states; the start is one
    st = rows(f.n)
    p.run_steps(d, u, c, v, STEPS, states=st, v_out=st[-1])
    assert torch.equal(st, want)
    for k in range(1, STEPS):
        st = rows(f.n)
        st[k].copy_(v)
        p.run_steps(d, u, c, st[k], STEPS, states=st)
        assert torch.equal(st, want)
    same = v.clone()
    p.run_steps(d, u, c, same, STEPS, v_out=same)
    assert torch.equal(same, want[-1])

    buf = torch.zeros(STEPS * f.n + 7, dtype=torch.float64, device="cuda")
    st, n = buf[:STEPS * f.n].view(STEPS, f.n), f.n
    other, out = rows(f.n), torch.empty_like(v)
    for kw in (dict(v_in=buf[:n], states=st), dict(v_in=buf[3:n + 3], states=st),
               dict(v_in=buf[2 * n + 1:3 * n + 1], states=st), dict(v_in=v, states=st, v_out=buf[n - 1:2 * n - 1]),
               dict(v_in=v, states=st, v_out=st[0]), dict(v_in=v, states=st, i_inj=st[2]),
               dict(v_in=buf[:n], v_out=buf[5:n + 5]), dict(v_in=v, v_out=out, i_inj=out),
               dict(v_in=v, states=st, traces=buf[7:7 + STEPS * f.ncells].view(STEPS, -1)),
               dict(v_in=buf[:n], states=other, traces=buf[7:7 + STEPS * f.ncells].view(STEPS, -1)),
               dict(v_in=v, v_out=buf[:n], traces=buf[n - 1:n - 1 + STEPS * f.ncells].view(STEPS, -1)),
               dict(v_in=v, states=other, i_inj=buf[:n], traces=buf[:STEPS * f.ncells].view(STEPS, -1))):
        with pytest.raises(RuntimeError):
            p.run_steps(d, u, c, kw.pop("v_in"), STEPS, **kw)
    for m in ("d", "u", "c"):
        with pytest.raises(RuntimeError):
            p.run_steps(*(st[1] if k == m else a for k, a in (("d", d), ("u", u), ("c", c))), v, STEPS, states=st)


def test_adjoint_steps(setting):
    import torch
    f, p, d, u, c, lam = setting
    G = torch.from_numpy(np.random.default_rng(83).standard_normal((STEPS, f.ncells))).cuda()
    want = rows(f.n)
    p.adjoint_steps(d, u, c, lam, G, want)
    for k in range(1, STEPS):
        lams = rows(f.n)
        lams[k].copy_(lam)
        p.adjoint_steps(d, u, c, lams[k], G, lams)
        assert torch.equal(lams, want)
    buf = torch.zeros(STEPS * f.n + 7, dtype=torch.float64, device="cuda")
    lams, n = buf[:STEPS * f.n].view(STEPS, f.n), f.n
    for bad in (buf[:n], buf[n + 1:2 * n + 1]):
        with pytest.raises(RuntimeError):
            p.adjoint_steps(d, u, c, bad, G, lams)
    with pytest.raises(RuntimeError):
        p.adjoint_steps(d, u, c, lam, buf[5:5 + STEPS * f.ncells].view(STEPS, -1), lams)
    for m in ("d", "u", "c"):
        with pytest.raises(RuntimeError):
            p.adjoint_steps(*(lams[1] if k == m else a for k, a in (("d", d), ("u", u), ("c", c))), lam, G, lams)
