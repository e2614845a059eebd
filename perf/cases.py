"""Workloads of the batched Hines solver, as a simulation program runs them.

Every case is a network of neuron-shaped cells in the numbering of the C-ABI
(include/hines.h): branches breadth first, compartments of a branch
consecutive.  A network repeats a pool of morphologies, as real networks do
(a few reconstructed cells of each type, placed many times); all values are
drawn per compartment.  The shapes are those of the repository's benchmark
configurations: ``c2`` cells (16 to 256 branches, 1,600 compartments on
average), ``c1`` cells (a full binary tree of 75 compartments), ``c3`` cells
(50, 500, 5,000 and 20,000 compartments mixed) and ``c5`` cells (1,000
compartments).

Fields of a case: ``call`` (the entry point), ``shape``, ``cells``, ``plan``
(which solver the plan selects), and per call ``dt``, ``steps`` (steps of a
time loop or of a trace), ``every`` (checkpoint distance), ``noise``, ``sweeps``.
"""
from __future__ import annotations

import numpy as np
import torch

from paper_1810_12742_amd import Plan
from paper_1810_12742_amd.adjoint import soma_traces

DEV = torch.device("cuda" if torch.cuda.is_available() else "cpu")
F64 = torch.float64

# Plan options by name: the default plan (packed groups), one lane per cell
# (depth-first walks and walks in index order), LDS-resident groups.
PLANS = {
    "default": {},
    "lanes": dict(cell_lanes=1),
    "index_lanes": dict(cell_lanes=2, cell_cut_percent=100, cell_max_cuts=3),
    "resident": dict(resident=True, rebalance_root=True, res_pack=3000),
}
SIGMA, NOISE_SEED = 0.1, 3
C3_SIZES, C3_WEIGHTS = (50, 500, 5000, 20000), (0.4, 0.3, 0.2, 0.1)


def listed():
    return [
        # a small circuit, solved once per step by a program with its own
        # right-hand side: latency and launches
        dict(name="solve_64", call="solve", shape="c2", cells=64, plan="default", dt=0.025),
        # many small identical cells (point-like neurons with short dendrites)
        dict(name="solve_binary_4096", call="solve", shape="c1", cells=4096, plan="default", dt=0.025),
        # an ordinary network with the default plan, a ragged cell count
        dict(name="solve_4099", call="solve", shape="c2", cells=4099, plan="default", dt=0.025),
        # the LDS-resident plan of the autotuner's list, re-rooted cells
        dict(name="solve_resident_2048", call="solve", shape="c2", cells=2048, plan="resident", dt=0.025),
        # a large network on the plan the autotuner picks for it (half of the
        # headline network of 65,536 cells)
        dict(name="solve_index_32768", call="solve", shape="c2", cells=32768, plan="index_lanes", dt=0.025),
        # matrix kept in FP32, solved in FP64, at a long time step
        dict(name="stored32_8191", call="stored32", shape="c2", cells=8191, plan="lanes", dt=1.0),
        # FP32 matrix with FP64 refinement, three sweeps
        dict(name="mixed_4096", call="mixed", shape="c2", cells=4096, plan="default", dt=0.025, sweeps=3),
        # a program that steps by itself with a constant injected current
        dict(name="step_current_8192", call="step", shape="c5", cells=8192, plan="default", dt=0.025),
        # captured time loop of a small circuit, constant current
        dict(name="loop_current_257", call="loop", shape="c2", cells=257, plan="default", dt=0.025, steps=100,
             noise=False),
        # captured time loop of a network of very unequal cells, noise current
        dict(name="loop_noise_c3_1000", call="loop", shape="c3", cells=1000, plan="default", dt=0.025, steps=20,
             noise=True),
        # captured time loop of a large network on cell lanes, noise current
        dict(name="loop_noise_lanes_12288", call="loop", shape="c2", cells=12288, plan="lanes", dt=0.025, steps=20,
             noise=True),
        # fitting conductances to soma traces: forward run and its adjoint
        dict(name="adjoint_1024", call="adjoint", shape="c5", cells=1024, plan="default", dt=0.025, steps=40,
             every=10),
    ]


# The ranges the listed cases stand for: cells from ... to, per kind of use.
RANGES = [
    dict(call="solve", shape="c2", plan="default", cells=(16, 8192)),
    dict(call="solve", shape="c1", plan="default", cells=(64, 16384)),
    dict(call="solve", shape="c2", plan="resident", cells=(256, 2048)),
    dict(call="solve", shape="c2", plan="index_lanes", cells=(2048, 24576)),
    dict(call="stored32", shape="c2", plan="lanes", cells=(512, 8192)),
    dict(call="mixed", shape="c2", plan="default", cells=(64, 4096)),
    dict(call="step", shape="c5", plan="default", cells=(64, 8192)),
    dict(call="loop", shape="c2", plan="default", cells=(16, 1024)),
    dict(call="loop", shape="c3", plan="default", cells=(64, 1000)),
    dict(call="loop", shape="c2", plan="lanes", cells=(1024, 12288)),
    dict(call="adjoint", shape="c5", plan="default", cells=(64, 1024)),
]


def draw(rng):
    r = rng.choice(RANGES)
    lo, hi = r["cells"]
    case = dict(r, cells=int(round(lo * (hi / lo) ** rng.random())))
    case["dt"] = rng.choice((0.001, 0.025, 1.0)) if case["call"] in ("stored32", "mixed") else 0.025
    if case["call"] == "mixed":
        case["sweeps"] = rng.choice((1, 2, 3, 3))
    if case["call"] == "loop":
        # the largest network of a loop runs no more steps than its listed case
        case["steps"] = rng.randint(5, 20) if case["plan"] == "lanes" or case["shape"] == "c3" else rng.randint(10, 100)
        case["noise"] = rng.random() < 0.5
    if case["call"] == "adjoint":
        case["steps"] = rng.randint(8, 40)
        case["every"] = rng.randint(3, 10)
    return case


# ---- morphologies --------------------------------------------------------------
def _cell(rng, shape):
    """(parent, branch of each compartment) of one cell; the root has parent -1."""
    if shape == "c1":  # full binary tree of depth 4, 5 compartments per branch
        par_b = [-1] + [(b - 1) // 2 for b in range(1, 15)]
        length = [5] * 15
    else:
        branches = int(rng.integers(16, 257)) if shape == "c2" else None
        size = None
        if shape == "c3":
            size = int(rng.choice(C3_SIZES, p=C3_WEIGHTS))
        elif shape == "c5":
            size = 1000
        par_b, length = [-1], [min(int(rng.geometric(1 / 12)), 64)]
        tips, total = [0], length[0]
        while (len(par_b) + 2 <= branches) if size is None else (total < size):
            new = []
            for t in tips:  # every tip splits with probability one half per round
                if rng.random() < 0.5 and (size is not None or len(par_b) + 2 <= branches):
                    for _ in range(2):
                        new.append(len(par_b))
                        par_b.append(t)
                        length.append(min(int(rng.geometric(1 / 12)), 64))
                        total += length[-1]
                else:
                    new.append(t)
            tips = new
        if size is not None:  # cut in creation order to the exact size
            keep, left = [], size
            for b in range(len(par_b)):
                if left <= 0:
                    break
                length[b] = min(length[b], left)
                left -= length[b]
                keep.append(b)
            par_b, length = par_b[:len(keep)], length[:len(keep)]
    # breadth-first branch numbering
    kids = [[] for _ in par_b]
    for b, p in enumerate(par_b):
        if p >= 0:
            kids[p].append(b)
    order = [0]
    for b in order:
        order.extend(kids[b])
    rank = {b: i for i, b in enumerate(order)}
    lens = np.array([length[b] for b in order], dtype=np.int64)
    end = np.cumsum(lens)
    parent = np.arange(-1, end[-1] - 1, dtype=np.int32)
    for i, b in enumerate(order):
        if i:
            parent[end[i] - lens[i]] = end[rank[par_b[b]]] - 1
    return parent, np.repeat(np.arange(len(order), dtype=np.int32), lens)


def _network(case, seed):
    """parent (int32[n]), cell_offsets (int64[cells + 1]) and the branch of every
    compartment (int32[n], numbered through the network)."""
    # the cells of a network are fixed by its shape and count (its size is then the
    # same for every seed); the seed says in which order they stand
    nc, shape = case["cells"], case["shape"]
    rng = np.random.default_rng(list(map(ord, shape)) + [nc])
    pool = [_cell(rng, shape) for _ in range(1 if shape == "c1" else min(nc, 192))]
    pick = rng.integers(0, len(pool), nc) if len(pool) < nc else np.arange(nc)
    np.random.default_rng(seed).shuffle(pick)
    sizes = np.array([len(p) for p, _ in pool], dtype=np.int64)[pick]
    nbr = np.array([int(b[-1]) + 1 for _, b in pool], dtype=np.int64)[pick]
    coff = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    boff = np.concatenate([[0], np.cumsum(nbr)[:-1]]).astype(np.int32)
    parent = np.concatenate([pool[k][0] for k in pick])
    parent += np.repeat(coff[:-1].astype(np.int32), sizes)
    parent[coff[:-1]] = -1
    branch = np.concatenate([pool[k][1] for k in pick])
    branch += np.repeat(boff, sizes)
    return parent, coff, branch


def _values(case, seed, parent, branch):
    """Cable coefficients on the device: edge conductances a, c = sigma c_m / dt,
    diag, upper, and draws b, v, i for right-hand side, state and current."""
    g = torch.Generator(device=DEV)
    g.manual_seed(seed * 7919 + 17)
    n = len(parent)
    par = torch.from_numpy(parent).to(DEV)
    root = par < 0
    rand = lambda m: torch.rand(m, generator=g, device=DEV, dtype=F64)  # noqa: E731
    if case["shape"] == "c1":
        a = 0.5 + 1.5 * rand(n)
        c = 0.1 + 0.9 * rand(n)
    else:
        rad = 0.2 + 1.8 * rand(int(branch[-1]) + 1)
        rb = rad[torch.from_numpy(branch).to(DEV).long()]
        a = 10.0 ** (4.0 * rand(n) - 2.0) * rb * rb
        c = (0.1 + 0.9 * rand(n)) / case["dt"]
    a = torch.where(root, torch.zeros_like(a), a)
    kids = torch.zeros(n, dtype=F64, device=DEV)  # at most two children: the sum has one rounding in any order
    kids.index_add_(0, par.clamp(min=0).long(), a)
    diag = (c + a) + kids
    normal = lambda m: torch.randn(m, generator=g, device=DEV, dtype=F64)  # noqa: E731
    return dict(a=a, c=c, diag=diag, upper=-a, b=normal(n), v=normal(n), i=0.1 * normal(n))


def _inputs(case, seed):
    parent, coff, branch = _network(case, seed)
    val = _values(case, seed, parent, branch)
    if case["call"] in ("mixed", "stored32"):
        val["diag"], val["upper"] = val["diag"].float(), val["upper"].float()
    if case["call"] == "adjoint":
        g = torch.Generator(device=DEV)
        g.manual_seed(seed * 104729 + 5)
        val["target"] = torch.randn(case["cells"], generator=g, device=DEV, dtype=F64)
    return parent, coff, val


# ---- what a program holds, and one pass ----------------------------------------
def prepare(case, seed):
    parent, coff, val = _inputs(case, seed)
    plan = Plan(parent, coff, keep_tables=False, **PLANS[case["plan"]])
    call = case["call"]
    st = dict(case=case, plan=plan)
    if call in ("solve", "stored32", "mixed"):
        st.update(d=val["diag"], u=val["upper"], b=val["b"], x=torch.empty_like(val["b"]))
    elif call == "step":
        st.update(d=val["diag"], u=val["upper"], c=val["c"], v=val["v"], i=val["i"], x=torch.empty_like(val["v"]))
    elif call == "loop":
        v = val["v"].clone()
        kw = dict(noise_sigma=SIGMA, noise_seed=NOISE_SEED) if case["noise"] else dict(i_inj=val["i"])
        loop = plan.timeloop(val["diag"], val["upper"], val["c"], v, case["steps"], **kw)
        st.update(v0=val["v"], v=v, loop=loop)
    elif call == "adjoint":
        st.update({k: val[k].clone().requires_grad_(True) for k in ("a", "c", "i")}, target=val["target"])
    return st


def run(st):
    case, plan = st["case"], st["plan"]
    call = case["call"]
    if call == "solve":
        return plan.solve(st["d"], st["u"], st["b"], out=st["x"])
    if call == "stored32":
        return plan.solve_stored32(st["d"], st["u"], st["b"], out=st["x"])
    if call == "mixed":
        return plan.solve_mixed(st["d"], st["u"], st["b"], out=st["x"], sweeps=case["sweeps"])
    if call == "step":
        return plan.timestep(st["d"], st["u"], st["c"], st["v"], st["x"], i_inj=st["i"])
    if call == "loop":  # a stretch of simulation from the stored state
        st["v"].copy_(st["v0"])
        st["loop"].launch()
        return st["v"]
    traces = soma_traces(plan, st["a"], st["c"], st["i"], case["steps"], case["every"])
    loss = ((traces - st["target"]) ** 2).sum()
    ga, gc, gi = torch.autograd.grad(loss, (st["a"], st["c"], st["i"]))
    return dict(traces=traces.detach(), grad_a=ga, grad_c=gc, grad_i=gi)


def _mean_size(shape):
    return {"c1": 75, "c2": 1600, "c5": 1000, "c3": int(np.dot(C3_SIZES, C3_WEIGHTS))}[shape]


def work(case):
    """Bytes a pass cannot do without (each input read once, each output written
    once) and its floating-point operations: elimination 3 multiply-adds, a
    division and a product, substitution one multiply-add per unknown."""
    n = case["cells"] * _mean_size(case["shape"])
    call, steps = case["call"], case.get("steps", 1)
    if call == "solve":
        return dict(bytes=32 * n, flops=9 * n)
    if call in ("stored32", "mixed"):
        return dict(bytes=24 * n, flops=9 * n)
    if call == "step":
        return dict(bytes=48 * n, flops=11 * n)
    if call == "loop":  # matrix, c, current and state in once, state out once; copy of the stored state
        noise = case["noise"]
        per = 6 + (60 if noise else 2)
        return dict(bytes=(56 if noise else 64) * n, flops=(4 + per * steps) * n)
    # forward: a, c, i in, traces out; backward: the same in, three gradients out
    return dict(bytes=(24 + 24 + 24) * n + 16 * steps * case["cells"], flops=(2 * 8 + 12) * steps * n)


# ---- the same results in plain 64-bit torch -------------------------------------
class _Tree:
    """Elimination and substitution level by level of the depth below the roots."""

    def __init__(self, parent, upper):
        p = torch.from_numpy(parent).to(DEV).long()
        self.root = p < 0
        depth = _depths(p)
        order = torch.argsort(depth, stable=True)
        ends = torch.cumsum(torch.bincount(depth), 0).tolist()
        self.idx = [order[a:b] for a, b in zip([0] + ends[:-1], ends)]
        self.par = [p[i] for i in self.idx]
        self.u = upper

    def factor(self, diag):
        self.d = diag.clone()
        self.f = torch.zeros_like(diag)
        for i, q in zip(reversed(self.idx[1:]), reversed(self.par[1:])):
            f = self.u[i] / self.d[i]
            self.f[i] = f
            self.d.index_add_(0, q, -f * self.u[i])
        return self

    def solve(self, rhs):
        b = rhs.clone()
        for i, q in zip(reversed(self.idx[1:]), reversed(self.par[1:])):
            b.index_add_(0, q, -self.f[i] * b[i])
        b /= self.d
        for i, q in zip(self.idx[1:], self.par[1:]):
            b[i] -= self.f[i] * b[q]
        return b


def _depths(p):
    """Depth of every compartment below its root, by pointer doubling."""
    up = torch.where(p < 0, torch.arange(len(p), device=p.device), p)
    dep = (p >= 0).long()
    while True:
        more = dep[up]
        if not bool(more.any()):
            return dep
        dep = dep + more
        up = up[up]


def _noise(step, n):
    """SIGMA times the standard normals of Philox4x32-10 keyed by compartment."""
    mask = 0xFFFFFFFF
    c0 = torch.arange(n, device=DEV, dtype=torch.int64)
    c1, c3 = torch.zeros_like(c0), torch.zeros_like(c0)
    c2 = torch.full_like(c0, step)
    k0, k1 = NOISE_SEED, 0

    def mul(m, x):  # 32 x 32 -> (high, low), the factors' halves multiplied apart
        lo, hi = m * (x & 0xFFFF), m * (x >> 16)
        mid = hi + (lo >> 16)
        return (mid >> 16) & mask, ((mid & 0xFFFF) << 16) | (lo & 0xFFFF)

    for _ in range(10):
        h0, l0 = mul(0xD2511F53, c0)
        h1, l1 = mul(0xCD9E8D57, c2)
        c0, c1, c2, c3 = h1 ^ c1 ^ k0, l1, h0 ^ c3 ^ k1, l0
        k0, k1 = (k0 + 0x9E3779B9) & mask, (k1 + 0xBB67AE85) & mask
    u1 = (((c0 << 20) | (c1 >> 12)).to(F64) + 0.5) * 2.0 ** -52
    u2 = (((c2 << 20) | (c3 >> 12)).to(F64) + 0.5) * 2.0 ** -52
    return SIGMA * torch.sqrt(-2.0 * torch.log(u1)) * torch.cos(2.0 * np.pi * u2)


def exact(case, seed):
    parent, coff, val = _inputs(case, seed)
    call = case["call"]
    if call in ("solve", "stored32", "mixed"):
        return _Tree(parent, val["upper"].double()).factor(val["diag"].double()).solve(val["b"])
    tree = _Tree(parent, val["upper"]).factor(val["diag"])
    if call == "step":
        return tree.solve(val["c"] * val["v"] + val["i"])
    if call == "loop":
        v = val["v"]
        for k in range(case["steps"]):
            v = tree.solve(val["c"] * v + (_noise(k, len(parent)) if case["noise"] else val["i"]))
        return v
    roots = torch.from_numpy(coff[:-1]).to(DEV)
    p = torch.from_numpy(parent).to(DEV).long().clamp(min=0)
    vs = [torch.zeros_like(val["c"])]
    for _ in range(case["steps"]):
        vs.append(tree.solve(val["c"] * vs[-1] + val["i"]))
    traces = torch.stack([v[roots] for v in vs[1:]])
    lam = torch.zeros_like(val["c"])
    ga, gc, gi = torch.zeros_like(lam), torch.zeros_like(lam), torch.zeros_like(lam)
    for k in range(case["steps"], 0, -1):
        mu = val["c"] * lam
        mu[roots] += 2.0 * (traces[k - 1] - val["target"])
        lam = tree.solve(mu)
        gi += lam
        gc += lam * (vs[k - 1] - vs[k])
        ga -= torch.where(tree.root, torch.zeros_like(lam), (lam - lam[p]) * (vs[k] - vs[k][p]))
    return dict(traces=traces, grad_a=ga, grad_c=gc, grad_i=gi)
