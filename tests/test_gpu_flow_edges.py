"""The scheduled groups at the edges of their staging, against the FP64 oracle (1e-12
per cell, the bound of every FP64 solve here).  A thread stages batches of four
elements, six in flight with a given right-hand side and four with a formed one, then
the rest in a loop; a group has one, two or four waves.  So a batch ends at 256, 512
or 1,024 compartments, and the loop begins at 1,536 or 1,024 (one wave) and at 4,096
(four waves, formed); two waves never hold enough for it."""
import numpy as np
import pytest

import oracle
from workloads import cable_values, grow_random_forest

pytestmark = pytest.mark.gpu


# every cell a group of its own: up to 512 groups run on four waves each, up to 1,023
# (three or four to a compute unit) on two, from 1,024 on one
@pytest.mark.parametrize("waves,sizes", [
    (4, [1, 4, 255, 256, 257, 1023, 1024, 1025, 2047, 2048, 2049, 3071, 3072, 3073, 4095, 4096, 4097]),
    (2, [1, 127, 128, 129, 511, 512, 513, 1023, 1024, 1025, 1535, 1536, 1537] * 50),
    (1, [1, 63, 64, 65, 255, 256, 257, 1023, 1024, 1025, 1535, 1536, 1537, 2559, 2560, 2561] * 70)])
def test_batch_edges(waves, sizes):
    import torch
    from paper_1810_12742_amd import Plan
    assert {4: len(sizes) <= 512, 2: 512 < len(sizes) < 1024, 1: len(sizes) >= 1024}[waves]
    f = grow_random_forest(np.random.default_rng(111), len(sizes), target_size=np.array(sizes))
    s = cable_values(f, np.random.default_rng(112), a_kind="cable", dt=0.025)
    p = Plan(f.parent, f.cell_offsets, max_group_unknowns=1)
    assert p.info["kernel"] == 1 and p.info["ngroups"] == len(sizes)
    d, u, b, c = (torch.from_numpy(a).cuda() for a in (s.diag, s.upper, s.rhs, s.c))
    I = 0.1 * np.random.default_rng(113).standard_normal(f.n)
    i = torch.from_numpy(I).cuda()
    noise = oracle.noise(3, 7, np.arange(f.n, dtype=np.int64), 0.1)
    d32, u32 = s.diag.astype(np.float32), s.upper.astype(np.float32)
    for got, diag, upper, rhs in (
            (p.solve(d, u, b), s.diag, s.upper, s.rhs), (p.timestep(d, u, c, b), s.diag, s.upper, s.c * s.rhs),
            (p.timestep(d, u, c, b, i_inj=i), s.diag, s.upper, s.c * s.rhs + I),
            (p.timestep(d, u, c, b, noise_sigma=0.1, noise_seed=3, step=7), s.diag, s.upper, s.c * s.rhs + noise),
            (p.solve_mixed(d.float(), u.float(), b, sweeps=1), d32.astype(float), u32.astype(float), s.rhs)):
        xo = oracle.solve(f, diag, upper, rhs)
        err = np.maximum.reduceat(np.abs(got.cpu().numpy() - xo), f.cell_offsets[:-1])
        assert np.max(err / np.maximum.reduceat(np.abs(xo), f.cell_offsets[:-1])) <= 1e-12
    p.close()
