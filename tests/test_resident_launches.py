"""Launches of the LDS-resident plan: classes with few groups share one, but only
where every image fits the LDS that the launch reserves.  The blob's share of a
class is not monotone (3,584 bytes in class 7, 3,328 in the larger class 6), so
cells of short branches in class 7 cannot run with cells of class 6."""
import numpy as np
import pytest

import oracle
from workloads import Forest, cable_values, grow_random_forest

CLASS_BYTES = (163840, 81920, 54528, 40960, 32768, 27136, 23296, 20480, 16384, 10240)
STRIDES = (6144, 3008, 1984, 1472, 1152, 960, 832, 704, 576, 320)


def network(*kinds):
    """(cells, compartments of each, mean branch length) one after the other."""
    rng = np.random.default_rng(5)
    par, coff, boff = [], [0], [0]
    for count, size, mean in kinds:
        f = grow_random_forest(rng, count, target_size=np.full(count, size), mean_len=mean)
        lo = coff[-1]
        par.append(np.where(f.parent >= 0, f.parent + lo, -1))
        coff += list(f.cell_offsets[1:] + lo)
        boff += list(f.branch_offsets[1:] + lo)
    return Forest(np.concatenate(par).astype(np.int32), np.array(coff, np.int64), np.array(boff, np.int64))


SHORT, LONG, MEDIUM, LARGE = (8, 680, 4.8), (8, 660, 6.0), (3, 780, 12.0), (1, 5000, 12.0)
# kinds, launches: class 7 too large beside class 6; class 7 that fits there; a
# still larger class takes both
CASES = [((SHORT, MEDIUM), 2), ((LONG, MEDIUM), 1), ((SHORT, MEDIUM, LARGE), 1), ((SHORT,), 1)]


@pytest.mark.parametrize("kinds,launches", CASES)
def test_classes_share_a_launch_that_holds_them(kinds, launches):
    from paper_1810_12742_amd import Plan
    f = network(*kinds)
    p = Plan(f.parent, f.cell_offsets, host_only=True, resident=True, res_pack=100)
    g = p.table("res_groups").reshape(-1, 16)
    classes, blob = g[:, 13], g[:, 7]
    p_launches = p.info["nclasses"]
    p.close()
    small = g[classes == 7]
    fit = np.all(24 * STRIDES[6] + 16 * small[:, 7] <= CLASS_BYTES[6])
    assert set(classes[:8]) == {7} and fit == (kinds[0] is LONG)
    assert p_launches == launches
    # some way to launch every group inside its LDS with that many launches exists
    used = sorted(set(classes))[:launches]
    assert all(any(s + 1 <= STRIDES[k] and 24 * STRIDES[k] + 16 * b <= CLASS_BYTES[k] for k in used)
               for s, b in zip(g[:, 2], blob))


@pytest.mark.gpu
@pytest.mark.parametrize("kinds,launches", CASES)
def test_solves(kinds, launches):
    import torch
    from paper_1810_12742_amd import Plan
    f = network(*kinds)
    s = cable_values(f, np.random.default_rng(62), a_kind="cable", dt=0.025)
    p = Plan(f.parent, f.cell_offsets, resident=True, res_pack=100)
    assert p.info["kernel"] == 4 and p.info["nclasses"] == launches
    d, u, b = (torch.from_numpy(a).cuda() for a in (s.diag, s.upper, s.rhs))
    x = p.solve(d, u, b).cpu().numpy()
    xo = oracle.solve(f, s.diag, s.upper, s.rhs)
    err = np.maximum.reduceat(np.abs(x - xo), f.cell_offsets[:-1])
    assert np.max(err / np.maximum.reduceat(np.abs(xo), f.cell_offsets[:-1])) <= 1e-12
    p.close()
