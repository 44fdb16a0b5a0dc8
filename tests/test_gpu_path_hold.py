"""A system whose open lists are too long for the walk's path form.

A wide softening leaves every pair of cells open; with a tight clump in it the
sphere's 1,700 cells of one level are all on the open lists of the clump's cells.
The first solve finds out, the next ones do not try again: one sort and one walk
each, and smaller systems are not affected.  Values against build and
evaluation on a fresh context, bit for bit (the walk's forms give the same lists
in the same order)."""
import numpy as np
import pytest

from conftest import gpu_available
from paper_1712_10116_amd import workloads as W

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]


def _clump(n, seed):
    pos, _, m = W.uniform_sphere(n, seed=seed)
    pos[:, -150:] = 0.2 + 1e-3 * pos[:, -150:]
    return pos, m


def _calls(s, call):
    s.profile(True)
    out = call()
    prof = s.profile_read()
    s.profile(False)
    return out, {k: c for k, (_, c) in prof.items() if k in ("sort", "walk")}


@pytest.mark.parametrize("predict", [False, True])
@pytest.mark.parametrize("n", [6390, 9000])  # queued to the end (400 leaves), and read first
def test_failed_path_walk_is_not_repeated(oracle, n, predict):
    import torch
    from paper_1712_10116_amd import fmm as F
    prm = dict(eps=3.0, theta=0.5)
    pos, m = _clump(n, 71)
    kw = dict(p_max=4, leaf_size=16, kernel=0, precision=0)
    ex = oracle.Tree(pos, p=4, leaf_size=16, kernel=0, **prm).export()
    leaf, lev = ex["is_leaf"] != 0, ex["level"]
    deep = lev[~leaf].max()  # open there: cells of the level, and leaves above
    assert (lev == deep).sum() + (leaf & (lev < deep)).sum() > 1024 >= (~leaf).sum()
    dev = [torch.from_numpy(x).cuda() for x in (pos, m)]
    f = F.Solver(n, **kw)
    f.build(dev[0], **prm)
    ra, rp = f.evaluate(*dev, p=4)
    f.close()
    s = F.Solver(n, **kw)
    s.set_level_prediction(predict)
    for k in range(4):
        (a, pt), calls = _calls(s, lambda: s.forces(*dev, p=4, **prm))
        assert torch.equal(a, ra) and torch.equal(pt, rp)
        if k >= (2 if predict else 1):  # a predicted sequence needs a first depth
            assert calls == {"sort": 1, "walk": 1}, (k, calls)
    small, _, ms = W.plummer(3000, seed=72)
    tp, tm = torch.from_numpy(small).cuda(), torch.from_numpy(ms).cuda()
    _, calls = _calls(s, lambda: s.forces(tp, tm, p=4, eps=0.01, theta=0.5))
    assert calls == {"sort": 1, "walk": 1}
    for _ in range(40):  # past the hold, when the path form is tried again
        a, pt = s.forces(*dev, p=4, **prm)
    assert torch.equal(a, ra) and torch.equal(pt, rp)
    s.close()
