"""Level prediction in a context that solves systems of different sizes.

* Solves of a few hundred particles between those of a large system (the rungs
  of an integrator) leave its predicted depth alone: one sort and one walk each.
* Systems of very different sizes in turn: the walk's form for the next one does
  not follow the last one's tree; values equal those of a fresh context.
* An empty system after a solve that failed reads its own header."""
import numpy as np
import pytest

from conftest import gpu_available
from paper_1712_10116_amd import workloads as W

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]


def test_small_solves_between_large_ones():
    import torch
    from paper_1712_10116_amd import fmm as F
    prm = dict(eps=0.01, theta=0.5, p=4)
    large, small = ([torch.from_numpy(x).cuda() for x in (s[0], s[2])]
                    for s in (W.plummer(30000, seed=61), W.uniform_sphere(500, seed=62)))
    s = F.Solver(30000, p_max=4, leaf_size=16, kernel=0, precision=0)
    s.set_level_prediction(True)
    s.forces(*large, **prm)
    ref = [x.clone() for x in s.forces(*large, **prm)]
    for _ in range(5):
        s.forces(*small, **prm)
    s.profile(True)
    out = s.forces(*large, **prm)
    prof = s.profile_read()
    assert (prof["sort"][1], prof["walk"][1]) == (1, 1)
    for a, b in zip(out, ref):
        assert torch.equal(a, b)
    s.close()


def test_sizes_in_turn():
    import torch
    from paper_1712_10116_amd import fmm as F
    prm = dict(eps=0.01, theta=0.5, p=4)
    kw = dict(p_max=4, leaf_size=16, kernel=0, precision=0)
    systems = [[torch.from_numpy(x).cuda() for x in (s[0], s[2])]
               for s in (W.plummer(7000, seed=63), W.plummer(400000, seed=64))]
    ref = []
    for pos, m in systems:
        f = F.Solver(m.numel(), **kw)
        f.build(pos, eps=0.01, theta=0.5)
        ref.append(f.evaluate(pos, m, p=4))
        torch.cuda.synchronize()
        f.close()
    s = F.Solver(400000, **kw)
    s.set_level_prediction(True)
    for k in (0, 0, 1, 1, 0, 1, 0):
        out = s.forces(*systems[k], **prm)
        for a, b in zip(out, ref[k]):
            assert torch.equal(a, b), k
    s.close()


def test_empty_system_after_a_failed_solve():
    import torch
    from paper_1712_10116_amd import fmm as F
    prm = dict(eps=0.01, theta=0.5, p=4)
    pos, m = (torch.from_numpy(x).cuda() for x in W.plummer(5000, seed=65)[::2])
    none = torch.zeros(0, dtype=torch.int32, device="cuda")
    bad = pos.clone()
    bad[2, 17] = float("nan")
    s = F.Solver(5000, p_max=4, leaf_size=16, kernel=0, precision=0)
    s.set_small_path(False)  # the predicted sequence for empty systems too
    s.set_level_prediction(True)
    s.forces(pos, m, **prm)
    s.forces(pos, m, none, **prm)
    with pytest.raises(F.FMMError):
        s.forces(bad, m, **prm)
    s.forces(pos, m, none, **prm)
    assert s.tree_info()["n"] == 0 and s.tree_info()["nodes"] == 1
    s.close()
