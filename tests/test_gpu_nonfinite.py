"""Positions that are not finite: FMM_ENONFINITE, outputs left alone, and the
context usable, on every route of a solve (one-workgroup build, small tree queued
to the end, tree size read first, predicted depth, several systems)."""
import numpy as np
import pytest

from conftest import gpu_available
from paper_1712_10116_amd import workloads as W

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]


@pytest.mark.parametrize("bad", [float("nan"), float("inf"), float("-inf")])
@pytest.mark.parametrize("n,predict,others", [(900, False, 0), (5000, False, 0), (30000, False, 0),
                                              (30000, True, 0), (200, False, 2), (200, False, 20)])
def test_outputs_are_left_alone(n, predict, others, bad):
    import torch
    from paper_1712_10116_amd import fmm as F
    pos, _, m = W.plummer(n, seed=23)
    small, _, ms = W.plummer(40, seed=24)
    prm = dict(eps=0.01, theta=0.5, p=4)
    s = F.Solver(n + 40 * others, p_max=4, leaf_size=16, kernel=0, precision=0)
    s.set_level_prediction(predict)
    tp, tm = torch.from_numpy(pos).cuda(), torch.from_numpy(m).cuda()
    acc = torch.empty(3, n, dtype=torch.float64, device="cuda")
    pot = torch.empty(n, dtype=torch.float64, device="cuda")
    systems = [dict(pos=tp, mass=tm, acc=acc, pot=pot)]
    systems += [dict(pos=torch.from_numpy(small).cuda(), mass=torch.from_numpy(ms).cuda())] * others

    def solve():
        acc.fill_(7.0)
        pot.fill_(7.0)
        reqs, _ = s._requests(systems, True)
        s._raise(F.lib().fmm_forces_batched(s._h, len(systems), reqs, prm["eps"], prm["theta"],
                                            prm["p"]))
        return acc.clone(), pot.clone()

    good = solve()
    good = solve()
    for at in (0, n // 2, n - 1):
        old = float(tp[1, at])
        tp[1, at] = bad
        with pytest.raises(F.FMMError) as ei:
            solve()
        assert ei.value.status == F.FMM_ENONFINITE
        torch.cuda.synchronize()
        assert bool((acc == 7.0).all()) and bool((pot == 7.0).all())
        tp[1, at] = old
        again = solve()
        assert torch.equal(good[0], again[0]) and torch.equal(good[1], again[1])
    s.close()
