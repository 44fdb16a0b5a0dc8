"""M2M and L2L where several levels of few cells share a workgroup.

Trees of more than 2048 cells, deep at the centre: runs of narrow levels at both
ends, launches of their own between them, and (p 1 to 6, both precisions) both
widths of the workgroup.  Against the oracle with the parity bounds (FP64 1e-12
of a particle's field, floor 1e-6 of the rms; mixed 2e-6 rms)."""
import numpy as np
import pytest

from conftest import gpu_available
from paper_1712_10116_amd import workloads as W

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("p,kernel", [(1, 0), (4, 0), (5, 1), (6, 0)])
def test_level_runs_match_oracle(oracle, p, kernel, precision):
    import torch
    from paper_1712_10116_amd import fmm as F
    n, leaf, prm = 16001, 8, dict(theta=0.6, eps=0.005)
    pos, _, m = W.plummer(n, seed=91)
    t = oracle.Tree(pos, p=p, leaf_size=leaf, kernel=kernel, **prm)
    assert t.n_nodes > 2048 and t.depth > 5
    ra, rp = t.evaluate(m)
    s = F.Solver(n, p_max=p, leaf_size=leaf, kernel=kernel, precision=precision)
    tp, tm = torch.from_numpy(pos).cuda(), torch.from_numpy(m).cuda()
    for _ in range(2):  # the second build sizes its launches from the first
        a, pot = (x.cpu().numpy() for x in s.forces(tp, tm, p=p, **prm))
        d, mag = np.sqrt(((a - ra) ** 2).sum(0)), np.sqrt((ra * ra).sum(0))
        if precision == 0:
            assert (d / np.maximum(mag, 1e-6 * np.sqrt((mag * mag).mean()))).max() < 1e-12
            assert (np.abs(pot - rp) / np.abs(rp)).max() < 1e-12
        else:
            assert np.sqrt((d * d).mean() / (mag * mag).mean()) < 2e-6
            assert np.sqrt(((pot - rp) ** 2).mean() / (rp * rp).mean()) < 2e-6
    s.close()
