"""Lists of around 2^31 entries: leaves of one particle that all list each other
(a softening beyond the size of the system).  Below the limit of the lists' int32
offsets the solve equals the direct sum (mixed, 2e-6 rms); above it the call
reports FMM_EOVERFLOW, and the context goes on to solve what does fit."""
import numpy as np
import pytest

from conftest import gpu_available
from paper_1712_10116_amd import workloads as W

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]


def test_lists_around_2_31_entries():
    import torch
    from paper_1712_10116_amd import fmm as F
    pos, _, m = W.uniform_sphere(47000, seed=19)
    prm = dict(theta=0.5, eps=3.0, p=1)
    s = F.Solver(47000, p_max=1, leaf_size=1, kernel=1, precision=1)
    tp, tm = torch.from_numpy(pos).cuda(), torch.from_numpy(m).cuda()
    with pytest.raises(F.FMMError) as ei:
        s.forces(tp, tm, **prm)
    assert ei.value.status == F.FMM_EOVERFLOW
    n = 45000
    tp, tm = tp[:, :n].contiguous(), tm[:n].contiguous()
    a, pt = s.forces(tp, tm, **prm)
    info = s.tree_info()
    s.close()
    assert info["leaves"] == n and 2 ** 30 < info["p2p_directed"] == n * n < 2 ** 31
    assert info["p2p_interactions"] == n * (n - 1)
    sinks = np.arange(0, n, 450)
    d = pos[:, sinks, None] - pos[:, None, :n]
    s2 = (d * d).sum(0) + prm["eps"] ** 2
    ra = -(m[:n] * s2 ** -1.5 * d).sum(2)
    rp = m[sinks] / prm["eps"] - (m[:n] * s2 ** -0.5).sum(1)
    a, pt = a.cpu().numpy()[:, sinks], pt.cpu().numpy()[sinks]
    assert np.sqrt(((a - ra) ** 2).sum(0).mean() / (ra ** 2).sum(0).mean()) < 2e-6
    assert np.sqrt(((pt - rp) ** 2).mean() / (rp ** 2).mean()) < 2e-6
