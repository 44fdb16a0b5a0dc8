"""FP64 far field of degrees 5 and 6, whose M2L reads its source rows through LDS.

Lists of none, of less than one and of several wavefronts of sources; rows as
wide as the degree's and, with a larger maximum degree, wider.  Against the
oracle with the FP64 parity bound (1e-12 of a particle's field, floor 1e-6 of
the rms): the same sums in another order, some hundred terms of rounding
2^-53 each, are a tenth of it."""
import numpy as np
import pytest

from conftest import gpu_available
from paper_1712_10116_amd import workloads as W

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]


@pytest.mark.parametrize("kernel", [0, 1])
@pytest.mark.parametrize("p,p_max", [(5, 5), (5, 6), (6, 6)])
@pytest.mark.parametrize("n,leaf,theta", [(20, 16, 0.5), (700, 16, 0.6), (6001, 8, 0.35)])
def test_staged_far_field_matches_oracle(oracle, n, leaf, theta, p, p_max, kernel):
    import torch
    from paper_1712_10116_amd import fmm as F
    pos, _, m = W.plummer(n, seed=80 + n % 7)
    prm = dict(theta=theta, eps=0.01)
    t = oracle.Tree(pos, p=p, leaf_size=leaf, kernel=kernel, **prm)
    ra, rp = t.evaluate(m)
    s = F.Solver(n, p_max=p_max, leaf_size=leaf, kernel=kernel, precision=0)
    tp, tm = torch.from_numpy(pos).cuda(), torch.from_numpy(m).cuda()
    a, pot = s.forces(tp, tm, p=p, **prm)
    a, pot = a.cpu().numpy(), pot.cpu().numpy()
    s.close()
    mag = np.sqrt((ra * ra).sum(0))
    ea = np.sqrt(((a - ra) ** 2).sum(0)) / np.maximum(mag, 1e-6 * np.sqrt((mag * mag).mean()))
    ep = np.abs(pot - rp) / np.maximum(np.abs(rp), 1e-6 * np.sqrt((rp * rp).mean()))
    assert ea.max() < 1e-12 and ep.max() < 1e-12, (ea.max(), ep.max())
