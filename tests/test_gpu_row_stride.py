"""FP64 far field of degrees 5 and 6 in contexts of a larger maximum degree.

The M2L reads its source rows in 16-byte units, so rows have to start on 16
bytes at every maximum degree (at 8 a row holds an odd number of values).
Against the oracle with the FP64 parity bound (1e-12 of a particle's field,
floor 1e-6 of the rms), forces and vector-source field."""
import numpy as np
import pytest

from conftest import gpu_available
from paper_1712_10116_amd import workloads as W

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]


def _off(a, ra):
    a, ra = np.atleast_2d(a), np.atleast_2d(ra)
    mag = np.sqrt((ra * ra).sum(0))
    return (np.sqrt(((a - ra) ** 2).sum(0))
            / np.maximum(mag, 1e-6 * np.sqrt((mag * mag).mean()))).max()


@pytest.mark.parametrize("kernel", [0, 1])
@pytest.mark.parametrize("p", [5, 6])
@pytest.mark.parametrize("p_max", [7, 8])
def test_rows_of_larger_maximum_degree(oracle, p_max, p, kernel):
    import torch
    from paper_1712_10116_amd import fmm as F
    n, leaf, prm = 3001, 8, dict(theta=0.5, eps=0.01)
    pos, _, m = W.plummer(n, seed=83)
    t = oracle.Tree(pos, p=p, leaf_size=leaf, kernel=kernel, **prm)
    s = F.Solver(n, p_max=p_max, leaf_size=leaf, kernel=kernel, precision=0)
    tp, tm = torch.from_numpy(pos).cuda(), torch.from_numpy(m).cuda()
    a, pot = s.forces(tp, tm, p=p, **prm)
    u, phi = s.evaluate_dipole(tp, tm, a, p=p)
    ru, rphi = t.evaluate_dipole(m, a.cpu().numpy())
    ra, rp = t.evaluate(m)
    for got, ref in ((a, ra), (pot, rp), (u, ru)):
        assert _off(got.cpu().numpy(), ref) < 1e-12
    assert np.abs(phi.cpu().numpy() - rphi).max() / np.sqrt((rphi ** 2).mean()) < 1e-12
    s.close()
