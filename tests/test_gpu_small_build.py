"""One-workgroup build of small batches.

* More systems than the context has cells (most of them empty): no cell is
  written past the workspace, which then grows, whether a system is split (leaf
  4) or none can be (leaf 128), with build and evaluation in two calls and in
  one.  Against the oracle with the parity bound (1e-12)."""
import numpy as np
import pytest

from conftest import gpu_available
from paper_1712_10116_amd import workloads as W

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]


def _systems(sizes, seed):
    """Particles of each system, and the dicts of device tensors that a solver takes."""
    import torch
    none = torch.zeros(0, dtype=torch.int32, device="cuda")
    one = torch.zeros(3, 1, dtype=torch.float64, device="cuda")
    host, dev = [], []
    for k, n in enumerate(sizes):
        if n == 0:
            host.append(None)
            dev.append(dict(pos=one, mass=one[0], active=none))
            continue
        pos, _, m = W.plummer(n, seed=seed + k)
        host.append((pos, m))
        dev.append(dict(pos=torch.from_numpy(pos).cuda(), mass=torch.from_numpy(m).cuda(),
                        active=None))
    return host, dev


def _forces(F, s, dev, one_call, **prm):
    if not one_call:
        return s.forces_batched(dev, **prm)
    reqs, out = s._requests(dev, True)
    s._raise(F.lib().fmm_forces_batched(s._h, len(dev), reqs, prm["eps"], prm["theta"], prm["p"]))
    return out


@pytest.mark.parametrize("one_call", [False, True])
@pytest.mark.parametrize("leaf,each", [(128, 1), (4, 9)])
def test_more_systems_than_cells(oracle, leaf, each, one_call):
    from paper_1712_10116_amd import fmm as F
    sizes = [0] * 3000
    sizes[2::75] = [each + k % 3 for k in range(40)]
    total = sum(sizes)
    assert len(sizes) > 8 * total // leaf + 1024 and (total <= leaf) == (leaf == 128)
    prm = dict(eps=0.01, theta=0.5, p=4)
    host, dev = _systems(sizes, 500)
    s = F.Solver(total, p_max=4, leaf_size=leaf, kernel=1, precision=0)
    for _ in range(2):  # the second on the workspace that the first grew
        out = _forces(F, s, dev, one_call, **prm)
        assert s.tree_info()["nodes"] >= len(sizes)
        for k in range(2, len(sizes), 75):
            ra, rp = oracle.fmm(*host[k], leaf_size=leaf, kernel=1, **prm)
            a, pt = (x.cpu().numpy() for x in out[k])
            assert np.abs(a - ra).max() <= 1e-12 * np.abs(ra).max()
            assert np.abs(pt - rp).max() <= 1e-12 * np.abs(rp).max()
    s.close()
