"""Near lists of every leaf in a system, cut into a bounded number of shares.

A softening length beyond the size of the system makes every pair near, so that every
leaf lists all leaves and would be cut into more shares than a list may have:
twice and four times the windows a share (32,768 and 131,072 particles, leaf
64), and whole chunks of the list (9,000 in leaves of 1).  With every pair near,
the direct sum is the reference: accelerations and potentials of random sinks
with the parity bounds (FP64 1e-12, mixed 2e-6 rms), their gradient with its own
(1e-10 of a tensor's size, 1e-5 rms), and the context's memory with its bound.

Small leaves: shares of whole chunks of the list, on both sides of the sizes where
a share's length changes, random sinks and the sparsest leaf's against the oracle
with the same bounds."""
import numpy as np
import pytest

from conftest import gpu_available
from paper_1712_10116_amd import workloads as W

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("n,leaf", [(32768, 64), (131072, 64), (9000, 1)])
def test_wide_softening(n, leaf, precision):
    import torch
    from paper_1712_10116_amd import fmm as F
    pos, _, m = W.uniform_sphere(n, seed=17)
    prm = dict(theta=0.5, eps=3.0)
    sinks = np.sort(np.random.default_rng(4).choice(n, 60, replace=False))
    # softened pair sums; the own pair (d = 0) adds to the potential only in the
    # sum below, and to the gradient's diagonal
    d = pos[:, sinks, None] - pos[:, None, :]
    s2 = (d * d).sum(0) + prm["eps"] ** 2
    w1, w3, w5 = m * s2 ** -0.5, m * s2 ** -1.5, 3.0 * m * s2 ** -2.5
    ra = -(w3 * d).sum(2)
    rp = m[sinks] / prm["eps"] - w1.sum(1)
    rg = np.stack([(w5 * d[i] * d[j] - (i == j) * w3).sum(1)
                   for i, j in ((0, 0), (1, 1), (2, 2), (0, 1), (0, 2), (1, 2))])
    rg[:3] += m[sinks] / prm["eps"] ** 3
    tp, tm = torch.from_numpy(pos).cuda(), torch.from_numpy(m).cuda()
    torch.cuda.synchronize()
    free = torch.cuda.mem_get_info()[0]
    s = F.Solver(n, p_max=4, leaf_size=leaf, kernel=1, precision=precision)
    base = free - torch.cuda.mem_get_info()[0]
    a, pt = s.forces(tp, tm, p=4, **prm)
    torch.cuda.synchronize()
    grown = free - torch.cuda.mem_get_info()[0] - base
    info = s.tree_info()
    leaves = info["leaves"]
    assert info["p2p_directed"] == leaves ** 2
    # a quarter of room on 32 bytes a row and item, 4 bytes a list entry; 64 MB of
    # torch's own
    rows, items = 127 * n, 128 * (leaves + n // 64)
    assert grown <= 1.25 * (32 * (rows + items) + 4 * leaves ** 2) + (64 << 20), grown
    a, pt = a.cpu().numpy()[:, sinks], pt.cpu().numpy()[sinks]
    mag = np.sqrt((ra * ra).sum(0))
    e = np.sqrt(((a - ra) ** 2).sum(0)) / np.maximum(mag, 1e-6 * np.sqrt((mag * mag).mean()))
    ep = np.abs(pt - rp) / np.abs(rp)
    if precision == 0:
        assert e.max() < 1e-12 and ep.max() < 1e-12, (e.max(), ep.max())
    else:
        assert np.sqrt((e * e).mean()) < 2e-6 and np.sqrt((ep * ep).mean()) < 2e-6
    a2, _, g = s.forces_grad(tp, tm, p=4, **prm)
    assert np.array_equal(a2.cpu().numpy()[:, sinks], a)
    eg = np.sqrt(((g.cpu().numpy()[:, sinks] - rg) ** 2).sum(0)) / np.sqrt((rg * rg).sum(0))
    if precision == 0:
        assert eg.max() < 1e-10, eg.max()
    else:
        assert np.sqrt((eg * eg).mean()) < 1e-5
    s.close()


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("n,leaf", [(1025, 1), (9001, 3), (32768, 5), (32769, 5), (140000, 15),
                                    (140000, 17)])
def test_small_leaves(oracle, n, leaf, precision):
    import torch
    from paper_1712_10116_amd import fmm as F
    pos, _, m = W.plummer(n, seed=29)
    prm = dict(theta=0.5, eps=0.01)
    t = oracle.Tree(pos, p=4, leaf_size=leaf, kernel=0, **prm)
    ref = t.export()
    far = int(np.argmax((pos ** 2).sum(0)))
    sinks = np.unique(np.append(np.random.default_rng(6).choice(n, 80, replace=False), far))
    ra, rp = t.evaluate_sinks(m, sinks)[:2]
    s = F.Solver(n, p_max=4, leaf_size=leaf, kernel=0, precision=precision)
    a, pt = (x.cpu().numpy() for x in s.forces(*(torch.from_numpy(x).cuda() for x in (pos, m)),
                                               p=4, **prm))
    assert s.tree_info()["leaves"] == int((ref["is_leaf"] != 0).sum())
    s.close()
    a, pt = a[:, sinks], pt[sinks]
    mag = np.sqrt((ra * ra).sum(0))
    e = np.sqrt(((a - ra) ** 2).sum(0)) / np.maximum(mag, 1e-6 * np.sqrt((mag * mag).mean()))
    ep = np.abs(pt - rp) / np.abs(rp)
    if precision == 0:
        assert e.max() < 1e-12 and ep.max() < 1e-12, (e.max(), ep.max())
    else:
        assert np.sqrt((e * e).mean()) < 2e-6 and np.sqrt((ep * ep).mean()) < 2e-6
