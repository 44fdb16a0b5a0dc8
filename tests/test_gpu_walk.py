"""Interaction lists of the walk's three forms against the oracle, bit-exact.

* path form (trees of at most 1600 split cells): a Plummer sphere whose sparse
  outer leaves descend through a large part of the tree (logged descents and,
  at leaf 4, more than the log holds), also through the single-workgroup build;
* an open list longer than the path form keeps (a softening length of half
  the system leaves every pair of cells unaccepted): walked by levels instead,
  with several blocks of candidates per group;
* level form, workgroup per group and wavefront per group (more than 1024
  groups in a level): small leaves of 60,000 particles."""
import numpy as np
import pytest

from conftest import gpu_available
from paper_1712_10116_amd import workloads as W

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]

CASES = {
    "path": (lambda: W.plummer(12000, seed=31)[0], 64, 0.5, 0.01),
    "path_small": (lambda: W.plummer(1000, seed=32)[0], 16, 0.5, 0.01),
    "path_long_descents": (lambda: W.plummer(5200, seed=33)[0], 8, 0.4, 0.01),
    "long_open_list": (lambda: W.uniform_sphere(6000, seed=34)[0], 4, 0.5, 1.0),
    "levels": (lambda: W.plummer(60000, seed=35)[0], 8, 0.5, 0.001),
}


@pytest.mark.parametrize("name", sorted(CASES))
def test_lists_bit_exact(oracle, name):
    import torch
    from paper_1712_10116_amd import fmm as F
    make, leaf, theta, eps = CASES[name]
    pos = make()
    t = oracle.Tree(pos, p=4, theta=theta, eps=eps, leaf_size=leaf, kernel=0)
    ref = t.export()
    split = int((ref["is_leaf"] == 0).sum())
    assert (split > 1600) == (name == "levels"), split
    s = F.Solver(pos.shape[1], p_max=4, leaf_size=leaf, kernel=0, precision=0)
    tp = torch.from_numpy(np.ascontiguousarray(pos)).cuda()
    for _ in range(2):  # the first build may regrow its list buffers
        s.build(tp, eps=eps, theta=theta)
        ex, info = s.export_tree(), s.tree_info()
        size = ref["end"] - ref["begin"]
        a, b = ref["p2p"][:, 0], ref["p2p"][:, 1]
        pairs = int((size[a] * size[b] * np.where(a == b, 1, 2)).sum()) - pos.shape[1]
        assert info["p2p_interactions"] == pairs
        for k in ("perm", "begin", "end", "m2l", "p2p"):
            np.testing.assert_array_equal(ex[k], ref[k], err_msg=k)
    s.close()


@pytest.mark.parametrize("n,leaf", [(900, 2), (1500, 4)])
def test_small_tree_that_outgrows_its_lists(oracle, n, leaf):
    """Solves queued without reading sizes back (one-workgroup build and small
    tree) whose lists do not fit at first: redone on regrown buffers, and right
    again when repeated."""
    import torch
    from paper_1712_10116_amd import fmm as F
    pos, _, m = W.uniform_sphere(n, seed=36)
    ra, rp = oracle.fmm(pos, m, p=4, theta=0.5, eps=1.0, leaf_size=leaf, kernel=0)
    s = F.Solver(n, p_max=4, leaf_size=leaf, kernel=0, precision=0)
    tp, tm = torch.from_numpy(pos).cuda(), torch.from_numpy(m).cuda()
    for _ in range(2):
        a, pt = s.forces(tp, tm, eps=1.0, theta=0.5, p=4)
        a, pt = a.cpu().numpy(), pt.cpu().numpy()
        mag = np.sqrt((ra * ra).sum(0))
        e = np.sqrt(((a - ra) ** 2).sum(0)) / np.maximum(mag, 1e-6 * np.sqrt((mag ** 2).mean()))
        assert e.max() < 1e-12 and (np.abs(pt - rp) / np.abs(rp)).max() < 1e-12
    s.close()
