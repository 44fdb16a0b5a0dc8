"""One-workgroup build of small batches.

* More systems than the context has cells (most of them empty): no cell is
  written past the workspace, which then grows, whether a system is split (leaf
  4) or none can be (leaf 128), with build and evaluation in two calls and in
  one.  Against the oracle with the parity bound (1e-12).
* Up to 1,024 particles in several systems, some empty, with coincident
  particles and particles on cell faces: cells, lists and values equal those of
  the multi-workgroup build bit for bit, system by system and together.
* Leaves larger than the build's level search holds (1,024 particles): taken too,
  since a batch of that few particles is not split then.
* Batches in which no system is split, queued in one call: as build and evaluation
  in two, bit for bit, and a system without masses left alone."""
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


def _lattice(n, seed):
    """Particles on the faces of their box's cells, in random order."""
    g = np.random.default_rng(seed)
    return g.integers(0, 17, (3, n)) / 16.0, g.uniform(0.5, 1.0, n)


def _same(n, seed):
    """Most of the particles at one point."""
    pos, _, m = W.plummer(n, seed=seed)
    pos[:, : 2 * n // 3] = pos[:, :1]
    return pos, m


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("leaf", [1, 7, 64])
@pytest.mark.parametrize("sizes", [[1024], [1023, 0, 1], [0, 300, 0, 0, 1, 2, 400, 63, 64, 65, 0],
                                   [0, 0, 5], [64] * 16])
def test_equals_general_build(sizes, leaf, precision):
    import torch
    from paper_1712_10116_amd import fmm as F
    prm = dict(eps=0.01, theta=0.5)
    host, dev = _systems(sizes, 900)
    for k, n in enumerate(sizes):
        if n >= 64:
            pos, m = (_lattice, _same)[k % 2](n, 40 + k) if k % 3 else host[k]
            dev[k].update(pos=torch.from_numpy(pos).cuda(), mass=torch.from_numpy(m).cuda())
    res = []
    for small in (True, False):
        s = F.Solver(1024, p_max=4, leaf_size=leaf, kernel=0, precision=precision)
        s.set_small_path(small)
        s.profile(True)
        s.build_batched(dev, **prm)
        calls = {k: c for k, (_, c) in s.profile_read().items()}
        assert (calls["sort"] == 0) == small  # the one-workgroup build has no sort of its own
        info = s.tree_info()
        out = [x.cpu().numpy() for o in s.evaluate_batched(dev, p=4) for x in o]
        trees = []
        for d, n in zip(dev, sizes):
            if n:
                s.build(d["pos"], **prm)
                trees.append(s.export_tree())
        res.append((info, out, trees))
        s.close()
    (i1, o1, t1), (i2, o2, t2) = res
    assert i1 == i2
    for a, b in zip(o1, o2):
        np.testing.assert_array_equal(a, b)
    for a, b in zip(t1, t2):
        for key in a:
            np.testing.assert_array_equal(a[key], b[key], err_msg=key)


@pytest.mark.parametrize("leaf", [1024, 1025, 4096])
@pytest.mark.parametrize("n", [1, 900, 1024])
def test_leaves_beyond_the_level_search(oracle, n, leaf):
    import torch
    from paper_1712_10116_amd import fmm as F
    prm = dict(eps=0.01, theta=0.5, p=4)
    pos, _, m = W.plummer(n, seed=33)
    s = F.Solver(n, p_max=4, leaf_size=leaf, kernel=1, precision=0)
    tp, tm = torch.from_numpy(pos).cuda(), torch.from_numpy(m).cuda()
    s.profile(True)
    a, pt = (x.cpu().numpy() for x in s.forces(tp, tm, **prm))
    assert s.profile_read()["sort"][1] == 0  # built by one workgroup
    assert s.tree_info()["nodes"] == 1
    s.close()
    ra, rp = oracle.fmm(pos, m, leaf_size=leaf, kernel=1, **prm)
    assert np.abs(a - ra).max() <= 1e-12 * np.abs(ra).max()
    assert np.abs(pt - rp).max() <= 1e-12 * np.abs(rp).max()


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("sizes", [[1], [64], [0, 5, 0, 64, 63], [64] * 16, [7, 64, 0, 33] * 75])
def test_systems_of_one_cell(sizes, precision):
    import torch
    from paper_1712_10116_amd import fmm as F
    prm = dict(eps=0.01, theta=0.5, p=5)
    _, dev = _systems(sizes, 1300)
    s = F.Solver(sum(sizes), p_max=5, leaf_size=64, kernel=0, precision=precision)
    ref = [[x.clone() for x in o] for o in _forces(F, s, dev, False, **prm)]
    for _ in range(2):
        for got, want in zip(_forces(F, s, dev, True, **prm), ref):
            assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1])
    reqs, out = s._requests(dev, True)
    last = len(sizes) - 1
    for x in out[last]:
        x.fill_(7.0)
    reqs[last].mass = None
    s._raise(F.lib().fmm_forces_batched(s._h, len(dev), reqs, prm["eps"], prm["theta"], prm["p"]))
    for k, (got, want) in enumerate(zip(out, ref)):
        for x, y in zip(got, want):
            assert bool((x == 7.0).all()) if k == last else torch.equal(x, y)
    s.close()
