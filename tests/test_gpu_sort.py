"""The sorted order itself: particles by (system, Morton key, slot).

The tree's permutation against numpy's stable sort of the keys (formed here as
the build defines them), and for several systems each one's own solve.  Sizes
around the tiles (1,024) and merges (16 tiles, 256 tiles: three merges above
262,144), and around the change to the radix sort; keys equal across tiles and
runs."""
import numpy as np
import pytest

from conftest import gpu_available
from paper_1712_10116_amd import workloads as W

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]


def _keys(pos):
    lo, hi = pos.min(axis=1), pos.max(axis=1)
    side = (hi - lo).max() or 1.0
    q = np.clip(np.floor((pos - (0.5 * (lo + hi) - 0.5 * side)[:, None]) * (2097152.0 / side)),
                0, 2097151).astype(np.uint64)
    key = np.zeros(pos.shape[1], dtype=np.uint64)
    one = np.uint64(1)
    for b in range(21):
        for d in range(3):
            key |= ((q[d] >> np.uint64(b)) & one) << np.uint64(3 * b + 2 - d)
    return key


def _particles(n, kind, seed):
    pos, _, _ = W.plummer(n, seed=seed)
    if kind == "equal":  # a few hundred distinct positions, spread over the slots
        pos = pos[:, np.random.default_rng(seed).integers(0, max(1, min(n, 300)), n)]
    elif kind == "sorted":
        pos = pos[:, np.argsort(_keys(pos), kind="stable")]
    elif kind == "reversed":
        pos = pos[:, np.argsort(_keys(pos), kind="stable")[::-1]]
    return np.ascontiguousarray(pos)


@pytest.mark.parametrize("kind", ["random", "equal", "sorted", "reversed"])
@pytest.mark.parametrize("n", [1023, 1024, 1025, 2049, 16384, 16385, 262144, 262145, 393216, 393217,
                               524289])
def test_one_system(n, kind):
    import torch
    from paper_1712_10116_amd import fmm as F
    pos = _particles(n, kind, n % 89)
    # equal positions down to the deepest level make one leaf each
    s = F.Solver(n, p_max=1, leaf_size=64, kernel=0, precision=1)
    s.build(torch.from_numpy(pos).cuda(), eps=0.01, theta=0.9)
    perm = s.export_tree()["perm"]
    s.close()
    np.testing.assert_array_equal(perm, np.argsort(_keys(pos), kind="stable"))


@pytest.mark.parametrize("kind", ["random", "equal"])
@pytest.mark.parametrize("sizes", [[1000, 1100, 0, 1, 3000, 24, 1024, 17000, 5, 16400],
                                   [300, 263000, 700, 40], [524289, 3, 2000],
                                   [200000, 189824, 200000], [200000, 189825, 200000],
                                   [131072] * 6 + [131071, 1], [131072] * 6 + [131071, 2]])
def test_several_systems(sizes, kind):
    import torch
    from paper_1712_10116_amd import fmm as F
    prm = dict(eps=0.01, theta=0.9)
    none = torch.zeros(0, dtype=torch.int32, device="cuda")
    dev = []
    for k, n in enumerate(sizes):
        pos = _particles(max(n, 1), kind, 7 + k)
        m = np.random.default_rng(k).uniform(0.5, 1.0, max(n, 1))
        dev.append(dict(pos=torch.from_numpy(pos).cuda(), mass=torch.from_numpy(m).cuda(),
                        active=none if n == 0 else None))
    # FP64 sums in sorted order: another order of a system's particles would show
    s = F.Solver(sum(sizes), p_max=1, leaf_size=64, kernel=0, precision=0)
    out = [[x.clone() for x in o] for o in s.forces_batched(dev, p=1, **prm)]
    for d, n, o in zip(dev, sizes, out):
        if n:
            for a, b in zip(s.forces(d["pos"], d["mass"], p=1, **prm), o):
                assert torch.equal(a, b), n
    s.close()
