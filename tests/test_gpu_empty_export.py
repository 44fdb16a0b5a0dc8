"""Export of an empty system's tree: its root alone, whatever was built before."""
import pytest

from conftest import gpu_available
from paper_1712_10116_amd import workloads as W

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]


@pytest.mark.parametrize("small", [True, False])
def test_empty_tree(small):
    import torch
    from paper_1712_10116_amd import fmm as F
    pos = torch.from_numpy(W.plummer(3000, seed=8)[0]).cuda()
    s = F.Solver(3000, p_max=4, leaf_size=8, kernel=0, precision=0)
    s.set_small_path(small)
    s.build(pos, eps=0.01, theta=0.5)  # lists and cells that an empty tree must not show
    s.build(pos, torch.zeros(0, dtype=torch.int32, device="cuda"), eps=0.01, theta=0.5)
    info, ex = s.tree_info(), s.export_tree()
    s.close()
    assert (info["n"], info["nodes"], info["m2l"], info["p2p"]) == (0, 1, 0, 1)
    assert ex["perm"].size == 0 and ex["m2l"].size == 0 and ex["p2p"].tolist() == [[0, 0]]
    assert (ex["level"][0], ex["prefix"][0], ex["begin"][0], ex["end"][0]) == (0, 0, 0, 0)
    assert ex["is_leaf"][0] == 1 and ex["half"][0] == 0.5
