"""Near-field launch shapes: what p2p_split asks for is what a plan has, the
automatic shapes, and FP64 leaves around the targets of a split block."""
import numpy as np
import pytest

from paper_2410_01626_amd import workloads as W
from tests.gpu_util import run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec,depth,n,blocks", [
    ("f32", 1, 2000, 1), ("f32", 1, 2100, 2), ("f32", 1, 4200, 4), ("fp64", 1, 320, 2), ("fp64", 1, 800, 4),
    ("fp64", 1, 2100, 2), ("fp64", 1, 4200, 4), ("f32", 3, 200000, 1), ("fp64", 3, 30000, 1)])
def test_blocks_per_leaf(prec, depth, n, blocks):
    import torch
    from paper_2410_01626_amd import fmm
    for split, want in ((0, blocks), (1, 1), (3, 3)):
        plan = fmm.Plan(depth, 4, periodic=True, precision=prec, max_atoms=n, p2p_split=split, p2p_waves=8,
                        device=torch.device("cuda:0"))
        assert plan.info()["p2p_split"] == want, split
        plan.close()


@pytest.mark.parametrize("prec", ["f32", "fp64"])
@pytest.mark.parametrize("n", [2300, 4500])
def test_one_block_on_request_gives_the_same_bits(prec, n):
    d = W.random_open(80 + n, n=n, edge=2.5, n_sites=3, depth=1, order=6)
    a, b = run(d, prec), run(d, prec, p2p_split=1)
    for k in ("F", "phi", "dVdl"):
        np.testing.assert_array_equal(a[k], b[k], err_msg=k)
    assert abs(a["E"] - b["E"]) <= n * 2.0 ** -53 * np.sum(np.abs(a["phi"]))


@pytest.mark.parametrize("depth,n", [(1, 200), (1, 260), (1, 330), (2, 1600), (2, 2600), (2, 3900), (2, 8100)])
def test_fp64_split_blocks(depth, n):
    """FP64, 8 wavefronts: 25 to 127 atoms a leaf on average take 1 to 4 blocks of
    32 targets, the last with the rest; the same pairs in another order, n sums
    of at most n terms each."""
    d = W.random_open(90 + n, n=n, edge=2.5, n_sites=3, depth=depth, order=6)
    a, b = run(d, "fp64", p2p_waves=8), run(d, "fp64", p2p_waves=8, p2p_split=1)
    for k in ("F", "phi", "dVdl"):
        assert np.abs(a[k] - b[k]).max() <= n * 2.0 ** -52 * np.abs(b[k]).max(), k
