"""Leaf multipoles of deep trees (a wavefront per leaf, fuller leaves by the
whole block) against the oracle: leaf populations around 16 atoms a pass, the
64 atoms of a wavefront and the 256 threads of a block."""
import numpy as np
import pytest

from gpu_util import assert_within, errors, reference, run

pytestmark = pytest.mark.gpu

COUNTS = [[1, 2, 3, 4, 15, 16, 17], [31, 32, 33, 47, 48, 49, 63], [64, 65, 64, 64, 128, 63, 1, 65],
          [255, 256, 257, 300, 64, 1]]


@pytest.mark.parametrize("prec,order", [("fp64", 12), ("f32", 6), ("f32", 10), ("bf16x3", 8), ("fp64", 15)])
@pytest.mark.parametrize("periodic", [True, False])
@pytest.mark.parametrize("counts", COUNTS)
def test_deep_tree_leaves_against_oracle(counts, periodic, prec, order):
    rng = np.random.default_rng(21)
    h = 0.25
    cells = rng.permutation(32 ** 3)[:max(4 * len(counts), 900 // sum(counts))]
    x = np.concatenate([(np.array(np.unravel_index(c, (32, 32, 32))) + rng.uniform(0.02, 0.98, (counts[k % len(counts)], 3))) * h
                        for k, c in enumerate(cells)])
    if not periodic:  # the cube of the extent: keep the leaves where they are
        x[0], x[1] = [1e-3 * h] * 3, [(32 - 1e-3) * h] * 3
    p = rng.permutation(x.shape[0])  # caller order is not leaf order
    x = x[p].astype(np.float32).astype(np.float64)
    n = x.shape[0]
    q = rng.uniform(-1, 1, n).astype(np.float32).astype(np.float64)
    d = {"x": x, "qA": q, "qB": (0.5 * q).astype(np.float32).astype(np.float64),
         "site": np.where(np.arange(n) % 7 == 0, np.arange(n) % 3, -1).astype(np.int32),
         "lam": np.array([0.2, 0.5, 0.9]), "box": [32 * h] * 3, "periodic": periodic, "depth": 5, "order": order}
    assert_within(errors(run(d, prec), reference(d)), order, label="%s %s %s" % (counts, periodic, prec))
