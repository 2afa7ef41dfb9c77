"""fmm_eval_adjoint_full with weights on a few atoms: leaves whose neighbourhood
has a weight take both sources' pair terms, the others the charges' alone."""
import numpy as np
import pytest

from paper_2410_01626_amd import workloads as W
from test_gpu_adjoint_full import _compare, _oracle, _run, _tol

pytestmark = pytest.mark.gpu


def _sparse(d, keep, which, seed):
    rng = np.random.default_rng(seed)
    n = d["x"].shape[0]
    gphi, gF = np.zeros(n), np.zeros((n, 3))
    at = rng.choice(n, keep, replace=False)
    if which != "F":
        gphi[at] = rng.standard_normal(keep).astype(np.float32)
    if which != "phi":
        gF[at, rng.integers(0, 3, keep)] = rng.standard_normal(keep).astype(np.float32)
    return gphi, gF


@pytest.mark.parametrize("prec", ["fp64", "f32", "bf16x3"])
@pytest.mark.parametrize("periodic,depth", [(True, 3), (False, 3), (True, 2)])
@pytest.mark.parametrize("keep,which", [(1, "F"), (1, "phi"), (6, "both")])
def test_few_weights_match_oracle(keep, which, periodic, depth, prec):
    d = (W.tiny_periodic(51, n=900, edge=2.0, n_sites=3, depth=depth, order=8) if periodic else
         W.random_open(52, n=900, edge=2.0, n_sites=3, depth=depth, order=8))
    gphi, gF = _sparse(d, keep, which, 7)
    res = _run(d, prec, 0.5, gphi, gF)
    _compare(res, _oracle(d, 0.5, gphi, gF), _tol(8), label="%s %s" % (which, prec))


@pytest.mark.parametrize("n", [300, 3000])
def test_few_weights_without_far_field(n):
    """Open, depth 1 (the pair sum alone; 3,000 atoms pass the source tile in
    several passes): the gradients of a full set of weights are the sum of those
    of its parts, of which one has a single weighted atom and one none."""
    d = W.random_open(53, n=n, edge=2.5, n_sites=3, depth=1, order=4)
    rng = np.random.default_rng(8)
    gphi, gF = rng.standard_normal(n), rng.standard_normal((n, 3))
    one = np.zeros(n)
    one[n // 2] = 1.0
    whole = _run(d, "fp64", 1.0, gphi, gF)
    parts = [_run(d, "fp64", 0.0, gphi * one, gF * one[:, None]),
             _run(d, "fp64", 0.0, gphi * (1 - one), gF * (1 - one)[:, None]),
             _run(d, "fp64", 1.0, np.zeros(n), np.zeros((n, 3)))]
    for k in ("grad_x", "grad_qA", "grad_qB", "grad_lambda"):
        # sums of at most 8 n terms each
        size = sum(np.abs(p[k]).max() for p in parts)
        assert np.abs(sum(p[k] for p in parts) - whole[k]).max() <= 8 * n * 2.0 ** -52 * size, k
