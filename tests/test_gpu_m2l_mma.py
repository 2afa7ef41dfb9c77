"""FP32 / FP64 matrix-core M2L (m2l_mma.hip) against the plain kernel at every
order (row-tile, k-chunk and tail sizes all follow from it), at the smallest
and largest column counts of a work-group, and in batches whose replicas share
column groups.

Bounds.  FP64: both kernels round sums of 189 K products in different orders;
each sum's error is at most 189 K 2^-53 times its sign-free size, and the
results are compared relative to the RMS of the field of like-signed charges
(an upper bound of that size): 189 * 256 * 2^-53 = 5.4e-12.  FP32: the error of
the matrix-core path against FP64 is at most 1.5 times the plain FP32 path's
(the bound of test_matrix_core_m2l_matches_plain)."""
import numpy as np
import pytest

from paper_2410_01626_amd import workloads as W
from tests.gpu_util import run

pytestmark = pytest.mark.gpu
TOL64 = 189 * 256 * 2.0 ** -53


def _rel(a, b, scale):
    return np.sqrt(np.mean((a - b) ** 2)) / np.sqrt(np.mean(scale ** 2))


def _unsigned(d):
    u = dict(d)
    u.update(qA=np.abs(d["qA"]), qB=np.abs(d["qB"]))
    return u


@pytest.mark.parametrize("periodic", [True, False])
@pytest.mark.parametrize("order", range(1, 16))
def test_fp64_orders(order, periodic):
    d = W.tiny_periodic(31, n=150, depth=2, order=order) if periodic else W.random_open(32, n=150, order=order)
    a = run(d, "fp64", m2l_kernel=1)
    b = run(d, "fp64")
    size = run(_unsigned(d), "fp64", m2l_kernel=1) if not periodic else a
    scale = {k: np.maximum(np.abs(size[k]), np.abs(a[k])) for k in ("phi", "F")}
    for k in ("phi", "F"):
        assert _rel(b[k], a[k], scale[k]) <= TOL64, k


@pytest.mark.parametrize("periodic", [True, False])
@pytest.mark.parametrize("order", range(1, 11))
def test_f32_orders(order, periodic):
    d = W.tiny_periodic(33, n=150, depth=2, order=order) if periodic else W.random_open(34, n=150, order=order)
    r = run(d, "fp64", m2l_kernel=1)
    a = run(d, "f32", m2l_kernel=1)
    b = run(d, "f32")
    for k in ("phi", "F"):
        ea, eb = _rel(a[k], r[k], r[k]), _rel(b[k], r[k], r[k])
        assert eb <= 1.5 * ea + 2.0 ** -22, (k, ea, eb)


@pytest.mark.parametrize("prec", ["fp64", "f32"])
@pytest.mark.parametrize("periodic,depth,chunk", [(True, 1, 0), (True, 3, 0), (True, 3, 189), (True, 4, 0),
                                                  (False, 2, 1), (False, 3, 65), (False, 4, 0)])
def test_depths_and_chunks(prec, periodic, depth, chunk):
    """From one target column per class (periodic depth 1) to several tiles,
    one chunk of all offsets and one chunk per offset."""
    d = W.tiny_periodic(35, n=300, depth=depth, order=5) if periodic else W.random_open(36, n=300, depth=depth,
                                                                                       order=5)
    r = run(d, "fp64", m2l_kernel=1)
    b = run(d, prec, m2l_chunk=chunk)
    if prec == "fp64":
        assert _rel(b["F"], r["F"], r["F"]) <= TOL64
        return
    a = run(d, prec, m2l_kernel=1)
    assert _rel(b["F"], r["F"], r["F"]) <= 1.5 * _rel(a["F"], r["F"], r["F"]) + 2.0 ** -22


@pytest.mark.parametrize("prec", ["fp64", "f32"])
def test_replicas_share_column_groups(prec):
    """Seven open replicas of odd sizes in one call against each alone."""
    import torch
    from paper_2410_01626_amd import fmm
    dev = torch.device("cuda:0")
    reps = [W.random_open(40 + r, n=60 + 17 * r, n_sites=2, depth=2, order=8) for r in range(7)]
    ao = np.cumsum([0] + [r["x"].shape[0] for r in reps])
    so = np.cumsum([0] + [r["lam"].size for r in reps])
    plan = fmm.Plan(2, 8, precision=prec, max_atoms=int(ao[-1]), max_sites=int(so[-1]), max_replicas=7, device=dev)
    cat = [torch.tensor(np.concatenate([r[k] for r in reps]), dtype=plan.dtype, device=dev)
           for k in ("x", "qA", "qB")]
    site = torch.tensor(np.concatenate([r["site"] for r in reps]), device=dev)
    lam = torch.tensor(np.concatenate([r["lam"] for r in reps]), device=dev)
    out = plan.eval_batched(ao, so, *cat, site, lam)
    for r, d in enumerate(reps):
        one = plan.eval(*(t[ao[r]:ao[r + 1]].clone() for t in cat), site[ao[r]:ao[r + 1]].clone(),
                        lam[so[r]:so[r + 1]].clone())
        torch.cuda.synchronize()
        # a column's sums do not depend on its place in the column groups
        assert torch.equal(out["F"][ao[r]:ao[r + 1]], one["F"])
    plan.close()
