"""bf16x3 M2L without resident sources (m2l_bf16x3.hip; m2l_kernel = 3 forces it
at any depth): every row-tile count (orders 1-10), depths with one and several
column tiles and mixed levels in a tile, open trees with absent sources, and
replicas.  Bound: the FP32 plain kernel's error against the FP64 one plus 2^-16
kappa, kappa the cancellation ratio RMS phi(|q|) / RMS phi (the bound and its
derivation are those of test_matrix_core_m2l_matches_plain)."""
import numpy as np
import pytest

from paper_2410_01626_amd import workloads as W
from tests.gpu_util import run

pytestmark = pytest.mark.gpu


def _check(d, **kw):
    def rel(u, v, k):
        return np.sqrt(np.sum((u[k] - v[k]) ** 2) / np.sum(v[k] ** 2))
    r = run(d, "fp64", m2l_kernel=1)
    a = run(d, "f32", m2l_kernel=1)
    b = run(d, "bf16x3", m2l_kernel=3, **kw)
    da = dict(d)
    da["periodic"] = False
    da["qA"], da["qB"] = np.abs(d["qA"]), np.abs(d["qA"])
    ab = run(da, "fp64", depth=1)
    for k in ("F", "phi"):
        kappa = np.sqrt(np.mean(ab[k] ** 2) / np.mean(r[k] ** 2))
        bound = rel(a, r, k) + 2.0 ** -16 * kappa
        assert rel(b, r, k) <= bound, (k, rel(b, r, k), bound)


@pytest.mark.parametrize("periodic", [True, False])
@pytest.mark.parametrize("order", range(1, 11))
def test_orders(order, periodic):
    mk = W.tiny_periodic if periodic else W.random_open
    _check(mk(51, n=1200, edge=2.0, n_sites=2, depth=3 if not periodic else 2, order=order))


@pytest.mark.parametrize("periodic,depth,chunk", [(True, 1, 0), (True, 3, 189), (True, 4, 0), (True, 4, 1),
                                                  (False, 2, 0), (False, 4, 0), (False, 4, 100)])
def test_depths_and_chunks(periodic, depth, chunk):
    mk = W.tiny_periodic if periodic else W.random_open
    _check(mk(52, n=2000, edge=2.2, n_sites=2, depth=depth, order=7), m2l_chunk=chunk)


def test_replicas_equal_single():
    import torch
    from paper_2410_01626_amd import fmm
    dev = torch.device("cuda:0")
    reps = [W.random_open(60 + r, n=400 + 131 * r, n_sites=2, depth=4, order=9) for r in range(3)]
    ao = np.cumsum([0] + [r["x"].shape[0] for r in reps])
    so = np.cumsum([0] + [r["lam"].size for r in reps])
    plan = fmm.Plan(4, 9, precision="bf16x3", max_atoms=int(ao[-1]), max_sites=int(so[-1]), max_replicas=3, device=dev)
    cat = [torch.tensor(np.concatenate([r[k] for r in reps]), dtype=plan.dtype, device=dev) for k in ("x", "qA", "qB")]
    site = torch.tensor(np.concatenate([r["site"] for r in reps]), device=dev)
    lam = torch.tensor(np.concatenate([r["lam"] for r in reps]), device=dev)
    out = plan.eval_batched(ao, so, *cat, site, lam)
    for r in range(3):
        one = plan.eval(*(t[ao[r]:ao[r + 1]].clone() for t in cat), site[ao[r]:ao[r + 1]].clone(),
                        lam[so[r]:so[r + 1]].clone())
        torch.cuda.synchronize()
        assert torch.equal(out["F"][ao[r]:ao[r + 1]], one["F"])
    plan.close()
