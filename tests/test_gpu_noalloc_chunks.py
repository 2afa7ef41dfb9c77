"""fmm_eval_noalloc of FP64 plans whose M2L chunk partials do not fit the static
scratch (32 MiB): the same bits as fmm_eval."""
import numpy as np
import pytest

from paper_2410_01626_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("depth,order,chunk,periodic", [
    (3, 15, 6, True), (3, 15, 6, False), (3, 9, 1, True), (3, 10, 1, False), (3, 11, 2, True), (3, 12, 4, False),
    (3, 13, 4, True), (3, 14, 5, True), (4, 9, 18, True), (4, 9, 18, False), (4, 10, 20, True)])
def test_noalloc_without_room_for_partials(depth, order, chunk, periodic):
    import torch
    from paper_2410_01626_amd import fmm
    dev = torch.device("cuda:0")
    n = 1500
    d = (W.tiny_periodic(41, n=n, edge=2.0, n_sites=3, depth=depth, order=order) if periodic else
         W.random_open(42, n=n, edge=2.0, n_sites=3, depth=depth, order=order))
    plan = fmm.Plan(depth, order, periodic=periodic, precision="fp64", max_atoms=n, max_sites=3, m2l_chunk=chunk,
                    device=dev)
    boxes = sum(8 ** lev for lev in range(1 if periodic else 2, depth + 1))
    partials = plan.info()["m2l_chunks"] * boxes * (order + 1) ** 2 * 8
    assert partials > 32 << 20  # no room: what this test is about
    t = [torch.tensor(d[k], device=dev) for k in ("x", "qA", "qB", "site", "lam")]
    box = d["box"] if periodic else None
    a, b = plan.eval(*t, box=box), plan.eval_noalloc(*t, box=box)
    torch.cuda.synchronize()
    for k in ("E", "F", "phi", "dVdl"):
        np.testing.assert_array_equal(a[k].cpu().numpy(), b[k].cpu().numpy(), err_msg=k)
    plan.close()
