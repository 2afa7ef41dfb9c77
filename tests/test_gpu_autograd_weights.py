"""Backward of the autograd wrapper takes the upstream weights as they come:
outputs that the loss leaves out, weights that are zero, a plan on a stream of
its own; no wait for the device in between."""
import numpy as np
import pytest

from paper_2410_01626_amd import workloads as W

pytestmark = pytest.mark.gpu
KEYS = ("grad_x", "grad_qA", "grad_qB", "grad_lambda")


@pytest.mark.parametrize("own_stream", [False, True])
@pytest.mark.parametrize("used", ["E", "F", "phi", "E+F", "F+phi", "E+0F"])
def test_backward_takes_the_weights_it_is_given(used, own_stream):
    import torch
    from paper_2410_01626_amd import fmm
    from paper_2410_01626_amd.autograd import fmm_coulomb
    dev = torch.device("cuda:0")
    d = W.tiny_periodic(98, n=400, edge=1.5, n_sites=3, depth=2, order=6)
    rng = np.random.default_rng(5)
    stream = torch.cuda.Stream(dev) if own_stream else None
    plan = fmm.Plan(2, 6, periodic=True, precision="fp64", max_atoms=400, max_sites=3, device=dev,
                    stream=stream)
    leaves = [torch.tensor(d[k], device=dev, requires_grad=True) for k in ("x", "qA", "qB")]
    x, qA, qB = leaves
    lam = torch.tensor(d["lam"], device=dev, requires_grad=True)
    site = torch.tensor(d["site"], device=dev)
    wF = torch.tensor(rng.standard_normal((400, 3)), device=dev)
    wp = torch.tensor(rng.standard_normal(400), device=dev)
    gE = torch.tensor([0.25 if "E" in used else 0.0], dtype=torch.float64, device=dev)
    torch.cuda.synchronize()
    ref = plan.eval_adjoint_full(x.detach(), qA.detach(), qB.detach(), site, lam.detach(), gE=gE,
                                 gphi=wp if "phi" in used else None,
                                 gF=wF if "F" in used and "0F" not in used else None, box=d["box"])
    torch.cuda.synchronize()
    E, F, phi, _ = fmm_coulomb(plan, x, qA, qB, site, lam, d["box"])
    torch.cuda.synchronize()
    loss = 0.0
    if "E" in used:
        loss = loss + 0.25 * E.sum()
    if "0F" in used:
        loss = loss + (0.0 * F).sum()
    elif "F" in used:
        loss = loss + (wF * F).sum()
    if "phi" in used:
        loss = loss + (wp * phi).sum()
    before = torch.cuda.get_sync_debug_mode()
    torch.cuda.set_sync_debug_mode("error")  # a wait for the device raises
    try:
        g = torch.autograd.grad(loss, [x, qA, qB, lam])
    finally:
        torch.cuda.set_sync_debug_mode(before)
    torch.cuda.synchronize()
    for a, k in zip(g, KEYS):
        r = ref[k].cpu().numpy()
        # FP64 throughout; the paths sum the same terms in another order
        np.testing.assert_allclose(a.cpu().numpy(), r, rtol=1e-11, atol=1e-11 * np.abs(r).max())
    plan.close()
