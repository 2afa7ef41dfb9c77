"""Near field of trees of few, full leaves, where several blocks share a leaf:
every force and potential equals the one-block form's bit for bit (the same
sums in the same order), the energy and dV/dlambda up to the order of their
FP64 partials.  Leaf populations around the target chunk (64), the round (512)
and the block counts; the plan's own maxima choose the form, so the one-block
reference is the same plan with more replica slots (and the M2L chunks, which
follow the slots too, set alike)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

COUNTS = [[0, 1, 64, 65, 511, 512, 513, 640], [700, 1025, 1100, 130, 1, 576, 33, 900],
          [300, 300, 300, 300, 320, 256, 257, 319]]


@pytest.mark.parametrize("prec", ["f32", "fp64"])
@pytest.mark.parametrize("periodic", [True, False])
@pytest.mark.parametrize("counts", COUNTS)
def test_shared_leaves_match_one_block(counts, periodic, prec):
    import torch
    from paper_2410_01626_amd import fmm
    dev = torch.device("cuda:0")
    rng = np.random.default_rng(7)
    x = np.concatenate([(np.array([o >> 2, (o >> 1) & 1, o & 1]) + rng.uniform(0.02, 0.98, (c, 3))) * 2.0
                        for o, c in enumerate(counts)])
    n, S = x.shape[0], 5
    x = x.astype(np.float32).astype(np.float64)
    q = rng.uniform(-1, 1, n).astype(np.float32).astype(np.float64)
    site = np.where(np.arange(n) % 97 == 0, np.arange(n) % S, -1).astype(np.int32)
    out = []
    for slots in (1, 32):
        plan = fmm.Plan(1, 6, periodic=periodic, precision=prec, max_atoms=n, max_sites=S, max_replicas=slots,
                        p2p_waves=8, m2l_chunk=7, device=dev)
        t = [torch.tensor(v, dtype=plan.dtype, device=dev) for v in (x, q, 0.5 * q)]
        r = plan.eval(*t, torch.tensor(site, device=dev), torch.linspace(0, 1, S, dtype=torch.float64, device=dev),
                      box=[4.0] * 3 if periodic else None)
        torch.cuda.synchronize()
        out.append({k: v.cpu().numpy() for k, v in r.items()})
        plan.close()
    a, b = out
    np.testing.assert_array_equal(a["F"], b["F"])
    np.testing.assert_array_equal(a["phi"], b["phi"])
    np.testing.assert_array_equal(a["dVdl"], b["dVdl"])
    size = np.sum(np.abs(q * a["phi"]))
    assert abs(a["E"][0] - b["E"][0]) <= n * 2.0 ** -53 * size
