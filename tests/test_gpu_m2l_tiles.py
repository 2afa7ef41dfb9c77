"""FP64 M2L of more column tiles than one grid dimension may have blocks
(65,536): 15 systems at depth 6 make 70,217 tiles.  Every system equals its own
evaluation bit for bit."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("periodic", [False, True])
def test_many_column_tiles(periodic):
    import torch
    from paper_2410_01626_amd import fmm
    dev = torch.device("cuda:0")
    rng = np.random.default_rng(3)
    R, n = 15, 40
    t = [torch.tensor(v, device=dev) for v in (rng.uniform(0, 2.0, (R * n, 3)), rng.uniform(-1, 1, R * n),
                                               rng.uniform(-1, 1, R * n))]
    site = torch.full((R * n,), -1, dtype=torch.int32, device=dev)
    lam = torch.zeros(0, dtype=torch.float64, device=dev)
    plan = fmm.Plan(6, 1, periodic=periodic, precision="fp64", max_atoms=R * n, max_sites=1, max_replicas=R,
                    device=dev)
    b = plan.eval_batched([n * i for i in range(R + 1)], [0] * (R + 1), *t, site, lam,
                          boxes=[[2.0] * 3] * R if periodic else None)
    plan.sync_check()
    for r in range(R):
        s = slice(r * n, (r + 1) * n)
        a = plan.eval(*[v[s].contiguous() for v in t], site[s], lam, box=[2.0] * 3 if periodic else None)
        torch.cuda.synchronize()
        assert torch.equal(a["F"], b["F"][s]) and torch.equal(a["phi"], b["phi"][s]) and a["E"][0] == b["E"][r], r
        assert bool((a["phi"] != 0).all())
    plan.close()
