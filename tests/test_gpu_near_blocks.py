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


@pytest.mark.parametrize("depth,n", [(1, 200), (1, 260), (1, 2000), (2, 1600), (2, 5100)])
def test_fp64_automatic_split_matches_one_block(depth, n):
    """FP64 trees of few leaves take a block per 32 targets: the same pairs in
    another order, n sums of at most n terms each."""
    from paper_2410_01626_amd import workloads as W
    from tests.gpu_util import run
    d = W.random_open(70 + n, n=n, edge=2.5, n_sites=3, depth=depth, order=6)
    a, b = run(d, "fp64"), run(d, "fp64", p2p_split=1)
    for k in ("F", "phi", "dVdl"):
        assert np.abs(a[k] - b[k]).max() <= n * 2.0 ** -52 * np.abs(b[k]).max(), k


@pytest.mark.parametrize("n", [1, 5, 1024, 16384, 70000])
def test_bounding_cube_forms_agree(n):
    """The cube of up to 16,384 atoms by one block, of more by two launches:
    a call with n atoms and one with 17,000 more atoms of zero charge inside their
    hull give the same potentials."""
    import torch
    from paper_2410_01626_amd import fmm
    dev = torch.device("cuda:0")
    rng = np.random.default_rng(n)
    x = rng.uniform(-1.0, 3.0, (n, 3)) + np.array([5.0, -7.0, 0.25])
    q = rng.uniform(-1, 1, n)
    pad = 17000
    c = 0.5 * (x.min(0) + x.max(0))
    # zero charges well inside the hull (a quarter of the way from its centre)
    xp = np.concatenate([x, c + 0.25 * (x.max(0) - x.min(0)) * rng.uniform(-1, 1, (pad, 3))])
    qp = np.concatenate([q, np.zeros(pad)])
    plan = fmm.Plan(2, 4, precision="fp64", max_atoms=n + pad, max_sites=1, p2p_split=1, device=dev)
    phi = []
    for xv, qv in ((x, q), (xp, qp)):
        t = [torch.tensor(v, dtype=torch.float64, device=dev) for v in (xv, qv, qv)]
        s = torch.full((len(qv),), -1, dtype=torch.int32, device=dev)
        out = plan.eval(*t, s, torch.zeros(0, dtype=torch.float64, device=dev))
        torch.cuda.synchronize()
        phi.append(out["phi"].cpu().numpy()[:n])
    plan.close()
    assert np.abs(phi[0] - phi[1]).max() <= (n + pad) * 2.0 ** -52 * (np.abs(phi[0]).max() + 1e-300)


@pytest.mark.parametrize("S", [4097, 32768, 32769, 40003])
def test_site_scan_tiles(S):
    """One atom per site past the in-block scan and around its tile of 32,768:
    dV/dlambda of a site is (qB - qA) phi of its atom."""
    import torch
    from paper_2410_01626_amd import fmm
    dev = torch.device("cuda:0")
    rng = np.random.default_rng(S)
    x = torch.tensor(rng.uniform(0, 8, (S, 3)), dtype=torch.float64, device=dev)
    qA = torch.tensor(rng.uniform(-1, 1, S), dtype=torch.float64, device=dev)
    qB = qA + torch.tensor(rng.uniform(-1, 1, S), dtype=torch.float64, device=dev)
    site = torch.tensor(rng.permutation(S), dtype=torch.int32, device=dev)
    lam = torch.rand(S, dtype=torch.float64, device=dev)
    plan = fmm.Plan(3, 2, precision="fp64", max_atoms=S, max_sites=S, device=dev)
    out = plan.eval(x, qA, qB, site, lam)
    torch.cuda.synchronize()
    want = torch.zeros(S, dtype=torch.float64, device=dev)
    want[site.long()] = (qB - qA) * out["phi"]
    assert (out["dVdl"] - want).abs().max() <= 4 * 2.0 ** -53 * want.abs().max()
    plan.close()


def test_leaf_scan_of_the_deepest_tree():
    """Depth 6 has eight scan tiles of leaves: every atom is found in its leaf
    (the potentials of a depth-2 solve, to the accuracy of order 10)."""
    from paper_2410_01626_amd import workloads as W
    from tests.gpu_util import TOL_F, run
    d = W.random_open(90, n=900, edge=2.0, n_sites=3, depth=2, order=10)
    a, b = run(d, "fp64"), run(d, "fp64", depth=6, m2l_kernel=0)
    e = np.sqrt(np.sum((a["phi"] - b["phi"]) ** 2) / np.sum(a["phi"] ** 2))
    assert e <= 2 * TOL_F[10]
