"""Near field of trees of many leaves where a few of them are crowded (systems
that fill a part of their cell): those leaves are done by whole blocks, found in
the order of work or through the leaf kernels' list."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _tensors(plan, x, q, site, reps):
    import torch
    t = [torch.tensor(np.concatenate([v] * reps), dtype=plan.dtype, device=plan.device) for v in (x, q, 0.5 * q)]
    lam = torch.linspace(0, 1, 3, dtype=torch.float64, device=plan.device).repeat(reps)
    return t + [torch.tensor(np.concatenate([site] * reps), device=plan.device), lam]


def _charges(n, seed):
    rng = np.random.default_rng(seed)
    q = rng.uniform(-1, 1, n).astype(np.float32).astype(np.float64)
    return q, np.where(np.arange(n) % 41 == 0, np.arange(n) % 3, -1).astype(np.int32)


@pytest.mark.parametrize("counts", [[64, 65, 63, 0, 1], [0, 128, 0, 0, 129, 2], [0] * 13 + [255, 256, 257, 33],
                                    [0] * 31 + [520, 700]])
def test_listed_leaves_match_block_per_leaf(counts):
    """Open, depth 2 (no order of work): 64 systems take the wavefront form and
    its list, one system a block per leaf; the same bits."""
    import torch
    from paper_2410_01626_amd import fmm
    dev = torch.device("cuda:0")
    rng = np.random.default_rng(5)
    x = [np.array([[0.0, 0, 0], [4.0, 4, 4]])]  # the cube's corners
    for leaf in range(64):
        o = np.array([leaf >> 4, (leaf >> 2) & 3, leaf & 3])
        x.append(o + rng.uniform(0.03, 0.97, (counts[leaf % len(counts)], 3)))
    x = np.concatenate(x).astype(np.float32).astype(np.float64)
    n = x.shape[0]
    assert n <= 48 * 64
    q, site = _charges(n, 6)
    plan = fmm.Plan(2, 6, precision="f32", max_atoms=64 * n, max_sites=192, max_replicas=64, p2p_waves=4, device=dev)
    out = []
    for reps in (1, 64, 64):  # (the list is empty again for the second)
        r = plan.eval_batched([n * i for i in range(reps + 1)], [3 * i for i in range(reps + 1)],
                              *_tensors(plan, x, q, site, reps))
        torch.cuda.synchronize()
        out.append({k: v.cpu().numpy() for k, v in r.items()})
    plan.close()
    for o in out[1:]:
        for k in ("F", "phi", "dVdl", "E"):
            for i in range(64):
                m = len(out[0][k])
                np.testing.assert_array_equal(out[0][k], o[k][i * m:(i + 1) * m], err_msg=k)


@pytest.mark.parametrize("prec,periodic", [("f32", True), ("bf16x3", False)])
def test_more_crowded_leaves_than_blocks(prec, periodic):
    """Depth 4 with 1,300 leaves of 70 to 560 atoms among 4,096: blocks come
    back to the list.  Against a block per 32 targets (FP32 sums of at most 27 *
    600 terms in another order), replayed from a graph, and through
    fmm_eval_noalloc, whose list starts in memory that other calls used."""
    import torch
    from paper_2410_01626_amd import fmm
    dev = torch.device("cuda:0")
    rng = np.random.default_rng(8)
    full = rng.permutation(4096)[:1300]
    pop = np.zeros(4096, int)
    pop[full] = 70
    pop[full[:40]] = [260, 560] * 20
    leaf = np.repeat(np.arange(4096), pop)
    o = np.stack([leaf >> 8, (leaf >> 4) & 15, leaf & 15], 1)
    x = (o + rng.uniform(0.03, 0.97, (len(leaf), 3))) * 0.5
    x = rng.permutation(x).astype(np.float32).astype(np.float64)
    n = len(x)
    q, site = _charges(n, 9)
    box = [8.0] * 3 if periodic else None
    got = {}
    with torch.cuda.stream(torch.cuda.Stream(dev)):
        for name, kw in (("list", {}), ("graph", {"graph": True}), ("blocks", {"p2p_split": 2})):
            plan = fmm.Plan(4, 4, periodic=periodic, precision=prec, max_atoms=n, max_sites=3, p2p_waves=4,
                            device=dev, **kw)
            t = _tensors(plan, x, q, site, 1)
            out = plan.eval(*t, box=box)
            for rep in range(3):
                for v in out.values():
                    v.fill_(float("nan"))
                plan.eval(*t, box=box, out=out)
                torch.cuda.synchronize()
                got[name, rep] = {k: v.cpu().numpy() for k, v in out.items()}
            if name == "list":
                size = plan.eval(t[0], t[1].abs(), t[2].abs(), *t[3:], box=box)["phi"].abs().cpu().numpy()
                for rep in range(2):
                    r = plan.eval_noalloc(*t, box=box)
                    torch.cuda.synchronize()
                    got["noalloc", rep] = {k: v.cpu().numpy() for k, v in r.items()}
            plan.close()
    ref = got["list", 0]
    for key, r in got.items():
        if key[0] == "blocks":
            assert np.abs(r["phi"] - ref["phi"]).max() <= 27 * 600 * 2.0 ** -24 * size.max()
        else:
            for k in ("F", "phi", "dVdl", "E"):
                np.testing.assert_array_equal(r[k], ref[k], err_msg="%s %s" % (key, k))


@pytest.mark.parametrize("prec,split", [("f32", 0), ("fp64", 0), ("f32", 3)])
def test_crowded_leaves_of_4096(prec, split):
    """Depth 4, a block (or several) per leaf: leaves of more than 32 times the
    mean population come first.  Every leaf is done once (outputs start as NaN),
    the energy is the charges' potentials', and repeated calls give the same
    bits."""
    import torch
    from paper_2410_01626_amd import fmm
    dev = torch.device("cuda:0")
    rng = np.random.default_rng(10)
    pop = np.full(4096, 5)
    pop[rng.permutation(4096)[:60]] = [13, 24, 300, 200, 190, 600] * 10
    pop[:8] = 0
    leaf = np.repeat(np.arange(4096), pop)
    o = np.stack([leaf >> 8, (leaf >> 4) & 15, leaf & 15], 1)
    x = (o + np.floor(rng.uniform(0.05, 0.95, (len(leaf), 3)) * 4096) / 4096) * 0.5
    n = len(x)
    q, site = _charges(n, 11)
    plan = fmm.Plan(4, 4, periodic=True, precision=prec, max_atoms=n, max_sites=3, p2p_waves=8, p2p_split=split,
                    device=dev)
    got = []
    t = _tensors(plan, x, q, site, 1)
    for _ in range(2):
        out = plan.eval(*t, box=[8.0] * 3)
        for v in out.values():
            v.fill_(float("nan"))
        plan.eval(*t, box=[8.0] * 3, out=out)
        torch.cuda.synchronize()
        r = {k: v.double().cpu().numpy() for k, v in out.items()}
        assert all(np.isfinite(v).all() for v in r.values())
        lam = np.linspace(0, 1, 3)[site] * (site >= 0)
        e = 0.5 * ((1 - 0.5 * lam) * q * r["phi"])
        assert abs(r["E"][0] - e.sum()) <= 4 * 2.0 ** (-24 if prec == "f32" else -52) * n ** 0.5 * np.abs(e).max()
        got.append(r)
    plan.close()
    for k in ("F", "phi", "E", "dVdl"):
        np.testing.assert_array_equal(got[0][k], got[1][k], err_msg=k)


def test_lists_of_both_forms_in_one_plan():
    """One plan, depth 4: a call with more atoms than the wavefront form takes
    lists other leaves than the next, which runs that form."""
    import torch
    from paper_2410_01626_amd import fmm
    dev = torch.device("cuda:0")
    rng = np.random.default_rng(12)
    many = rng.uniform(0, 8.0, (48 * 4096 + 1, 3))
    many[:5000] = 0.5 + rng.uniform(0, 0.5, (5000, 3))
    many = many.astype(np.float32).astype(np.float64)
    few = np.concatenate([rng.uniform(0, 8.0, (9000, 3)), 3.01 + rng.uniform(0, 0.48, (700, 3)),
                          rng.uniform(0, 0.5, (90, 3))]).astype(np.float32).astype(np.float64)
    got = []
    for first in (many, None):
        plan = fmm.Plan(4, 4, periodic=True, precision="f32", max_atoms=len(many), max_sites=3, p2p_waves=4, device=dev)
        for x in ([many, few] if first is not None else [few]):
            r = plan.eval(*_tensors(plan, x, *_charges(len(x), 13), 1), box=[8.0] * 3)
        torch.cuda.synchronize()
        got.append({k: v.cpu().numpy() for k, v in r.items()})
        plan.close()
    for k in ("F", "phi", "E", "dVdl"):
        np.testing.assert_array_equal(got[0][k], got[1][k], err_msg=k)
