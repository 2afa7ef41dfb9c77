"""The near field's forms for special trees (blocks that share few, full leaves;
a wavefront per leaf with blocks for crowded leaves) with the options of a call:
check mode's coincident atoms, four charge forms, exclusions."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
EDGE = 4.0


def _leaves(depth, pop, seed):
    """pop[leaf] atoms in every leaf of the cube [0, EDGE), in mixed order."""
    rng = np.random.default_rng(seed)
    nb = 1 << depth
    leaf = rng.permutation(np.repeat(np.arange(nb ** 3), pop))
    o = np.stack([leaf // (nb * nb), leaf // nb % nb, leaf % nb], 1)
    x = (o + rng.uniform(0.03, 0.97, (len(leaf), 3))) * (EDGE / nb)
    return x.astype(np.float32).astype(np.float64), leaf


def _shared(seed=1):  # 8 leaves of 560 atoms: four blocks share one
    return _leaves(1, np.full(8, 560), seed) + (dict(depth=1, p2p_waves=8), 1)


def _listed(seed=2):  # 4,096 leaves, crowded ones found through the list
    pop = np.full(4096, 4)
    pop[[5, 900, 4095]] = [70, 300, 600]
    return _leaves(4, pop, seed) + (dict(depth=4, p2p_waves=4), 1)


def _ordered(seed=3):  # 8 systems of 512 leaves, crowded ones found in the order of work
    pop = np.full(512, 8)
    pop[[0, 77, 511]] = [70, 300, 600]
    return _leaves(3, pop, seed) + (dict(depth=3, p2p_waves=4), 8)


FORMS = {"shared": _shared, "listed": _listed, "ordered": _ordered}


def _plan(form, prec, periodic, **more):
    import torch
    from paper_2410_01626_amd import fmm
    x, leaf, kw, reps = FORMS[form]()
    kw = dict(kw, **more)
    n = len(x)
    plan = fmm.Plan(kw.pop("depth"), 4, periodic=periodic, precision=prec, max_atoms=n * reps, max_sites=3 * reps,
                    max_replicas=reps, device=torch.device("cuda:0"), **kw)
    if form == "shared":
        assert plan.info()["p2p_split"] == (4 if "p2p_split" not in more else more["p2p_split"])
    return plan, x, leaf, reps


def _inputs(plan, x, reps, forms=2, last=None):
    """reps copies of the system (the last of them at the positions `last`)."""
    import torch
    rng = np.random.default_rng(4)
    n = len(x)
    xs = np.concatenate([x] * (reps - 1) + [x if last is None else last])
    q = [rng.uniform(-1, 1, n).astype(np.float32).astype(np.float64) for _ in range(forms)]
    site = np.where(np.arange(n) % 41 == 0, np.arange(n) % 3, -1).astype(np.int32)
    t = [torch.tensor(xs, dtype=plan.dtype, device=plan.device)]
    t += [torch.tensor(np.concatenate([v] * reps), dtype=plan.dtype, device=plan.device) for v in q]
    t += [torch.tensor(np.concatenate([site] * reps), device=plan.device)]
    t += [torch.linspace(0, 1, 3, dtype=torch.float64, device=plan.device).repeat(reps)]
    return [n * i for i in range(reps + 1)], [3 * i for i in range(reps + 1)], t


@pytest.mark.parametrize("periodic", [False, True])
@pytest.mark.parametrize("form,prec", [("shared", "f32"), ("shared", "fp64"), ("listed", "f32"), ("ordered", "bf16x3")])
def test_check_mode_reports_coincident_atoms(form, prec, periodic):
    from paper_2410_01626_amd import fmm
    plan, x, leaf, reps = _plan(form, prec, periodic, check=True)
    boxes = [[EDGE] * 3] * reps if periodic else None

    def call(last=None):
        ao, so, t = _inputs(plan, x, reps, last=last)
        plan.eval_batched(ao, so, *t, boxes=boxes)
        plan.sync_check()

    call()  # no flag
    for lf in {"shared": [0, 7], "listed": [5, 17, 900, 4095], "ordered": [0, 9, 77, 511]}[form]:
        at = np.nonzero(leaf == lf)[0]
        for i, j in ((at[0], at[-1]), (at[len(at) // 2], at[1])):
            y = x.copy()
            y[i] = np.round(y[i] * 1024) / 1024  # (exact after a shift by the edge)
            y[j] = y[i] + (np.array([EDGE, 0.0, -EDGE]) if periodic else 0.0)
            with pytest.raises(fmm.FmmError) as e:
                call(y)
            assert e.value.status == fmm.FMM_E_COINCIDENT, (lf, i, j)
            call()  # and the flag is spent
    plan.close()


@pytest.mark.parametrize("periodic", [False, True])
@pytest.mark.parametrize("form", ["shared", "ordered"])
@pytest.mark.parametrize("excl", [False, True])
def test_options_match_block_per_leaf(form, periodic, excl):
    """Four charge forms, with and without exclusions: the bits of the form with
    a block per leaf (one block of a leaf's on request; one system alone)."""
    import torch
    boxes = [EDGE] * 3 if periodic else None
    out = []
    for ref in (False, True):
        plan, x, leaf, reps = _plan(form, "f32", periodic, **({"p2p_split": 1} if ref and form == "shared" else {}))
        n, reps = len(x), 1 if ref else reps
        if excl:  # pairs of atoms (2 i, 2 i + 1) of every system
            m = n * reps
            assert n % 2 == 0
            plan.set_exclusions(np.arange(m + 1), np.arange(m) ^ 1)
        ao, so, t = _inputs(plan, x, reps, forms=4)
        lt = torch.linspace(1, 0, 3, dtype=torch.float64, device=plan.device).repeat(reps)
        r = plan.eval_tautomer_batched(ao, so, *t, lt, boxes=[boxes] * reps if periodic else None)
        torch.cuda.synchronize()
        out.append({k: v.cpu().numpy() for k, v in r.items() if k != "E"})
        plan.close()
    for k, v in out[1].items():
        np.testing.assert_array_equal(out[0][k][-len(v):], v, err_msg=k)
