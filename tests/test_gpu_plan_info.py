"""fmm_plan_info of the matrix-core M2L: work-groups and LDS of the launch that a
plan of one system makes."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["f32", "fp64", "bf16x3"])
@pytest.mark.parametrize("depth,order,kernel", [(1, 2, 0), (3, 8, 0), (3, 8, 3), (4, 6, 0), (5, 8, 0)])
def test_m2l_launch(prec, depth, order, kernel):
    import torch
    from paper_2410_01626_amd import fmm
    if kernel and prec != "bf16x3":
        pytest.skip("a bf16x3 form")
    plan = fmm.Plan(depth, order, periodic=True, precision=prec, max_atoms=1000, m2l_kernel=kernel,
                    device=torch.device("cuda:0"))
    i = plan.info()
    plan.close()
    # columns of the eight classes: their boxes at levels 1 to depth
    columns = 8 * sum(8 ** (lev - 1) for lev in range(1, depth + 1))
    # a work-group has at most 80 columns (bf16x3 without resident sources 160, of
    # one row tile 320) and one chunk; all chunks and columns are covered
    most = {"f32": 80, "fp64": 64, "bf16x3": 320}[prec]
    assert i["m2l_workgroups"] * most >= columns * i["m2l_chunks"]
    # two operator buffers at least, and within a CU's LDS
    K, size = (order + 1) ** 2, {"f32": 4, "fp64": 8, "bf16x3": 4}[prec]
    parts = 1 if prec == "bf16x3" else 2  # (an operator's rows may be cut in parts)
    assert 2 * K * K * size // parts <= i["m2l_lds_bytes"] <= 160 * 1024
