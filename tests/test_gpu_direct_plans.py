"""Plans on both sides of 2^20 visibilities, up to where the scatter writes tile order itself."""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_1906_07102_amd as lmg  # noqa: E402

DEV = "cuda:0"


@pytest.mark.parametrize("channels", [1, 3])
@pytest.mark.parametrize("prec", [lmg.F32, lmg.F64])
def test_direct_and_ordered_scatter_give_the_same_plan(prec, channels):
    """2^20 visibilities, and the same with three more that are dropped: the same grids, visibilities and plan order to the
    bit."""
    print(f"direct plans prec={prec} channels={channels}", flush=True)
    n, N = 1 << 20, 512
    cdt = torch.complex128 if prec == lmg.F64 else torch.complex64
    table = lmg.Table.create(5, 0.25, 300, 3)
    g = torch.Generator(device=DEV).manual_seed(channels)
    uv = (torch.rand(n, 2, generator=g, device=DEV, dtype=torch.float64) - 0.5) * torch.randn(
        n, 1, generator=g, device=DEV, dtype=torch.float64) * 100.0
    vis = torch.randn(n, generator=g, device=DEV, dtype=cdt)
    offsets = [0, n // 3, n // 2, n] if channels == 3 else [0, n]
    direct = lmg.BatchPlan(table, N, uv, offsets, prec)
    bad = torch.full((3, 2), float("nan"), device=DEV, dtype=torch.float64)
    longer = lmg.BatchPlan(table, N, torch.cat([uv, bad]), offsets[:-1] + [n + 3], prec)
    vis3 = torch.cat([vis, vis[:3]])
    assert longer.info()["valid"] == direct.info()["valid"] == n
    grid = direct.grid(vis)
    assert torch.equal(grid, longer.grid(vis3))
    assert torch.equal(direct.degrid(grid), longer.degrid(grid)[:n])
    assert torch.equal(direct.to_plan_order(vis)[:n], longer.to_plan_order(vis3)[:n])
    assert torch.equal(direct.from_plan_order(direct.to_plan_order(vis)), vis)
