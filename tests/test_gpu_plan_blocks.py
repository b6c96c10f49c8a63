"""The plan's streaming passes at the edges of their blocks, whose size follows the number of visibilities."""
import numpy as np
import pytest

from oracle import imaging as im
from oracle import lmtable as lt

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_1906_07102_amd as lmg  # noqa: E402

DEV = "cuda:0"


def _table(W=5):
    otab, h = lt.make_table(W, 0.25, 300, 3)
    return otab, lmg.Table.from_nodes(W, 0.25, 300, 3, h, otab.nodes)


@pytest.mark.parametrize("n", [1, 63, 1023, 1024, 1025, 8193, 256 * 1024, 256 * 1024 + 1])
def test_block_edges(n):
    """One visibility less and more than a block's step and than 256 of the smallest blocks: every visibility keeps
    its place through plan order and back (one dropped), and the grid matches the oracle to 1e-12 in FP64."""
    print(f"block edges n={n}", flush=True)
    otab, gtab = _table()
    N = 128
    rng = np.random.default_rng(n)
    uv = rng.uniform(-32.0, 32.0, (n, 2))
    if n > 1:
        uv[n // 2] = np.nan
    vis = rng.standard_normal(n) + 1j * rng.standard_normal(n)
    keep = np.isfinite(uv).all(axis=1)
    plan = lmg.Plan(gtab, N, torch.from_numpy(uv).to(DEV), lmg.F64)
    vd = torch.from_numpy(vis).to(DEV)
    assert plan.info()["valid"] == keep.sum()
    back = plan.from_plan_order(plan.to_plan_order(vd)).cpu().numpy()
    np.testing.assert_array_equal(back, np.where(keep, vis, 0))
    want = im.grid(uv[keep], vis[keep], None, N, otab)
    got = plan.grid(vd).cpu().numpy()
    assert np.linalg.norm(got - want) < 1e-12 * np.linalg.norm(want)


@pytest.mark.parametrize("prec", [lmg.F32, lmg.F64])
def test_block_size_does_not_change_the_sums(prec):
    """A channel of 30,000 visibilities alone (blocks of 1,024) and beside one of 600,000 (blocks of 3,072): its grid
    has the same bits, since a tile's visibilities keep the caller's order."""
    print(f"block sizes prec={prec}", flush=True)
    _, gtab = _table()
    N, a, b = 128, 30_000, 600_000
    rng = np.random.default_rng(7)
    uv = torch.from_numpy(rng.uniform(-32.0, 32.0, (a + b, 2))).to(DEV)
    vis = torch.from_numpy(rng.standard_normal(a + b) + 1j * rng.standard_normal(a + b))
    vis = vis.to(DEV, torch.complex128 if prec == lmg.F64 else torch.complex64)
    both = lmg.BatchPlan(gtab, N, uv, [0, a, a + b], prec)
    alone = lmg.Plan(gtab, N, uv[:a].contiguous(), prec)
    assert torch.equal(both.grid(vis)[0], alone.grid(vis[:a].contiguous()))
