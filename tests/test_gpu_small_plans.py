"""Plans small enough to be counted, scanned and scattered by one workgroup, against the passes that larger plans take."""
import numpy as np
import pytest

from oracle import imaging as im
from oracle import lmtable as lt

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_1906_07102_amd as lmg  # noqa: E402

DEV = "cuda:0"


@pytest.mark.parametrize("prec", [lmg.F32, lmg.F64])
@pytest.mark.parametrize("N, n", [(64, 1), (64, 1023), (128, 1025), (128, 4096), (256, 4097), (4096, 3000), (8192, 4096)])
def test_small_plan_is_the_general_plan(N, n, prec):
    """The same visibilities alone and as the first channel of a batch (which takes the general passes; the second
    channel is empty): counts, grid and prediction have the same bits, with dropped coordinates among them, and in FP64
    the grid matches the oracle to 1e-12."""
    print(f"small plan N={N} n={n} prec={prec}", flush=True)
    otab, h = lt.make_table(5, 0.25, 300, 3)
    gtab = lmg.Table.from_nodes(5, 0.25, 300, 3, h, otab.nodes)
    rng = np.random.default_rng(n)
    uv = rng.uniform(-N / 4, N / 4, (n, 2))
    uv[: n // 3] *= 0.05                       # dense tiles beside sparse ones
    if n > 1:
        uv[n // 2, 1] = np.inf
        uv[-1, 0] = np.nan
    vis = rng.standard_normal(n) + 1j * rng.standard_normal(n)
    keep = np.isfinite(uv).all(axis=1)
    dt = torch.complex128 if prec == lmg.F64 else torch.complex64
    ud, vd = torch.from_numpy(uv).to(DEV), torch.from_numpy(vis).to(DEV, dt)
    plan = lmg.Plan(gtab, N, ud, prec)
    general = lmg.BatchPlan(gtab, N, ud, [0, n, n], prec, tile=plan.info()["tile"])
    for key in ("items", "busy_tiles", "valid"):
        assert plan.info()[key] == general.info()[key]
    assert plan.info()["valid"] == keep.sum()
    got = plan.grid(vd)
    both = general.grid(vd)
    assert torch.equal(got, both[0]) and not both[1].any()
    assert torch.equal(plan.degrid(got), general.degrid(both))
    if prec == lmg.F64 and N <= 256:
        want = im.grid(uv[keep], vis[keep], None, N, otab)
        assert np.linalg.norm(got.cpu().numpy() - want) < 1e-12 * np.linalg.norm(want)
