"""Work items that are quadrants of 64-cell tiles (8192^2 grids)."""
import numpy as np
import pytest

from oracle import imaging as im
from oracle import lmtable as lt

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_1906_07102_amd as lmg  # noqa: E402

DEV = "cuda:0"
TOL = {lmg.F32: 1e-5, lmg.F32_KAHAN: 1e-5, lmg.F64: 1e-12}


@pytest.mark.parametrize("prec,W", [(lmg.F32, 7), (lmg.F32_KAHAN, 4), (lmg.F64, 7), (lmg.F64, 16)])
def test_quadrant_items(prec, W):
    """Visibilities on and around the corners of quadrants and tiles, around the grid's edge (footprints that wrap)
    and piled up in one cell (several items of one tile): the whole grid's non-zero cells, overwriting and
    accumulating, the degridding and a second channel of the same data, against the FP64 oracle at the usual
    tolerances (FP64 1e-12, FP32 1e-5)."""
    print(f"quadrants prec={prec} W={W}", flush=True)
    N = 8192
    h = lt.optimal_h(7, 0.25)
    otab = lt.Table(W, 0.25, 300 // W, 3, lt.table_nodes(h, W, 0.25, 300 // W, 3))
    gtab = lmg.Table.from_nodes(W, 0.25, 300, 3, h, otab.nodes)
    rng = np.random.default_rng(60 + W)
    corners = 32.0 * rng.integers(-4, 4, (3000, 2)) + rng.uniform(-W, W, (3000, 2))
    edge = np.stack([rng.uniform(-4096, -4040, 2000), rng.uniform(4040, 4096, 2000)], axis=1)
    pile = rng.uniform(70.0, 71.0, (9000, 2))
    uv = np.concatenate([corners, edge, pile])
    vis = rng.standard_normal(len(uv)) + 1j * rng.standard_normal(len(uv))
    cdt = torch.complex128 if prec == lmg.F64 else torch.complex64
    uvd, vd = torch.from_numpy(uv).to(DEV), torch.from_numpy(vis).to(DEV, cdt)
    plan = lmg.Plan(gtab, N, uvd, prec)
    assert plan.info()["tile"] == 64
    want = torch.from_numpy(im.grid(uv, vis, None, N, otab)).to(DEV)
    scale = want.norm()
    g = plan.grid(vd)
    assert (g.to(torch.complex128) - want).norm() < TOL[prec] * scale
    g2 = plan.grid(vd, out=g.clone(), accumulate=True)
    assert (g2.to(torch.complex128) - 2 * want).norm() < 2 * TOL[prec] * scale
    got = plan.degrid(want.to(cdt)).cpu().numpy()
    ref = im.degrid(uv, want.cpu().numpy(), otab)
    assert np.linalg.norm(got - ref) < TOL[prec] * np.linalg.norm(ref)
    if prec == lmg.F32:
        both = lmg.BatchPlan(gtab, N, torch.cat([uvd, uvd]), [0, len(uv), 2 * len(uv)], prec).grid(torch.cat([vd, vd]))
        assert torch.equal(both[0], g) and torch.equal(both[1], g)


def test_few_visibilities_keep_the_allocation_free_call():
    """1,500 scattered visibilities on 8192^2: whole tiles' patches fit the allocation-free call's scratch, four
    quadrants' would not, so the plan keeps whole tiles and the call keeps working, with the planned call's bits."""
    N, n = 8192, 1500
    gtab = lmg.Table.create(7, 0.25, 300, 3)
    rng = np.random.default_rng(3)
    uv = torch.from_numpy(rng.uniform(-2000, 2000, (n, 2))).to(DEV)
    vis = torch.from_numpy((rng.standard_normal(n) + 1j * rng.standard_normal(n)).astype(np.complex64)).to(DEV)
    plan = lmg.Plan(gtab, N, uv, lmg.F32)
    assert torch.equal(plan.grid_noalloc(vis), plan.grid(vis))
