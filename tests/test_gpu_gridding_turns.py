"""The gridding kernel's turns: waves that share an LDS patch flush in the order of the plan's pieces.

The number of waves of a workgroup must not change a bit of the grid; items of many full pieces (dealt to different
turns) and supports that take several passes over a piece are compared with the FP64 oracle too (relative RMS 1e-12
in FP64, 1e-5 in FP32, as everywhere).
"""
import os

import numpy as np
import pytest

from oracle import imaging as im
from oracle import lmtable as lt

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_1906_07102_amd as lmg  # noqa: E402

DEV = "cuda:0"
TOL = {lmg.F32: 1e-5, lmg.F32_KAHAN: 1e-5, lmg.F64: 1e-12}


def _grid(gtab, N, uv, vis, prec, waves):
    old = os.environ.get("LMG_GRID_WAVES")
    try:
        if waves:
            os.environ["LMG_GRID_WAVES"] = str(waves)
        return lmg.Plan(gtab, N, uv, prec).grid(vis)
    finally:
        os.environ.pop("LMG_GRID_WAVES", None)
        if old is not None:
            os.environ["LMG_GRID_WAVES"] = old


@pytest.mark.parametrize("W", [3, 7, 9])
@pytest.mark.parametrize("prec", [lmg.F32, lmg.F32_KAHAN, lmg.F64])
def test_waves_of_a_workgroup_do_not_change_the_sums(prec, W):
    """30,000 visibilities over some 60 cells of four tiles (items with hundreds of full pieces of few cells, the
    same cell several times in a turn) and 3,000 spread thinly (turns of single-entry tails, a ragged last turn)."""
    print(f"turns prec={prec} W={W}", flush=True)
    h = lt.optimal_h(7, 0.25)
    otab = lt.Table(W, 0.25, 300 // W, 3, lt.table_nodes(h, W, 0.25, 300 // W, 3))
    gtab = lmg.Table.from_nodes(W, 0.25, 300, 3, h, otab.nodes)
    N = 128
    rng = np.random.default_rng(50 + W)
    uv = np.concatenate([rng.uniform(-4.0, 4.0, (30000, 2)), rng.uniform(-32.0, 32.0, (3000, 2))])
    vis = rng.standard_normal(len(uv)) + 1j * rng.standard_normal(len(uv))
    uvd = torch.from_numpy(uv).to(DEV)
    vd = torch.from_numpy(vis).to(DEV, torch.complex128 if prec == lmg.F64 else torch.complex64)
    ref = _grid(gtab, N, uvd, vd, prec, 0)
    for waves in (2, 4, 8):                                               # two patches at this tile
        assert torch.equal(_grid(gtab, N, uvd, vd, prec, waves), ref), waves
    want = im.grid(uv, vis, None, N, otab)
    got = ref.cpu().numpy()
    assert np.linalg.norm(got - want) < TOL[prec] * np.linalg.norm(want)
    odd = _grid(gtab, N, uvd, vd, prec, 3).cpu().numpy()                  # three waves on one patch
    assert np.linalg.norm(odd - want) < TOL[prec] * np.linalg.norm(want)
