"""Degridding with one workgroup per compute unit (batches of a few items each) against the channels alone, with two."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_1906_07102_amd as lmg  # noqa: E402

DEV = "cuda:0"


@pytest.mark.parametrize("prec,W", [(lmg.F32, 8), (lmg.F32_KAHAN, 9), (lmg.F32, 14), (lmg.F64, 4), (lmg.F64, 8)])
def test_a_batch_of_few_items(prec, W):
    N, nchan, per = 512, 8, 12001                       # 514 expected items, ragged channels
    counts = np.full(nchan, per) + np.arange(nchan) * 37
    off = np.concatenate([[0], np.cumsum(counts)])
    rng = np.random.default_rng(W)
    uv = torch.from_numpy(rng.uniform(-N / 4, N / 4, (off[-1], 2))).to(DEV)
    assert off[-1] >= 128 * (nchan * (N // 32) ** 2 // 4 + off[-1] // 8192)
    dt = torch.complex128 if prec == lmg.F64 else torch.complex64
    grid = torch.from_numpy(rng.standard_normal((nchan, N, N)) + 1j * rng.standard_normal((nchan, N, N))).to(DEV, dt)
    table = lmg.Table.create(W, 0.25, 300, 3)
    got = lmg.BatchPlan(table, N, uv, off, prec).degrid(grid)
    for c in range(nchan):
        a, b = int(off[c]), int(off[c + 1])
        alone = lmg.Plan(table, N, uv[a:b].contiguous(), prec).degrid(grid[c].contiguous())
        assert torch.equal(got[a:b], alone), c
