"""The image calls on the largest tiles of the largest grid, where a whole grid is assembled from the fewest tiles."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_1906_07102_amd as lmg  # noqa: E402

DEV = "cuda:0"


@pytest.mark.parametrize("W", [1, 3])
def test_image_on_128_cell_tiles(W):
    """Visibilities over the whole of an 8192^2 grid, its edges included, by 128-cell tiles and by the default ones: the
    same image and prediction to the FP32 tolerance of 1e-5."""
    print(f"128-cell tiles W={W}", flush=True)
    N, n = 8192, 20_001
    table = lmg.Table.create(W, 0.25, 30, 3)
    rng = np.random.default_rng(W)
    uv = torch.from_numpy(rng.uniform(-N / 2, N / 2, (n, 2))).to(DEV)
    vis = torch.from_numpy(rng.standard_normal(n) + 1j * rng.standard_normal(n)).to(DEV, torch.complex64)
    large = lmg.BatchPlan(table, N, uv, [0, n], lmg.F32, tile=128)
    usual = lmg.Plan(table, N, uv, lmg.F32)
    got, want = large.make_dirty_image(vis), usual.make_dirty_image(vis)
    assert torch.linalg.vector_norm(got - want) < 1e-5 * torch.linalg.vector_norm(want)
    got, want = large.predict_visibilities(want), usual.predict_visibilities(want)
    assert torch.linalg.vector_norm(got - want) < 1e-5 * torch.linalg.vector_norm(want)
