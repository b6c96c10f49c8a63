"""Image calls without a plan: over the whole grid up to 1024^2, over the occupied band above."""
import gc

import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_1906_07102_amd as lmg  # noqa: E402

DEV = "cuda:0"


@pytest.mark.parametrize("prec", [lmg.F32, lmg.F64])
@pytest.mark.parametrize("N, n", [(64, 0), (64, 500), (512, 7001), (1024, 300), (2048, 9000)])
def test_oneshot_images_match_the_plan(N, n, prec):
    """Dirty image and prediction equal a plan's (transforms of log2 N stages: 2 eps log2 N of the norm), with dropped
    coordinates and where all are dropped, and the table may go as soon as the calls have returned."""
    print(f"one-shot images N={N} n={n} prec={prec}", flush=True)
    rng = np.random.default_rng(N + n)
    uv = rng.uniform(-N / 9, N / 9, (n, 2))
    uv[n // 2 : n // 2 + 1] = np.nan
    dt = torch.complex128 if prec == lmg.F64 else torch.complex64
    eps = 2.0**-53 if prec == lmg.F64 else 2.0**-24
    tol = 2 * eps * np.log2(N)
    keep = lmg.Table.create(5, 0.25, 300, 3)
    vis = torch.from_numpy(rng.standard_normal(n) + 1j * rng.standard_normal(n)).to(DEV, dt)
    M = N // 2
    image = torch.from_numpy(rng.standard_normal((M, M)) + 1j * rng.standard_normal((M, M))).to(DEV, dt)
    for coords in (uv, np.full_like(uv, np.inf)):
        ud = torch.from_numpy(coords).to(DEV)
        table = lmg.Table.create(5, 0.25, 300, 3)
        dirty = lmg.make_dirty_image(table, N, ud, vis)
        model = lmg.predict_visibilities(table, N, ud, image)
        del table
        gc.collect()
        plan = lmg.Plan(keep, N, ud, prec)
        want_d, want_m = plan.make_dirty_image(vis), plan.predict_visibilities(image)
        assert torch.linalg.vector_norm(dirty - want_d) <= tol * torch.linalg.vector_norm(want_d)
        assert torch.linalg.vector_norm(model - want_m) <= tol * torch.linalg.vector_norm(want_m)
