"""8192^2 plans in the modes whose 64-cell tiles are gridded as quadrants: every count of visibilities, several channels,
plan order, the allocation-free call and the image calls."""
import numpy as np
import pytest

from oracle import imaging as im
from oracle import lmtable as lt

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_1906_07102_amd as lmg  # noqa: E402

DEV = "cuda:0"
N = 8192
TOL = {lmg.F32_KAHAN: 1e-5, lmg.F64: 1e-12}
MODES = [lmg.F32_KAHAN, lmg.F64]


def ctype(prec):
    return torch.complex128 if prec == lmg.F64 else torch.complex64


def table(W):
    h = lt.optimal_h(7, 0.25)
    otab = lt.Table(W, 0.25, 300 // W, 3, lt.table_nodes(h, W, 0.25, 300 // W, 3))
    return otab, lmg.Table.from_nodes(W, 0.25, 300, 3, h, otab.nodes)


def inputs(n, seed, prec, extent=2000.0):
    rng = np.random.default_rng(seed)
    uv = rng.uniform(-extent, extent, (n, 2))
    near = np.arange(n) % 2 == 1                 # every other one near one of five places: cells of many summands
    uv[near] = 32.0 * rng.integers(-2, 3, (5, 2))[rng.integers(0, 5, n)][near] + rng.uniform(-3.0, 3.0, (n, 2))[near]
    vis = rng.standard_normal(n) + 1j * rng.standard_normal(n)
    return uv, vis, torch.from_numpy(uv).to(DEV), torch.from_numpy(vis).to(DEV, ctype(prec))


@pytest.mark.parametrize("prec", MODES)
@pytest.mark.parametrize("n", [1, 300, 724, 800, 854, 1500, 2900])
def test_a_channel_alone_and_in_a_batch(prec, n):
    """Visibilities from one to as many as the allocation-free call's scratch takes, with a second channel of
    other data: each channel's grid and visibilities are those of the channel alone to the bit; so are the allocation-free
    call's grid (whole tiles took up to 853 visibilities there), the plan-order call's and twice the accumulated one."""
    print(f"alone and batched prec={prec} n={n}", flush=True)
    _, gtab = table(7)
    _, _, uv0, v0 = inputs(n, n, prec)
    _, _, uv1, v1 = inputs(2 * n + 7, n + 1, prec, 100.0)
    plan = lmg.Plan(gtab, N, uv0, prec)
    assert plan.info()["tile"] == 64
    g0 = plan.grid(v0)
    g1 = lmg.Plan(gtab, N, uv1, prec).grid(v1)
    both = lmg.BatchPlan(gtab, N, torch.cat([uv0, uv1]), [0, n, 3 * n + 7], prec)
    gb = both.grid(torch.cat([v0, v1]))
    assert torch.equal(gb[0], g0) and torch.equal(gb[1], g1)
    out = both.degrid(gb)
    assert torch.equal(out[:n], plan.degrid(g0))
    del gb, g1
    assert torch.equal(plan.grid_noalloc(v0), g0)
    assert torch.equal(plan.grid_ordered(plan.to_plan_order(v0)), g0)
    assert torch.equal(plan.grid(v0, out=g0.clone(), accumulate=True), 2 * g0)


@pytest.mark.parametrize("prec,W,n", [(lmg.F32_KAHAN, 7, 800), (lmg.F64, 4, 3000)])
def test_sparse_grids_and_images(prec, W, n):
    """Grid, degridding, dirty image and prediction of few visibilities (their patches numbered by entry), against the
    oracle's grid and degridding with torch's transforms in FP64, at the usual tolerances (1e-5, FP64 1e-12)."""
    print(f"sparse quadrants prec={prec} W={W}", flush=True)
    otab, gtab = table(W)
    uv, vis, uvd, vd = inputs(n, 9, prec)
    uv[:40] = np.random.default_rng(4).uniform(-4096, -4050, (40, 2))           # footprints that wrap
    uvd = torch.from_numpy(uv).to(DEV)
    plan = lmg.Plan(gtab, N, uvd, prec)
    h = torch.from_numpy(np.asarray(gtab.correction(N))).to(DEV)[N // 4:3 * N // 4]
    want = torch.from_numpy(im.grid(uv, vis, None, N, otab)).to(DEV)
    close = lambda a, b: (a.to(torch.complex128) - b).norm() < TOL[prec] * b.norm()     # noqa: E731
    assert close(plan.grid(vd), want)
    image = torch.fft.fftshift(torch.fft.ifft2(torch.fft.ifftshift(want), norm="forward"))
    image = image[N // 4:3 * N // 4, N // 4:3 * N // 4] * h[:, None] * h[None, :]
    assert close(plan.make_dirty_image(vd), image)
    model = image / image.abs().max()
    G = torch.zeros(N, N, dtype=torch.complex128, device=DEV)
    G[N // 4:3 * N // 4, N // 4:3 * N // 4] = model * h[:, None] * h[None, :]
    G = torch.fft.fftshift(torch.fft.fft2(torch.fft.ifftshift(G)))
    ref = torch.from_numpy(im.degrid(uv, G.cpu().numpy(), otab)).to(DEV)
    assert close(plan.predict_visibilities(model.to(ctype(prec))), ref)
    assert close(plan.degrid(G.to(ctype(prec))), ref)


@pytest.mark.parametrize("W", [6, 8])
def test_degridding_by_quadrants(W):
    """6,000,003 visibilities in FP64, which are degridded by quadrants, give the bits of the same visibilities in two plans
    of half as many, which are degridded by whole tiles."""
    print(f"degridding by quadrants W={W}", flush=True)
    n = 6_000_003
    gtab = lmg.Table.create(W, 0.25, 300, 3)
    g = torch.Generator(device=DEV).manual_seed(W)
    uv = torch.rand(n, 2, generator=g, device=DEV, dtype=torch.float64) * 8192 - 4096
    grid = torch.randn(N, N, generator=g, device=DEV, dtype=torch.complex128)
    out = lmg.Plan(gtab, N, uv, lmg.F64).degrid(grid)
    for a, b in ((0, n // 2), (n // 2, n)):
        assert torch.equal(out[a:b], lmg.Plan(gtab, N, uv[a:b].contiguous(), lmg.F64).degrid(grid))
