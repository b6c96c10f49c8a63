"""Workloads of the gridding / degridding path for timing, with 64-bit references.

A case is a dict of plain values: what is called (``kind``), the grid edge ``N``, the support ``W``, the interpolation
``degree`` of a 300-entry table, the precision (``f32``, ``kahan`` or ``f64``), the number of visibilities ``n`` and
where they lie (``tracks``: a 64-antenna array tracked over six hours, time-major; ``uniform``: scattered over the
central half of the grid); for batches also the number of channels, each with its own grid and visibility count.

kind            one pass
oneshot         make_dirty_image and predict_visibilities without a plan (what a script does once per data set)
step            a plan, a dirty image and a prediction from it (a new uv set: one integration of a streaming imager)
cycle           predict, subtract, image the residuals through a kept plan (one CLEAN major cycle)
image_grad      differentiable dirty image, forward and backward to visibilities and weights, through a kept plan
predict_grad    differentiable prediction, forward and backward to the image, through a kept plan
unit            gridding and degridding through a kept plan, data in the caller's order
ordered         gridding and degridding on data kept in the plan's order, results brought back to the caller's order
batch           gridding and degridding of many channels through one kept batched plan
batch_oneshot   grid_batched and degrid_batched without a plan
"""
import math

import numpy as np
import torch

import paper_1906_07102_amd as lmg

X0 = 0.25            # retained field |x| <= x0, as in the paper
TABLE = 300          # table entries, as in the paper
N_ANT = 64
BASELINES = N_ANT * (N_ANT - 1) // 2
TAU = 2.0 * math.pi

# ln h(x) of the least-misfit correcting function at x0 = 1/4, as the coefficients of (x / x0)^2, ^4, ... ^14 fitted to
# the optimiser's 33 samples; the integrated misfit is the optimum's to 11 digits.
LN_H = {
    3: (0.38017748033, 0.010061585041, 0.00068517526122, 7.1356281724e-05, -0.00011465618419, -1.4266435729e-05,
        -3.0577453144e-05),
    4: (0.5142548849, 0.014376559106, 0.00078714162285, 5.1921050255e-05, -1.2988052609e-05, 3.5791084839e-05,
        -1.9185882387e-05),
    5: (0.64786756708, 0.01809179404, 0.00099759802805, 7.304566822e-05, -2.143675074e-06, 6.3516963171e-06,
        -1.8196534911e-06),
    6: (0.79172823814, 0.02234077246, 0.0012342282938, 8.4775558709e-05, 6.5547047052e-06, 5.1082713889e-07,
        6.3477806418e-08),
    7: (0.93192854394, 0.02668757817, 0.0014895746322, 0.00010291573823, 7.9892986351e-06, 6.1675606129e-07,
        8.2277405331e-08),
    8: (1.0636973994, 0.030447534859, 0.0017055285721, 0.00011834764465, 9.2226294723e-06, 7.1359040412e-07,
        9.5715143085e-08),
}

PRECISION = {"f32": (lmg.F32, torch.complex64), "kahan": (lmg.F32_KAHAN, torch.complex64),
             "f64": (lmg.F64, torch.complex128)}


def _case(name, kind, N, W, prec, n, uv="tracks", degree=3, channels=1):
    return {"name": name, "kind": kind, "N": N, "W": W, "precision": prec, "n": n, "uv": uv, "degree": degree,
            "channels": channels}


def listed():
    return [
        # the smoke-sized call: 2,000 visibilities on 128^2, launches and host time
        _case("oneshot-2k-128-w7-f32", "oneshot", 128, 7, "f32", 2000, "uniform"),
        # a small interactive major cycle in double precision, an odd count
        _case("cycle-10k-256-w5-f64", "cycle", 256, 5, "f64", 10007, "uniform"),
        # a script's single call on a ragged set with an even support, compensated
        _case("oneshot-100k-512-w4-kahan", "oneshot", 512, 4, "kahan", 100003, "uniform"),
        # a snapshot of the array: 100 integrations, new uv each time
        _case("step-202k-1024-w7-f32", "step", 1024, 7, "f32", 100 * BASELINES),
        # gradients of an image loss on the 1,008,000-visibility observation at the support where FP32 is enough
        _case("imagegrad-1m-2048-w5-kahan", "image_grad", 2048, 5, "kahan", 500 * BASELINES),
        # the double-precision major cycle of a longer observation
        _case("cycle-4m-4096-w7-f64", "cycle", 4096, 7, "f64", 2081 * BASELINES),
        # plan-ordered data (iterative solvers), an even support, a ragged count
        _case("ordered-8m-4096-w6-f32", "ordered", 4096, 6, "f32", 4161 * BASELINES - 77),
        # the benchmark's workload: plan, dirty image, prediction
        _case("step-16m-4096-w7-f32", "step", 4096, 7, "f32", 8322 * BASELINES),
        # the same visibilities gridded and degridded through a kept plan
        _case("unit-16m-4096-w7-f32", "unit", 4096, 7, "f32", 8322 * BASELINES),
        # a 4096^2 image predicted and differentiated on the largest grid
        _case("predictgrad-16m-8192-w7-kahan", "predict_grad", 8192, 7, "kahan", 8322 * BASELINES),
        # spectral-line imaging: 256 channels of uneven counts, kept plan
        _case("batch-256x1024-w5-kahan", "batch", 1024, 5, "kahan", 15_800_000, channels=256),
        # a few channels in one call without a plan
        _case("batchonce-24x512-w5-f32", "batch_oneshot", 512, 5, "f32", 1_000_003, channels=24),
    ]


def draw(rng):
    """One more case of the ranges above. Counts are spread over their logarithm, supports over 3 .. 8."""
    kind = rng.choice(["oneshot", "step", "cycle", "image_grad", "predict_grad", "unit", "ordered", "batch",
                       "batch_oneshot"])
    W = rng.randint(3, 8)
    prec = rng.choice(["f32", "f32", "kahan", "f64"])
    uv = rng.choice(["tracks", "tracks", "uniform"])
    degree = rng.choice([3, 3, 3, 1])
    if kind in ("batch", "batch_oneshot"):
        N = rng.choice([256, 512, 1024])
        channels = int(round(math.exp(rng.uniform(math.log(4), math.log(64)))))
        lo, hi = 1000 * channels, 50_000 * channels
    else:
        N = rng.choice([128, 256, 512, 1024, 2048, 4096, 8192])
        channels = 1
        lo, hi = max(1000, N * N // 256), min(6_000_000, 2 * N * N)
    if prec == "f64":
        hi = min(hi, 3_000_000)
        lo = min(lo, hi)
    n = int(math.exp(rng.uniform(math.log(lo), math.log(hi))))
    c = _case("", kind, N, W, prec, n, uv, degree, channels)
    del c["name"]
    return c


# ------------------------------------------------------------------ the table
def _taps(W):
    """Tap positions t_j and the lower end of the offset interval."""
    ref = (W - 1) / 2.0 if W % 2 else W / 2.0 - 1.0
    return np.arange(W) - ref, (-0.5 if W % 2 else 0.0)


def _h_samples(W):
    x = np.arange(33) / 32.0
    return np.exp(sum(c * x ** (2 * k + 2) for k, c in enumerate(LN_H[W])))


def _kernel(h, W, delta):
    """C(t_j - delta), W x n: the normal equations on the 33 samples of h."""
    x = np.arange(33) * (X0 / 32)
    tau = np.full(33, X0 / 32)
    tau[0] *= 0.5
    tau[-1] *= 0.5
    t, _ = _taps(W)
    A = 2.0 * (np.cos(TAU * (t[:, None] - t[None, :])[:, :, None] * x) @ (tau * h * h))
    B = 2.0 * (np.cos(TAU * (t[:, None] - np.asarray(delta)[None, :])[:, :, None] * x) @ (tau * h))
    return np.linalg.solve(A, B)


def _nodes(W, degree):
    Ms = TABLE // W
    h = _h_samples(W)
    return h, Ms, _kernel(h, W, _taps(W)[1] + np.arange(Ms + 1 + degree) / Ms)


def _table(case):
    W, degree = case["W"], case["degree"]
    h, _, nodes = _nodes(W, degree)
    return lmg.Table.from_nodes(W, X0, TABLE, degree, h, nodes)


# ----------------------------------------------------------------- the inputs
def _counts(case):
    """Visibilities per channel: log-uniform over a factor of 20, the total as asked."""
    nch, n = case["channels"], case["n"]
    if nch == 1:
        return [n]
    g = np.exp(np.random.default_rng(nch).uniform(0.0, math.log(20.0), nch))
    edges = np.floor(np.concatenate([[0.0], np.cumsum(g) / g.sum()]) * n).astype(np.int64)
    edges[-1] = n
    return np.diff(edges).tolist()


def _tracks(n, wavelength, seed, dev):
    """n time-major (u, v) of a 64-antenna Gaussian array (sigma 1 km) over +-3 h at declination 45 degrees."""
    rng = np.random.default_rng(seed)
    east, north = rng.normal(0.0, 1000.0, N_ANT), rng.normal(0.0, 1000.0, N_ANT)
    lat, dec = math.radians(34.08), math.radians(45.0)
    X, Y, Z = -north * math.sin(lat), east, north * math.cos(lat)
    i, j = np.triu_indices(N_ANT, k=1)
    b = torch.as_tensor(np.stack([X[j] - X[i], Y[j] - Y[i], Z[j] - Z[i]]) / wavelength, device=dev)
    nt = -(-n // BASELINES)
    ha = (-3.0 + (torch.arange(nt, device=dev, dtype=torch.float64) + 0.5) * (6.0 / nt)) * (math.pi / 12.0)
    s, c = torch.sin(ha)[:, None], torch.cos(ha)[:, None]
    u = b[0] * s + b[1] * c
    v = -math.sin(dec) * c * b[0] + math.sin(dec) * s * b[1] + math.cos(dec) * b[2]
    return torch.stack([u, v], dim=-1).reshape(-1, 2)[:n]


def _uv(case, seed, dev):
    counts = _counts(case)
    nch = len(counts)
    if case["uv"] == "uniform":
        g = torch.Generator(device=dev).manual_seed(seed)
        q = case["N"] / 4.0
        return (torch.rand(case["n"], 2, generator=g, device=dev, dtype=torch.float64) * (2 * q) - q).contiguous()
    lam = [0.21 * (0.8 + 0.4 * c / max(1, nch - 1)) for c in range(nch)]
    uv = torch.cat([_tracks(m, l, seed, dev) for m, l in zip(counts, lam)])
    return (uv * ((case["N"] / 4.0 - case["W"]) / uv.abs().max())).contiguous()


def _inputs(case, seed):
    """uv in cells, a sky of 20 sources observed with noise, natural weights, an image with the sources."""
    dev = torch.device("cuda")
    N, n, M = case["N"], case["n"], int(2 * X0 * case["N"])
    dtype = PRECISION[case["precision"]][1]
    uv = _uv(case, seed, dev)
    rng = np.random.default_rng(seed)
    g = torch.Generator(device=dev).manual_seed(seed + 1)
    vis = 0.1 * torch.randn(n, generator=g, device=dev, dtype=torch.complex128)
    image = 0.01 * torch.randn(M, M, generator=g, device=dev, dtype=torch.complex128)
    for _ in range(20):
        p, q, f = int(rng.integers(-M // 2, M // 2)), int(rng.integers(-M // 2, M // 2)), float(rng.uniform(0.1, 1.0))
        ph = (uv[:, 0] * p + uv[:, 1] * q) * (-TAU / N)
        vis += f * torch.polar(torch.ones_like(ph), ph)
        image[q + M // 2, p + M // 2] += f
    weights = torch.rand(n, generator=g, device=dev, dtype=torch.float32) + 0.5
    upstream = None
    if case["kind"] == "image_grad":
        upstream = torch.randn(M, M, generator=g, device=dev, dtype=dtype)
    elif case["kind"] == "predict_grad":
        upstream = torch.randn(n, generator=g, device=dev, dtype=dtype)
    offsets = np.concatenate([[0], np.cumsum(_counts(case))]).astype(np.int64)
    return uv, vis.to(dtype), weights, image.to(dtype), upstream, offsets


def prepare(case, seed):
    prec, dtype = PRECISION[case["precision"]]
    uv, vis, weights, image, upstream, offsets = _inputs(case, seed)
    kind, N = case["kind"], case["N"]
    s = {"kind": kind, "N": N, "table": _table(case), "precision": prec, "kahan": case["precision"] == "kahan",
         "uv": uv, "vis": vis, "weights": weights, "offsets": offsets}
    if kind in ("oneshot", "cycle", "predict_grad"):
        s["image"] = image
    if upstream is not None:
        s["upstream"] = upstream
    if kind in ("cycle", "image_grad", "predict_grad", "unit", "ordered"):
        s["plan"] = lmg.Plan(s["table"], N, uv, prec)
    if kind == "batch":
        s["plan"] = lmg.BatchPlan(s["table"], N, uv, offsets, prec)
    if kind in ("unit", "ordered", "batch"):
        s["grid"] = torch.empty(s["plan"].grid_shape, dtype=dtype, device=uv.device)
    if kind == "ordered":
        s["vis_plan"] = s["plan"].to_plan_order(vis, weights)
        s["out_plan"] = torch.zeros_like(s["vis_plan"])
    return s


def run(s):
    kind, N = s["kind"], s["N"]
    if kind == "oneshot":
        image = lmg.make_dirty_image(s["table"], N, s["uv"], s["vis"], s["weights"], kahan=s["kahan"])
        return image, lmg.predict_visibilities(s["table"], N, s["uv"], s["image"])
    if kind == "step":
        plan = lmg.Plan(s["table"], N, s["uv"], s["precision"])
        image = plan.make_dirty_image(s["vis"], s["weights"])
        return image, plan.predict_visibilities(image)
    if kind == "cycle":
        model = s["plan"].predict_visibilities(s["image"])
        return model, s["plan"].make_dirty_image(s["vis"] - model, s["weights"])
    if kind == "image_grad":
        vis, weights = s["vis"].requires_grad_(), s["weights"].requires_grad_()
        image = lmg.MakeDirtyImage.apply(s["plan"], vis, weights)
        return (image.detach(), *torch.autograd.grad(image, (vis, weights), s["upstream"]))
    if kind == "predict_grad":
        image = s["image"].requires_grad_()
        vis = lmg.PredictVisibilities.apply(s["plan"], image)
        return (vis.detach(), *torch.autograd.grad(vis, image, s["upstream"]))
    if kind in ("unit", "batch"):
        grid = s["plan"].grid(s["vis"], s["weights"], out=s["grid"])
        return grid, s["plan"].degrid(grid)
    if kind == "ordered":
        grid = s["plan"].grid_ordered(s["vis_plan"], out=s["grid"])
        return grid, s["plan"].from_plan_order(s["plan"].degrid_ordered(grid, out=s["out_plan"]))
    grids = lmg.grid_batched(s["table"], N, s["uv"], s["offsets"], s["vis"], s["weights"], kahan=s["kahan"])
    return grids, lmg.degrid_batched(s["table"], N, s["uv"], s["offsets"], grids)


def work(case):
    """Coordinates, visibilities, weights and images or grids read and written once; the taps' and the transforms'
    operations (two pruned transforms of N / 2 rows each per image)."""
    n, N, W, kind = case["n"], case["N"], case["W"], case["kind"]
    c = 16 if case["precision"] == "f64" else 8
    M2, G2 = (2 * X0 * N) ** 2 * c, case["channels"] * N * N * c
    taps = n * (4.0 * W * W + 12 * W)
    fft = 5.0 * N * N * math.log2(N)
    vis = n * (16.0 + c)                                  # coordinates and values
    images = {"oneshot": 2, "step": 1, "cycle": 2, "image_grad": 2, "predict_grad": 2}.get(kind)
    values = {"oneshot": 1, "step": 1, "cycle": 1, "image_grad": 1, "predict_grad": 1, "unit": 1, "ordered": 1,
              "batch": 1, "batch_oneshot": 1}[kind] * n * c
    weights = {"image_grad": 8.0, "predict_grad": 0.0, "ordered": 0.0}.get(kind, 4.0) * n
    if images is None:
        return {"bytes": vis + values + weights + G2, "flops": 2 * taps}
    return {"bytes": vis + values + weights + images * M2, "flops": 2 * taps + 2 * fft}


# ------------------------------------------------------- 64-bit references
class _Reference:
    """Gridding, transforms and degridding of one uv set by their definitions, in complex128."""

    def __init__(self, case, uv):
        self.N, self.W = case["N"], case["W"]
        h, Ms, nodes = _nodes(self.W, case["degree"])
        self.h, self.Ms, self.degree = h, Ms, case["degree"]
        self.nodes = torch.as_tensor(nodes, device=uv.device)
        self.cell, self.weight = zip(*(self._axis(uv[:, a]) for a in (0, 1)))

    def _axis(self, u):
        first = torch.ceil(u - 0.5 * self.W)
        t, low = _taps(self.W)
        s = (u - first + t[0] - low) * self.Ms            # t_0 = -(offset of the reference tap)
        k = torch.floor(s)
        t, k = s - k, k.long()
        out, f = [], [self.nodes[:, k + i] for i in range(self.degree + 1)]
        acc, coef = f[0].clone(), torch.ones_like(t)
        for i in range(1, self.degree + 1):
            f = [b - a for a, b in zip(f, f[1:])]
            coef = coef * (t - (i - 1)) / i
            acc += coef * f[0]
        return first.long() + self.N // 2, acc

    def _index(self, r, c):
        N = self.N
        return ((self.cell[1] + r) % N) * N + (self.cell[0] + c) % N

    def grid(self, v):
        G = torch.zeros(2, self.N * self.N, dtype=torch.float64, device=v.device)
        for r in range(self.W):
            for c in range(self.W):
                x = v * (self.weight[1][r] * self.weight[0][c])
                i = self._index(r, c)
                G[0].index_add_(0, i, x.real.contiguous())
                G[1].index_add_(0, i, x.imag.contiguous())
        return torch.complex(G[0], G[1]).reshape(self.N, self.N)

    def degrid(self, G):
        G = G.reshape(-1)
        out = torch.zeros(len(self.cell[0]), dtype=torch.complex128, device=G.device)
        for r in range(self.W):
            for c in range(self.W):
                out += G[self._index(r, c)] * (self.weight[1][r] * self.weight[0][c])
        return out

    def correction(self, device):
        """h(x_p) on the retained pixels: the ratio of the kernel's first to its second moment over the offset."""
        M = int(2 * X0 * self.N)
        t, low = _taps(self.W)
        z, wz = np.polynomial.legendre.leggauss(64)
        d, wd = low + 0.5 * (z + 1.0), 0.5 * wz
        x = (np.arange(M) - M // 2) / self.N
        S = sum(C[:, None] * np.exp(1j * TAU * np.outer(tj - d, x)) for C, tj in zip(_kernel(self.h, self.W, d), t))
        return torch.as_tensor((wd @ S.real) / (wd @ np.abs(S) ** 2), device=device)

    def image(self, G):
        N, M = self.N, int(2 * X0 * self.N)
        F = torch.fft.fftshift(torch.fft.ifft2(torch.fft.ifftshift(G), norm="forward"))
        a, h = N // 2 - M // 2, self.correction(G.device)
        return F[a:a + M, a:a + M] * h[:, None] * h[None, :]

    def dirty(self, v):
        return self.image(self.grid(v))

    def predict(self, image):
        N, M = self.N, int(2 * X0 * self.N)
        a, h = N // 2 - M // 2, self.correction(image.device)
        G = torch.zeros(N, N, dtype=torch.complex128, device=image.device)
        G[a:a + M, a:a + M] = image * h[:, None] * h[None, :]
        return self.degrid(torch.fft.fftshift(torch.fft.fft2(torch.fft.ifftshift(G))))


def exact(case, seed):
    uv, vis, weights, image, upstream, offsets = _inputs(case, seed)
    kind = case["kind"]
    vis, image, w = vis.to(torch.complex128), image.to(torch.complex128), weights.double()
    if kind in ("batch", "batch_oneshot"):
        grids, out = [], []
        for a, b in zip(offsets[:-1], offsets[1:]):
            ref = _Reference(case, uv[a:b])
            grids.append(ref.grid(vis[a:b] * w[a:b]))
            out.append(ref.degrid(grids[-1]))
        return torch.stack(grids), torch.cat(out)
    ref = _Reference(case, uv)
    if kind == "oneshot":
        return ref.dirty(vis * w), ref.predict(image)
    if kind == "step":
        img = ref.dirty(vis * w)
        return img, ref.predict(img)
    if kind == "cycle":
        model = ref.predict(image)
        return model, ref.dirty((vis - model) * w)
    if kind == "image_grad":
        d = ref.predict(upstream.to(torch.complex128))
        return ref.dirty(vis * w), d * w, (vis.conj() * d).real
    if kind == "predict_grad":
        return ref.predict(image), ref.dirty(upstream.to(torch.complex128))
    grid = ref.grid(vis * w)
    return grid, ref.degrid(grid)
