"""lmg_fft2_centred through the C ABI with the scratch that lmgrid.h documents: N x N elements and not a byte more."""
import numpy as np
import pytest

from conftest import rel_rms

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_1906_07102_amd as lmg  # noqa: E402


@pytest.mark.parametrize("prec", [lmg.F32, lmg.F64])
@pytest.mark.parametrize("N", [4, 8, 64, 512])
def test_scratch_of_the_documented_size(prec, N):
    """The scratch is the front of a larger buffer, whose rest must keep what it held; the transform is compared with
    numpy.fft at the tolerances of the other sizes (FP32 2e-6, FP64 1e-13), on two streams."""
    print(f"fft2 scratch prec={prec} N={N}", flush=True)
    cdt = torch.complex128 if prec == lmg.F64 else torch.complex64
    rng = np.random.default_rng(N)
    G = rng.standard_normal((N, N)) + 1j * rng.standard_normal((N, N))
    want = np.fft.fftshift(np.fft.fft2(np.fft.ifftshift(G)))
    for stream in (torch.cuda.current_stream(), torch.cuda.Stream()):
        stream.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(stream):
            d = torch.from_numpy(G).to("cuda:0", cdt)
            buf = torch.full((N * N + 4 * N + 64,), 7.5, dtype=cdt, device="cuda:0")
            st = lmg.load().lmg_fft2_centred(N, prec, -1, d.data_ptr(), buf.data_ptr(), stream.cuda_stream)
            assert st == 0
            stream.synchronize()
            assert bool((buf[N * N:] == 7.5).all())
            assert rel_rms(d.cpu().numpy(), want) < (1e-13 if prec == lmg.F64 else 2e-6)
