"""LDS transforms of every radix (2 .. 11, 13; the composites 6, 8, 9, 10 for double
data) and at both sides of the length tiers, against numpy."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2603_17166_amd.plan import fft

pytestmark = pytest.mark.gpu

SINGLE = [1, 2, 3, 4, 5, 6, 7, 8, 9, 10, 11, 13]  # one pass
MIXED = [14, 16, 18, 64, 81, 90, 143, 156, 169, 182, 350, 512, 520, 1000, 1024, 1029, 1859, 2025, 2048, 2058, 2310, 2366,
         2430, 2560, 2574, 3744, 4050, 4095, 4096, 4116, 5376, 7203, 8192, 8232, 10000, 10240]


@pytest.mark.parametrize("fp32", [False, True])
@pytest.mark.parametrize("n", SINGLE + MIXED)
def test_lengths(n, fp32):
    rng = np.random.default_rng(n)
    x = rng.standard_normal((3, n)) + 1j * rng.standard_normal((3, n))
    xt = torch.as_tensor(x).to(torch.complex64 if fp32 else torch.complex128).cuda()
    ref = {-1: np.fft.fft(xt.cpu().numpy().astype(np.complex128), axis=1)}
    ref[1] = np.fft.ifft(xt.cpu().numpy().astype(np.complex128), axis=1) * n
    eps = 6e-8 if fp32 else 1.1e-16
    for sign in (-1, 1):
        y = fft(xt, sign).cpu().numpy()
        # a few roundings per factor of two; the twiddles of a pass are powers of
        # one entry, up to the 12th
        err = np.linalg.norm(y - ref[sign]) / np.linalg.norm(ref[sign])
        assert err < 8 * eps * (1 + np.log2(n)), (n, sign, err)
