"""Repeated transforms of one length do not search for its factors again."""
import time

import pytest

torch = pytest.importorskip("torch")

from paper_2603_17166_amd import _lib

pytestmark = pytest.mark.gpu


def _host_us(n, calls=2000):
    """Host time of a call without rows: everything but the launch."""
    lib = _lib.load()
    stream = torch.cuda.current_stream().cuda_stream
    best = float("inf")
    for _ in range(5):
        t0 = time.perf_counter()
        for _ in range(calls):
            _lib.check(lib.psht_fft(n, 0, 1, 0, None, None, stream))
        best = min(best, (time.perf_counter() - t0) / calls * 1e6)
    return best


def test_host_time_does_not_depend_on_the_factors():
    torch.cuda.init()
    short, long = _host_us(8), _host_us(9360)   # 2^3 and 2^4 3^2 5 13
    print("host time per call: n = 8 %.2f us, n = 9360 %.2f us" % (short, long), flush=True)
    assert long <= 3 * short + 2


def test_unsupported_lengths_stay_refused():
    lib = _lib.load()
    for n in (17, 2 * 17, 10241):
        with pytest.raises(_lib.PshtError):
            _lib.check(lib.psht_fft(n, 0, 1, 0, None, None, None))
