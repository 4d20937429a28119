"""Accuracy of the coefficient rotation's recurrence: its factors G_l(x)
(csrc/rot_factor.h) against 128-bit arithmetic on the CPU, and on the GPU the
columns d^l_{m 0} (whose seeds are exact to a few units of roundoff) against
extended precision, no further off than the plain three-term recurrence."""
import math
import os
import subprocess

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
SRC = os.path.join(HERE, "rot_factor_check.cpp")
INC = os.path.join(ROOT, "paper_2603_17166_amd", "csrc")
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")


@pytest.fixture(scope="module")
def harness(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("rot") / "rot_factor_check")
    subprocess.run(["g++", "-O2", "-std=c++17", "-ffp-contract=off", "-D__HIP_PLATFORM_AMD__", "-I",
                    os.path.join(ROCM, "include"), "-I", INC, SRC, "-lquadmath", "-o", exe], check=True)
    return exe


@pytest.mark.parametrize("lmax", [1, 2, 7, 64, 1024, 4096, 16383])
def test_factors_are_correctly_rounded(harness, lmax):
    out = subprocess.run([harness, str(lmax)], check=True, capture_output=True, text=True).stdout.split()
    # half a unit in the last place of values that may lie just above a power of two
    assert int(out[1]) >= min(lmax, 64) and float(out[3]) <= 1.12e-16, out


def _columns(lmax, beta, dtype):
    """d^l_{m 0}(beta), m = 0..3, l = 0..lmax, by the plain recurrence in dtype."""
    one = dtype(1)
    cb, sb = np.cos(np.longdouble(beta)), np.sin(np.longdouble(beta))
    if dtype is np.float64:
        cb = np.float64(math.cos(beta))
    else:
        cb = np.longdouble(math.cos(beta))  # the argument the kernels work with
    d = np.zeros((4, lmax + 1), dtype=dtype)
    for m in range(4):
        binom = math.comb(2 * m, m)
        d[m, m] = dtype((-1) ** m * np.sqrt(np.longdouble(binom)) * (sb / 2) ** m)
        M = dtype(m)
        for l in range(m, lmax):
            L = dtype(l)
            a1, a0 = np.sqrt((L + one) ** 2 - M * M), np.sqrt(L * L - M * M)
            prev = a0 * d[m, l - 1] if l > m else dtype(0)
            d[m, l + 1] = ((2 * L + one) * cb * d[m, l] - prev) / a1
    return d


@pytest.mark.gpu
@pytest.mark.parametrize("beta", [1.1, 2.0, 2.6])
def test_recurrence_is_as_accurate_as_the_plain_one(beta):
    import torch

    from paper_2603_17166_amd import rotate as rot
    from paper_2603_17166_amd import synthetic as syn

    lmax = 4096
    a = np.zeros((1, syn.nalm(lmax)), dtype=np.complex128)
    a[0, :lmax + 1] = 1.0  # m' = 0
    got = rot.rotate_alm(torch.as_tensor(a).cuda(), lmax, 0.0, beta, 0.0).cpu().numpy()[0]
    ref, plain = _columns(lmax, beta, np.longdouble), _columns(lmax, beta, np.float64)
    worst = float(np.max(np.abs(plain - ref)))
    for m in range(4):
        at = np.arange(m, lmax + 1) + m * (2 * lmax + 1 - m) // 2
        err = float(np.max(np.abs(got[at].real - ref[m, m:])))
        print("beta %.1f m %d: error %.2e, plain recurrence %.2e" % (beta, m, err, worst), flush=True)
        # two such recurrences differ by their roundings; one unit for the seed
        assert err <= 2 * worst + 2.3e-16
