"""Rotation of coefficients at the edges of its tiles (16 values of |m'| and 64
orders per workgroup, sums flushed every 8 degrees) against the oracle, and its
scratch use at the smallest band limits."""
import ctypes
import math

import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle
from paper_2603_17166_amd import _lib
from paper_2603_17166_amd import rotate as rot
from paper_2603_17166_amd import synthetic as syn

pytestmark = pytest.mark.gpu


def _alm(lmax, nc):
    a = syn.gaussian_alm(lmax, 0, 300 + lmax)[:nc].copy()
    m, _ = syn.alm_m_l(lmax)
    a[:, m == 0] = a[:, m == 0].real
    return a


@pytest.mark.parametrize("nc", [1, 2])
@pytest.mark.parametrize("lmax", [1, 2, 3, 4, 15, 16, 17, 63, 64, 65, 79])
def test_tile_edges(lmax, nc):
    a = _alm(lmax, nc)
    for ang in [(0.4, 0.9, -1.3), (1.0, math.pi, 0.5), (0.2, 1e-4, 2.0), (3.0, -2.2, 0.1)]:
        got = rot.rotate_alm(torch.as_tensor(a).cuda(), lmax, *ang).cpu().numpy()
        ref = oracle.rotate_alm(a, lmax, *ang)
        # the bar of the rotation tests: 1e-12 of the largest coefficient
        assert np.max(np.abs(got - ref)) <= 1e-12 * np.max(np.abs(ref)), (lmax, nc, ang)


@pytest.mark.parametrize("nc", [1, 2])
@pytest.mark.parametrize("lmax", [0, 1, 2, 3, 9])
def test_workspace_is_enough(lmax, nc):
    """The documented size, with bytes behind it that have to stay as they are."""
    lib = _lib.load()
    need = ctypes.c_size_t()
    _lib.check(lib.psht_rotate_alm_workspace(lmax, nc, ctypes.byref(need)))
    assert need.value == nc * (lmax + 1) * (2 * lmax + 1) * 16
    a = torch.as_tensor(_alm(lmax, nc)).cuda()
    out = torch.full_like(a, float("nan"))
    ws = torch.full((need.value + 4096,), 91, dtype=torch.uint8, device="cuda")
    _lib.check(lib.psht_rotate_alm(lmax, nc, 0.3, 1.2, -0.4, a.data_ptr(), out.data_ptr(), ws.data_ptr(), need.value,
                                   torch.cuda.current_stream().cuda_stream))
    torch.cuda.synchronize()
    assert bool((ws[need.value:] == 91).all())
    ref = oracle.rotate_alm(a.cpu().numpy(), lmax, 0.3, 1.2, -0.4)
    assert np.max(np.abs(out.cpu().numpy() - ref)) <= 1e-12 * np.max(np.abs(ref))


def test_non_finite_degree_stays_in_its_degree():
    lmax = 40
    a = torch.as_tensor(_alm(lmax, 1)).cuda()
    clean = rot.rotate_alm(a, lmax, 0.3, 1.2, -0.4)
    m, l = (torch.as_tensor(x).cuda() for x in syn.alm_m_l(lmax))
    a[0, (l == 17) & (m == 5)] = float("nan")
    got = rot.rotate_alm(a, lmax, 0.3, 1.2, -0.4)
    assert bool(torch.isfinite(torch.view_as_real(got[:, l != 17])).all())
    assert float((got[:, l != 17] - clean[:, l != 17]).abs().max()) <= 1e-12 * float(clean.abs().max())
