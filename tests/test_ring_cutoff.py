"""Polar cut-off of the orders per ring (host only): beyond a ring's cut-off no
order contributes more than the plan's threshold, also at spins next to lmax,
where the significant orders are a narrow band around s cos(theta)."""
import math

import numpy as np
import pytest

from paper_2603_17166_amd.plan import legendre_column, plan_geometry

DEG = math.pi / 180


@pytest.mark.parametrize("lmax,spin,deg", [(128, 100, 20.0), (64, 50, 20.0), (64, 60, 20.0), (64, 64, 30.0),
                                           (96, 95, 5.0), (128, 40, 20.0), (128, 2, 20.0), (128, 0, 20.0)])
def test_nothing_significant_beyond_the_cutoff(lmax, spin, deg):
    eps = 1e-10
    info, th, w, cut = plan_geometry(lmax, spin, deg * DEG, eps, "fp64")
    assert info["mmax"] == cut.max()
    for j in range(len(th)):
        for m in range(int(cut[j]) + 1, lmax + 1):
            lp, lm = legendre_column(lmax, spin, m, th[j])
            assert max(np.max(np.abs(lp)), np.max(np.abs(lm))) < eps, (j, m, int(cut[j]))


@pytest.mark.parametrize("lmax,spin", [(64, 50), (64, 60), (96, 95)])
def test_full_sky_rings(lmax, spin):
    info, th, w, cut = plan_geometry(lmax, spin, math.pi, 1e-10, "fp64", full_sky=True)
    for j in range(0, len(th), 3):
        for m in range(int(cut[j]) + 1, lmax + 1):
            lp, lm = legendre_column(lmax, spin, m, th[j])
            assert max(np.max(np.abs(lp)), np.max(np.abs(lm))) < 1e-10, (j, m, int(cut[j]))


@pytest.mark.gpu
@pytest.mark.parametrize("lmax,spin,deg", [(128, 100, 20.0), (256, 255, 20.0), (256, 64, 5.0),
                                           (331, 38, 1.1)])
def test_transforms_at_high_spin(lmax, spin, deg):
    import torch

    import oracle
    from paper_2603_17166_amd import synthetic as syn
    from paper_2603_17166_amd.plan import Plan

    eps = 1e-10
    th, ph = syn.uniform_cap(400, deg * DEG, 18000 + lmax)
    p = Plan(th, ph, lmax, spin, eps, "fp64")
    a = syn.gaussian_alm(lmax, spin, 18100)
    ref = oracle.synth(a, th, ph, lmax, spin)
    f = p.synth(torch.as_tensor(a).cuda())
    e1 = np.linalg.norm(f.cpu().numpy() - ref) / np.linalg.norm(ref)
    aref = oracle.adjoint(ref, th, ph, lmax, spin)
    d = p.adjoint(torch.as_tensor(ref).cuda()).cpu().numpy() - aref
    e2 = math.sqrt(oracle.alm_dot(d, d, lmax) / oracle.alm_dot(aref, aref, lmax))
    print("lmax %d spin %d: synth %.2e adjoint %.2e" % (lmax, spin, e1, e2), flush=True)
    assert e1 <= 10 * eps and e2 <= 10 * eps
    p.close()
