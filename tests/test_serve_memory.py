"""Admission estimate of the memory a plan holds against plans of different
sizes: the recurrence states are most of it."""
import math

import pytest

torch = pytest.importorskip("torch")

from paper_2603_17166_amd import synthetic as syn
from paper_2603_17166_amd.serve import PlanKey, TorchExecutor, legendre_state_bytes


@pytest.mark.parametrize("spin,size", [(0, 16), (2, 32)])
def test_state_estimate_counts_every_order(spin, size):
    """At least one state per ring and order up to lmax sin(theta)."""
    from paper_2603_17166_amd.plan import plan_geometry

    for lmax in (0 + spin, 64, 2048):
        for deg in (1.0, 5.0, 20.0, 35.0):
            info = plan_geometry(lmax, spin, deg * math.pi / 180, 1e-10, "fp64", rings=False)[0]
            step = 2 * info["theta_max"] / info["n2"]
            least = sum(int(lmax * math.sin(step * j)) + 1 for j in range(info["Lmax"] + 1))
            assert legendre_state_bytes(info) >= size * least


@pytest.mark.gpu
@pytest.mark.parametrize("lmax,spin,deg,eps", [(128, 0, 10.0, 1e-10), (1024, 2, 1.0, 1e-5), (2048, 0, 10.0, 1e-5),
                                               (3000, 2, 18.0, 1e-10), (4096, 2, 20.0, 1e-5), (4096, 2, 34.0, 1e-5),
                                               (1500, 2, 65.0, 1e-10), (2048, 200, 30.0, 1e-10)])
def test_estimate_covers_what_a_plan_holds(lmax, spin, deg, eps):
    ex = TorchExecutor(n_slots=1)
    th, ph = syn.uniform_cap(2000, deg * math.pi / 180, 17000 + lmax)
    ex.add_patch("p", torch.as_tensor(th).cuda(), torch.as_tensor(ph).cuda())
    key = PlanKey("p", lmax, spin, eps, "auto")
    plan, own, _, shared = ex.create_plan(key)
    est = ex.plan_bytes_estimate(key)
    print("lmax %d spin %d %g deg: holds %.1f + %.1f MB, estimate %.1f MB" % (lmax, spin, deg, own / 1e6, shared / 1e6,
                                                                          est / 1e6), flush=True)
    # not below what it holds, and not more than half above its own part but for the table allowance
    assert own + shared <= est <= 1.6 * own + 1.01 * shared + (3 << 20)
    plan.close()
