"""Performance cases of the partial-sky transforms: calls that users of the library make, from a 20 000-point cap at
lmax 128 to the 21.6 M-point patch at lmax 4096, with the patch shapes, band limits, spins and tolerances of the
benchmark and the tests.

`prepare` draws the inputs on the GPU and builds the plan, which a user's program keeps; `run` is one pass through
the public entry points; `exact` is the direct sum over every coefficient and point (or every order, for the
rotation) in 64 bits, written from the definitions, for the cases small enough for it.
"""
import math

import torch

from paper_2603_17166_amd import autograd, rotate
from paper_2603_17166_amd.plan import Plan

DEG = math.pi / 180.0
ARCMIN = DEG / 60.0
JITTER = 2.5 * ARCMIN  # RMS deflection of lensed points

# RA/Dec rectangles (half width in RA, declination range, raster step in arcminutes) by name.
RECTS = {
    "rect1658": (50.0, -71.0, -41.0, 1.0),   # 5.98 M points
    "rect1501": (48.4, -70.0, -42.0, 0.5),   # 21.6 M points
    "rect999": (37.5, -70.0, -45.0, 1.0),    # 3.6 M points
}
RECT_AREA = {"rect1658": 1658.0, "rect1501": 1501.0, "rect999": 999.0}
RECT_RADIUS = {"rect1658": 35.3, "rect1501": 33.8, "rect999": 25.5}


def _disc(name, op, radius, npoints, lmax, spin, eps, nmaps=1):
    return {"name": name, "op": op, "patch": "disc", "radius": radius, "npoints": npoints, "lmax": lmax, "spin": spin,
            "eps": eps, "nmaps": nmaps}


def _rect(name, op, patch, lmax, spin, eps):
    return {"name": name, "op": op, "patch": patch, "radius": RECT_RADIUS[patch], "npoints": 0, "lmax": lmax,
            "spin": spin, "eps": eps, "nmaps": 1}


def listed():
    return [
        # the smallest call: a spin-0 map of a small cap, where launches and latency count
        _disc("cap10_l128_s0_fp64_synth", "synth", 10.0, 20000, 128, 0, 1e-10),
        # requests of the served mix (discs at 1', eps 1e-5 in the FP32 form), smallest to largest
        _disc("disc2_l512_s0_fp32_adjoint", "adjoint", 2.0, 45234, 512, 0, 1e-5),
        _disc("disc5_l1024_s2_fp32_synth", "synth", 5.0, 282563, 1024, 2, 1e-5),
        _disc("disc10_l2048_s0_fp32_synth", "synth", 10.0, 1128103, 2048, 0, 1e-5),
        _disc("disc20_l4096_s2_fp32_adjoint", "adjoint", 20.0, 4478132, 4096, 2, 1e-5),
        # eight requests of one kind in one call (the server's batches, simulations of one field)
        _disc("disc5_l2048_s2_fp32_synth8", "synth", 5.0, 282563, 2048, 2, 1e-5, 8),
        # a deep field at the paper's tolerance: polarization data of a small patch brought to coefficients
        _disc("disc7_l4000_s2_eps7_adjoint", "adjoint", 7.0, 750001, 4000, 2, 1e-7),
        # polarization map of a wide survey patch, FP64
        _rect("rect1658_l2048_s2_fp64_synth", "synth", "rect1658", 2048, 2, 1e-10),
        # one gradient step of a fit of coefficients to a map: forward, loss and backward
        _rect("rect999_l3000_s2_fp64_grad", "grad", "rect999", 3000, 2, 1e-10),
        # the largest patch in the FP32 form, and in FP64 (synthesis and adjoint: one step of an iterative solver)
        _rect("rect1501_l4096_s2_fp32_synth", "synth", "rect1501", 4096, 2, 1e-5),
        _rect("rect1501_l4096_s2_fp64_step", "step", "rect1501", 4096, 2, 1e-10),
        # coefficients of a polarization field moved into the patch frame
        {"name": "rotate_l1024", "op": "rotate", "lmax": 1024, "ncomp": 2, "theta_c": 143.5, "phi_c": 31.0},
    ]


def draw(rng):
    def spread(lo, hi):
        return math.exp(rng.uniform(math.log(lo), math.log(hi)))

    if rng.random() < 0.1:
        return {"op": "rotate", "lmax": int(spread(64, 1024.99)), "ncomp": rng.choice((1, 2)),
                "theta_c": round(rng.uniform(20.0, 160.0), 2), "phi_c": round(rng.uniform(0.0, 360.0), 2)}
    lmax = int(spread(96, 4096.99))
    op = rng.choice(("synth", "synth", "adjoint", "adjoint", "grad", "step"))
    nmaps = rng.choice((2, 3, 5, 8)) if op in ("synth", "adjoint") and lmax <= 2048 and rng.random() < 0.2 else 1
    return {"op": op, "patch": "disc", "radius": round(spread(2.0, 34.0), 3),
            "npoints": int(spread(2000, 8e6 if nmaps == 1 else 1e6)), "lmax": lmax,
            "spin": rng.choice((0, 0, 1, 2, 2, 2, 3)), "eps": rng.choice((1e-5, 1e-5, 1e-7, 1e-10, 1e-10)),
            "nmaps": nmaps}


# ------------------------------------------------------------------ inputs


def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed) * 2 + 1)


def _randn(gen, *shape):
    return torch.randn(shape, generator=gen, dtype=torch.float64, device="cuda")


def _unit(theta, phi):
    st = torch.sin(theta)
    return torch.stack([st * torch.cos(phi), st * torch.sin(phi), torch.cos(theta)])


def _angles(v):
    return torch.atan2(torch.hypot(v[0], v[1]), v[2]), torch.remainder(torch.atan2(v[1], v[0]), 2 * math.pi)


def _raster(first, step, count):
    """Row-major raster: row i holds count[i] points first[i], first[i] + step[i], ..."""
    row = torch.repeat_interleave(torch.arange(count.numel(), device="cuda"), count)
    k = torch.arange(row.numel(), device="cuda") - (torch.cumsum(count, 0) - count)[row]
    return row, first[row] + k * step[row]


def _jitter(theta, phi, gen):
    """Every point displaced along a geodesic by a Gaussian deflection of RMS JITTER; unit vectors."""
    dt, dp = _randn(gen, 2, theta.numel()) * (JITTER / math.sqrt(2.0))
    ct, st, cp, sp = torch.cos(theta), torch.sin(theta), torch.cos(phi), torch.sin(phi)
    a = torch.hypot(dt, dp)
    sinc = torch.sinc(a / math.pi)
    ca = torch.cos(a)
    return torch.stack([ca * st * cp + sinc * (dt * ct * cp - dp * sp), ca * st * sp + sinc * (dt * ct * sp + dp * cp),
                        ca * ct - sinc * dt * st])


def _points(case, gen):
    """(theta, phi) in the patch frame: a jittered raster of a polar disc, or of an RA/Dec rectangle turned so that
    the centre of the smallest cap around it lies on the pole."""
    if case["patch"] == "disc":
        rad = case["radius"] * DEG
        res = math.sqrt(2 * math.pi * (1 - math.cos(rad)) / case["npoints"])
        th = torch.arange(0.5 * res, rad, res, dtype=torch.float64, device="cuda")
        count = torch.clamp(torch.round(2 * math.pi * torch.sin(th) / res).long(), min=1)
        row, ph = _raster(torch.zeros_like(th), 2 * math.pi / count, count)
        return _angles(_jitter(th[row], ph, gen))
    half, d0, d1, res = RECTS[case["patch"]]
    dec = torch.arange(d0 * DEG, d1 * DEG + 0.5 * res * ARCMIN, res * ARCMIN, dtype=torch.float64, device="cuda")
    step = res * ARCMIN / torch.cos(dec)
    count = ((2 * half * DEG + 0.5 * step) / step).ceil().long()
    row, ra = _raster(torch.full_like(dec, -half * DEG), step, count)
    v = _jitter(0.5 * math.pi - dec[row], ra, gen)
    # the centre (at RA 0) nearest to the two corners that face the equator, the points farthest from it
    psi = 0.5 * math.pi - math.atan(math.tan(d1 * DEG) / math.cos(half * DEG))
    x = v[0] * math.cos(psi) - v[2] * math.sin(psi)
    z = v[0] * math.sin(psi) + v[2] * math.cos(psi)
    return _angles(torch.stack([x, v[1], z]))


def _m_l(lmax):
    """(m, l) of every coefficient, m-major."""
    mm = torch.arange(lmax + 1, device="cuda")
    m = torch.repeat_interleave(mm, lmax + 1 - mm)
    return m, torch.arange(m.numel(), device="cuda") - m * (2 * lmax + 1 - m) // 2


def _alm(lmax, spin, n, gen):
    """n coefficient arrays with E|a_lm|^2 = (l + 1)^-2, real at m = 0, zero below the spin."""
    m, l = _m_l(lmax)
    z = _randn(gen, 2, n, m.numel())
    a = torch.complex(z[0], z[1]) / math.sqrt(2.0)
    a = torch.where(m == 0, torch.complex(z[0], torch.zeros_like(z[0])), a)
    return a / (l + 1.0) * (l >= spin)


def _inputs(case, seed):
    """Everything of a case that is drawn: points, coefficients and maps (the maps in the plan's precision)."""
    gen = _gen(seed)
    if case["op"] == "rotate":
        return {"alm": _alm(case["lmax"], 0, case["ncomp"], gen)}
    theta, phi = _points(case, gen)
    nm, n, lmax = case["nmaps"], theta.numel(), case["lmax"]
    got = {"theta": theta, "phi": phi}
    if case["op"] != "adjoint":
        a = _alm(lmax, case["spin"], 2 * nm, gen).reshape(nm, 2, -1)
        got["alm"] = a if nm > 1 else a[0]
    if case["op"] != "synth":
        z = _randn(gen, 2, nm, n)
        f = torch.complex(z[0], z[1]).to(torch.complex64 if case["eps"] >= 1e-6 else torch.complex128)
        got["map"] = f if nm > 1 else f[0]
    return got


# -------------------------------------------------------------------- runs


def _frame(case):
    return rotate.patch_angles(case["theta_c"] * DEG, case["phi_c"] * DEG)


def prepare(case, seed):
    state = dict(_inputs(case, seed), case=case)
    if case["op"] != "rotate":
        # the plan keeps its own sorted copy of the points
        state["plan"] = Plan(state.pop("theta"), state.pop("phi"), case["lmax"], case["spin"], case["eps"])
        state["plan"].workspace(case["nmaps"])
    if case["op"] == "grad":
        state["alm"].requires_grad_(True)
    return state


def run(state):
    case, op = state["case"], state["case"]["op"]
    if op == "rotate":
        return rotate.rotate_alm(state["alm"], case["lmax"], *_frame(case))
    plan = state["plan"]
    if op == "synth":
        return plan.synth(state["alm"])
    if op == "adjoint":
        return plan.adjoint(state["map"])
    if op == "step":
        return plan.synth(state["alm"]), plan.adjoint(state["map"])
    f = autograd.synth(state["alm"], plan)
    r = torch.view_as_real(f - state["map"])
    loss = (r * r).sum()
    (grad,) = torch.autograd.grad(loss, state["alm"])
    return {"loss": loss.detach(), "map": f.detach(), "grad": grad}


def work(case):
    lmax = case["lmax"]
    nalm = (lmax + 1) * (lmax + 2) // 2
    if case["op"] == "rotate":
        # one recurrence and one accumulation per (l, m >= 0, m'); coefficients in and out
        steps = sum((l + 1) * (2 * l + 1) for l in range(lmax + 1))
        return {"bytes": 2 * 16 * case["ncomp"] * nalm, "flops": steps * (4 + 4 * case["ncomp"])}
    rad = case["radius"] * DEG
    n = case["npoints"] or RECT_AREA[case["patch"]] * DEG ** 2 / (RECTS[case["patch"]][3] * ARCMIN) ** 2
    width = math.ceil(-math.log10(case["eps"]) - 1e-9) + 1
    # Legendre terms inside the classical region of the cap's rings; interpolation or spreading per point
    terms = lmax ** 3 * (1 - math.cos(rad)) / (2 * math.pi)
    one = {"bytes": 2 * 16 * nalm + n * (16 + (8 if case["eps"] >= 1e-6 else 16)),
           "flops": terms * (16 if case["spin"] else 12) + n * 4 * width ** 2}
    times = case["nmaps"] * (2 if case["op"] in ("grad", "step") else 1)
    return {k: v * times for k, v in one.items()}


# ------------------------------------------------------------------- exact
#
# lambda+-_lm(theta) = sqrt((2l+1)/4 pi) d^l_{m,-+s}(theta) for every order and point at once, degree by degree:
#   l A_{l+1} d^{l+1} = (2l+1)(l(l+1) cos theta - m m') d^l - (l+1) A_l d^{l-1},  A_l = sqrt((l^2 - m^2)(l^2 - m'^2)).


def _wigner_rows(lmax, m, mp, theta):
    """Yields (l, d) for l = 0..lmax: d^l_{m m'}(theta) for the column tensors m >= 0 and m' (broadcast against the
    row theta), zero where l < max(m, |m'|)."""
    l0 = torch.maximum(m.abs(), mp.abs())
    big = m.abs() >= mp.abs()
    # the single term of the explicit sum at l0
    x = torch.where(big, mp, m)
    pc = torch.where(big, m + mp, torch.where(mp > 0, mp + m, l0 - m))
    ps = torch.where(big, m - mp, torch.where(mp > 0, mp - m, l0 + m))
    odd = torch.where(big, m - mp, torch.where(mp > 0, torch.zeros_like(m), m + l0)) % 2
    top = (2 * l0 + 1, l0 + x + 1, l0 - x + 1)
    lb = 0.5 * torch.lgamma(top[0].double()) - 0.5 * sum(torch.lgamma(t.double()) for t in top[1:])
    lc, ls = torch.log(torch.cos(theta / 2)), torch.log(torch.sin(theta / 2))
    seed = (1 - 2 * odd) * torch.exp(lb + torch.where(pc > 0, pc * lc, 0.0 * lc) + torch.where(ps > 0, ps * ls, 0.0))
    x = torch.cos(theta)
    cur, prev = torch.zeros_like(seed), torch.zeros_like(seed)
    m, mp = m.double(), mp.double()

    def amp(l):
        return torch.sqrt(torch.clamp((l * l - m * m) * (l * l - mp * mp), min=0.0))

    for l in range(lmax + 1):
        cur = torch.where(l0 == l, seed, cur)
        yield l, cur
        if l == 0:
            nxt = x * cur / torch.clamp(amp(1), min=1e-300)
        else:
            scale = 1.0 / torch.clamp(l * amp(l + 1), min=1e-300)
            nxt = (2 * l + 1) * scale * (l * (l + 1) * x - m * mp) * cur - (l + 1) * amp(l) * scale * prev
        prev, cur = cur, torch.where(l0 <= l, nxt, 0.0)


def _orders(case, theta):
    """Orders whose harmonics do not vanish (to far below rounding) on the patch."""
    lmax = case["lmax"]
    return torch.arange(min(lmax, int(1.2 * lmax * math.sin(min(theta.max().item(), 0.5 * math.pi))) + 64) + 1,
                        device="cuda")[:, None]


def _chunks(m, n):
    step = max(1, 12_000_000 // m.numel())
    return [slice(i, min(n, i + step)) for i in range(0, n, step)]


def _exact_synth(case, alm, theta, phi):
    lmax, s = case["lmax"], case["spin"]
    m, out = _orders(case, theta), []
    base = (m * (2 * lmax + 1 - m) // 2)[:, 0]
    g, c = alm[0].clone(), alm[1].clone()
    g[: lmax + 1], c[: lmax + 1] = g[: lmax + 1].real + 0j, c[: lmax + 1].real + 0j  # m = 0: real
    for q in _chunks(m, theta.numel()):
        th = theta[q][None, :]
        pos = torch.zeros((m.numel(), th.numel(), 2), dtype=torch.float64, device="cuda")
        neg = torch.zeros_like(pos)
        for (l, dp), (_, dm) in zip(_wigner_rows(lmax, m, torch.full_like(m, -s), th),
                                    _wigner_rows(lmax, m, torch.full_like(m, s), th)):
            if l < s:
                continue
            norm = math.sqrt((2 * l + 1) / (4 * math.pi))
            k = torch.clamp(base + l, max=g.numel() - 1)
            on = (m[:, 0] <= l).double() * norm
            a, b = (g[k] + 1j * c[k]) * on, (g[k].conj() + 1j * c[k].conj()) * on
            for acc, d, w in ((pos, dp, a), (neg, dm, b)):
                acc[..., 0].addcmul_(d, w.real[:, None])
                acc[..., 1].addcmul_(d, w.imag[:, None])
        turn = torch.exp(1j * (m * phi[q][None, :]))
        f = -(torch.view_as_complex(pos) * turn).sum(0)
        out.append(f - (-1) ** s * (torch.view_as_complex(neg)[1:] * turn[1:].conj()).sum(0))
    return torch.cat(out)


def _exact_adjoint(case, fmap, theta, phi):
    lmax, s = case["lmax"], case["spin"]
    m = _orders(case, theta)
    base = (m * (2 * lmax + 1 - m) // 2)[:, 0]
    out = torch.zeros((2, (lmax + 1) * (lmax + 2) // 2), dtype=torch.complex128, device="cuda")
    for q in _chunks(m, theta.numel()):
        th = theta[q][None, :]
        back = torch.exp(-1j * (m * phi[q][None, :]))
        u, v = torch.view_as_real(fmap[q][None, :] * back), torch.view_as_real(fmap[q].conj()[None, :] * back)
        for (l, dp), (_, dm) in zip(_wigner_rows(lmax, m, torch.full_like(m, -s), th),
                                    _wigner_rows(lmax, m, torch.full_like(m, s), th)):
            if l < s:
                continue
            norm = math.sqrt((2 * l + 1) / (4 * math.pi))
            a = norm * torch.view_as_complex(torch.stack([(dp * u[..., i]).sum(1) for i in (0, 1)], -1))
            b = norm * (-1) ** s * torch.view_as_complex(torch.stack([(dm * v[..., i]).sum(1) for i in (0, 1)], -1))
            n = min(l, m.numel() - 1) + 1
            out[0, base[:n] + l] += -0.5 * (a + b)[:n]
            out[1, base[:n] + l] += 0.5j * (a - b)[:n]
    out[:, : lmax + 1].imag.zero_()
    return out


def _exact_rotate(case, alm):
    lmax, (alpha, beta, gamma) = case["lmax"], _frame(case)
    m = torch.arange(lmax + 1, device="cuda")[:, None]
    mp = torch.arange(-lmax, lmax + 1, device="cuda")[None, :]
    base = (m * (2 * lmax + 1 - m) // 2)[:, 0]
    k = mp[0].abs()
    sign = torch.where((mp[0] < 0) & (k % 2 == 1), -1.0, 1.0)
    turn_in, turn_out = torch.exp(-1j * gamma * mp[0].double()), torch.exp(-1j * alpha * m[:, 0].double())
    out = torch.zeros_like(alm)
    # d^l_{m m'}(beta) for beta < 0 is that of |beta| times (-1)^(m - m')
    flip = torch.where(((m - mp) % 2 == 1) & (beta < 0), -1.0, 1.0)
    theta = torch.full((1, 1), abs(beta), dtype=torch.float64, device="cuda")
    for l, d in _wigner_rows(lmax, m.expand(-1, 2 * lmax + 1), mp.expand(lmax + 1, -1), theta):
        a = alm[:, torch.clamp(base[k] + l, max=alm.shape[1] - 1)] * (k <= l)
        a = sign * torch.where(mp[0] < 0, a.conj(), a)
        a = torch.where(k == 0, a.real + 0j, a) * turn_in
        r = (d * flip)[: l + 1].to(torch.complex128) @ a.T
        out[:, base[: l + 1] + l] = (r * turn_out[: l + 1, None]).T
    return out


def exact(case, seed):
    lmax = case["lmax"]
    if case["op"] == "rotate":  # above lmax 800 the seeds of some pairs of orders leave the double range
        return _exact_rotate(case, _inputs(case, seed)["alm"]) if lmax <= 800 else None
    # about 20 passes over (orders x points) doubles per degree: a few seconds at most; lmax <= 1024 keeps the
    # seeds of every order that matters inside the double range
    rad = min(case["radius"] * DEG + JITTER, 0.5 * math.pi)
    cost = case["npoints"] * (1.2 * lmax * math.sin(rad) + 64) * lmax * case["nmaps"]
    if case["patch"] != "disc" or lmax > 1024 or cost > (3.0e10 if case["op"] in ("grad", "step") else 6.0e10):
        return None
    d = _inputs(case, seed)
    theta, phi, op = d["theta"], d["phi"], case["op"]

    def each(fn, x):
        x = x.to(torch.complex128)
        return torch.stack([fn(case, y, theta, phi) for y in x]) if case["nmaps"] > 1 else fn(case, x, theta, phi)

    if op == "synth":
        return each(_exact_synth, d["alm"])
    if op == "adjoint":
        return each(_exact_adjoint, d["map"])
    f = each(_exact_synth, d["alm"])
    if op == "step":
        return f, each(_exact_adjoint, d["map"])
    r = f - d["map"].to(torch.complex128)
    twice = torch.full(((lmax + 1) * (lmax + 2) // 2,), 2.0, dtype=torch.float64, device="cuda")
    twice[: lmax + 1] = 1.0  # the gradient of an order m >= 1 counts the pair (m, -m)
    return {"loss": torch.view_as_real(r).square().sum(), "map": f, "grad": twice * each(_exact_adjoint, 2.0 * r)}
