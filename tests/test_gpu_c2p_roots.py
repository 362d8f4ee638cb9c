"""Primitive recovery of given normalised states in flat space (D = 1, so that
the master function's coefficients are the inputs themselves), on the GPU:
states whose function has no finite value at the lower end of the bracket, and
the accuracy of the root at any field strength."""
import math
from decimal import Decimal as Dec

import numpy as np
import pytest

from paper_2311_04989_amd import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def recover(S, tau, B, mhd, **params):
    """Primitives (rho, ut^i, p) and status of cells with D = 1 in flat space."""
    from paper_2311_04989_amd import z4c as Z
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    n = len(tau)
    print(f"c2p roots: {n} cells mhd {mhd} {params}", flush=True)
    mb = W.MatterBatch([W.MBlock(n, 1, 1, 4, 3, 0.5, (0.0, 0.0, 0.0))])
    cell = lambda kind, arr, f: mb.view(kind, arr, 0, f)[3, 3, 3:3 + n]  # noqa: E731
    for f in range(7):
        mb.view("geom", mb.geom, 0, f)[...] = float(f in (0, 1, 4, 6))   # chi, gxx, gyy, gzz
    mb.view("cons", mb.cons, 0, 0)[...] = 1.0
    for f, v in enumerate([S[:, 0], S[:, 1], S[:, 2], tau, B[:, 0], B[:, 1], B[:, 2]]):
        cell("cons", mb.cons, 1 + f)[...] = v
    plan = Z.mplan_for(mb)
    dev = lambda a: torch.from_numpy(a.copy()).to("cuda:0")  # noqa: E731
    out, st = dev(np.zeros_like(mb.prim)), dev(np.full_like(mb.status, -1))
    plan.c2p(Z.c2p_params(mhd=mhd, gamma_ad=2.0, rho_atm=1e-12, **params), 0, dev(mb.geom),
             dev(mb.cons), out, st)
    torch.cuda.synchronize()
    plan.close()
    got = out.cpu().numpy()
    return (np.stack([cell("prim", got, f) for f in range(5)], axis=1),
            cell("status", st.cpu().numpy(), 0).copy())


X = np.array([1.0, 0.0, 0.0])


@pytest.mark.parametrize("S, tau, B, mhd", [
    (0 * X, 0.5, 1e160 * X, 1),           # b^2 beyond double
    (0 * X, 0.5, np.array([np.inf, 0.0, 0.0]), 1),
    (X, 0.5, 1e160 * X[::-1], 1),
    (1e200 * X, 1e200, 0 * X, 0),         # r^2 beyond double
    (1e200 * X, 1e200, 1e-3 * X, 1),
    (X, np.inf, 0 * X, 0),
    (X, np.inf, 1e-3 * X, 1)])
def test_states_beyond_double_become_atmosphere(S, tau, B, mhd):
    # g(0) = 0 D - 1 is no number: no sign change, status 3
    prim, st = recover(S[None], np.array([tau]), B[None], mhd)
    assert st[0] == 3
    assert prim[0, 0] == 1e-12 and (prim[0, 1:4] == 0.0).all()


def _g(mu, q, r2, b2, rb2, W=None):
    """g(mu) = mu D - 1 and W in 28 digits (adiabatic index 2, below the ceiling)."""
    x = 1 / (1 + mu * b2)
    rb = r2 * x * x + mu * x * (1 + x) * rb2
    qb = q - b2 / 2 - mu * mu * x * x * (b2 * r2 - rb2) / 2
    W = 1 / (1 - mu * mu * rb).sqrt()
    return mu * ((1 + 2 * max(W * (qb - mu * rb + 1) - 1, Dec(0))) / W + mu * rb) - 1, W


def _states(seed, wmax, mag):
    """Seeded D = 1 states with h = 1 .. 21, W = 1 .. wmax, b^2 / rho in `mag`, whose S
    and B have 12 bits (their squares and products are exact), tau on a root."""
    rng = np.random.default_rng(W.SEED_BASE + seed)
    cut = lambda v: float(np.ldexp(np.round(np.ldexp(np.frexp(v)[0], 12)), np.frexp(v)[1] - 12))  # noqa: E731
    out = []
    while len(out) < 200:
        Wl, h = 1.0 + (wmax - 1.0) * rng.uniform() ** 2, 1.0 + 2.0 * 10.0 ** rng.uniform(-2, 1)
        b2, c = 10.0 ** rng.uniform(*mag), rng.uniform(-1, 1)
        v = math.sqrt(1 - Wl ** -2)
        B2 = b2 * Wl ** 2 / (1 + (Wl * v * c) ** 2)      # b^2 W^2 = B^2 + (W v B c)^2
        Bx, By = math.sqrt(B2) * c, math.sqrt(B2 * (1 - c * c))
        # S = ((h + b^2) W^2 - (alpha b^0)^2) v - alpha b^0 B / W, rho = 1 / W
        k, ab = (h + b2) * Wl ** 2 - (Wl * v * Bx) ** 2, v * Bx
        s = np.array([k * v - ab * Bx, -ab * By]) / Wl
        s, B = [cut(t) for t in s], [cut(t / math.sqrt(Wl)) for t in (Bx, By)]
        r2, b2, rb2 = (Dec(s[0]) ** 2 + Dec(s[1]) ** 2, Dec(B[0]) ** 2 + Dec(B[1]) ** 2,
                       (Dec(s[0]) * Dec(B[0]) + Dec(s[1]) * Dec(B[1])) ** 2)
        mu = Dec(1 / (h * Wl))
        x = 1 / (1 + mu * b2)
        rb = r2 * x * x + mu * x * (1 + x) * rb2
        if not mu * mu * rb < Dec("0.99"):
            continue
        W_ = 1 / (1 - mu * mu * rb).sqrt()
        eps = ((1 / mu - mu * rb) * W_ - 1) / 2
        if eps < Dec("0.001"):
            continue
        tau = float((eps + 1) / W_ - 1 + mu * rb + b2 / 2 + mu * mu * x * x * (b2 * r2 - rb2) / 2)
        lo, hi = mu * Dec("0.999"), mu * Dec("1.001")
        args = (Dec(tau), r2, b2, rb2)
        if not _g(lo, *args)[0] < 0 < _g(hi, *args)[0]:
            continue
        for _ in range(110):
            m = (lo + hi) / 2
            lo, hi = (m, hi) if _g(m, *args)[0] < 0 else (lo, m)
        d = lo * Dec("1e-15")
        (ga, Wa), (gb, Wb) = _g(lo - d, *args), _g(lo + d, *args)
        out.append((s, tau, B, _g(lo, *args)[1], float((gb - ga) / (2 * d) * lo),
                    float((Wb - Wa) / (2 * d) * lo / Wa)))
    return out


@pytest.mark.parametrize("wmax, mag", [(3.0, (0, 1)), (3.0, (2, 3)), (3.0, (4, 4)), (3.0, (6, 6)),
                                       (10.0, (0, 4))])
def test_root_is_exact_to_rounding_at_any_field_strength(wmax, mag):
    # Of one evaluation of g near the root, a few roundings of half an ulp (rms
    # 2^-53 in sum) move mu by that over mu g', and mu itself is rounded; W
    # follows by L = d ln W / d ln mu, and by W^2 from the rounding of v^2.
    st = _states(71, wmax, mag)
    S = np.array([[*s, 0.0] for s, *_ in st])
    B = np.array([[*b, 0.0] for _, _, b, *_ in st])
    prim, status = recover(S, np.array([t for _, t, *_ in st]), B, 1, ut_max=1e3)
    assert (status == 0).all()
    r = [float((1 / Dec(float(p[0]))) / Wr - 1) / (2.0 ** -53 * ((1 / slope + 1) * abs(L) + float(Wr) ** 2))
         for p, (_, _, _, Wr, slope, L) in zip(prim, st)]
    print(f"W to {wmax}, b^2/rho 10^{mag}: rms {np.sqrt(np.mean(np.square(r))):.3f} of the bound, "
          f"max {np.abs(r).max():.3f}")
    assert np.sqrt(np.mean(np.square(r))) <= 1.0
