"""Primitive recovery at the ends of the range its Newton iteration covers, on
the GPU: cold gas (the root on the end of the bracket), gas nearly at rest,
nearly at the velocity ceiling, strongly magnetised, and a state that the
iteration limit cuts off (the bracketing fallback's status)."""
import numpy as np
import pytest

import oracle.c2p as OC
from paper_2311_04989_amd import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
SYM = [(0, 0), (0, 1), (0, 2), (1, 1), (1, 2), (2, 2)]

# largest W, largest b^2 / rho, range of log10(p / rho) (None: p = 0)
KINDS = {"cold": (3.0, 1e-2, None), "at rest": (1.0 + 1e-9, 1e-2, (-6.0, 0.0)),
         "fast": (19.0, 1.0, (-3.0, 1.0)), "magnetised": (3.0, 1e4, (-3.0, 1.0)),
         "plain": (2.0, 1.0, (-2.0, 0.0))}


def _case(kind, mhd, limit=100):
    """Recovers seeded states; yields (rho, ut, p, b2/rho, W, recovered, status)."""
    from paper_2311_04989_amd import z4c as Z
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print(f"c2p solver: {kind} mhd {mhd} limit {limit}", flush=True)
    wmax, mag, pr = KINDS[kind]
    mb = W.random_matter_batch(70 + mhd, nblocks=1, nmax=6)
    rng = np.random.default_rng(W.SEED_BASE + 70)
    W.c2p_states(mb, rng, wmax=wmax, mag=mag)
    rho, p = mb.view("prim", mb.prim, 0, 0), mb.view("prim", mb.prim, 0, 4)
    p[...] = 0.0 if pr is None else rho * 10.0 ** rng.uniform(*pr, size=rho.shape)
    if not mhd:
        for f in (5, 6, 7):
            mb.view("prim", mb.prim, 0, f)[...] = 0.0
    gam = np.zeros(rho.shape + (3, 3))
    for q, (a, c) in enumerate(SYM):
        gam[..., a, c] = gam[..., c, a] = (mb.view("geom", mb.geom, 0, 1 + q)
                                          / np.maximum(mb.view("geom", mb.geom, 0, 0), 1e-6))
    cells = list(np.ndindex(rho.shape))
    prim = [mb.view("prim", mb.prim, 0, f) for f in range(8)]
    for i in cells:
        D, S, tau, B = OC.p2c(prim[0][i], np.array([prim[f][i] for f in (1, 2, 3)]), prim[4][i],
                              np.array([prim[f][i] for f in (5, 6, 7)]), gam[i], 2.0)
        for f, v in enumerate([D, *S, tau, *B]):
            mb.view("cons", mb.cons, 0, f)[i] = v
    plan = Z.mplan_for(mb)
    dev = lambda a: torch.from_numpy(a.copy()).to("cuda:0")  # noqa: E731
    out, st = dev(np.zeros_like(mb.prim)), dev(np.full_like(mb.status, -1))
    plan.c2p(Z.c2p_params(mhd=mhd, gamma_ad=2.0, rho_atm=1e-12, max_iter=limit), 3, dev(mb.geom),
             dev(mb.cons), out, st)
    torch.cuda.synchronize()
    plan.close()
    got, st = out.cpu().numpy(), mb.view("status", st.cpu().numpy(), 0, 0)
    for i in cells:
        ut = np.array([prim[f][i] for f in (1, 2, 3)])
        B = np.array([prim[f][i] for f in (5, 6, 7)])
        Wl = np.sqrt(1.0 + ut @ gam[i] @ ut)
        b2 = ((ut @ gam[i] @ B) ** 2 + B @ gam[i] @ B) / Wl ** 2
        yield (prim[0][i], ut, prim[4][i], b2 / prim[0][i], Wl,
               [mb.view("prim", got, 0, f)[i] for f in range(5)], st[i])


@pytest.mark.parametrize("mhd", [0, 1])
@pytest.mark.parametrize("kind", list(KINDS))
def test_recovers_states(kind, mhd):
    # The conservatives hold the energy (rho h + b^2) W^2 to half an ulp; per
    # unit of D that is (h + b^2 / rho) W, and the inversion amplifies an error
    # of the velocity by W^2 into W.  64 roundings of that size are allowed.
    for rho, ut, p, m, Wl, got, st in _case(kind, mhd):
        h = 1.0 + 2.0 * p / rho
        tol = 64 * 2.0 ** -53 * (h + m) * Wl ** 3
        assert st == 0, (rho, ut, p, m, st)
        assert abs(got[0] - rho) <= tol * rho, (rho, got[0], tol)
        assert np.abs(np.array(got[1:4]) - ut).max() <= tol * max(1.0, np.abs(ut).max())
        assert abs(got[4] - p) <= tol * rho * (h + m)


@pytest.mark.parametrize("mhd", [0, 1])
def test_iteration_limit_gives_status_3(mhd):
    states = list(_case("fast", mhd, limit=1))
    assert all(st in (0, 3) for *_, st in states)
    assert any(st == 3 for *_, st in states)
    for *_, got, st in states:
        if st == 3:
            assert got[0] == 1e-12 and got[1:4] == [0.0, 0.0, 0.0]
