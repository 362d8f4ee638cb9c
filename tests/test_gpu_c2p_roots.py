"""Primitive recovery of given normalised states in flat space (D = 1, so that
the master function's coefficients are the inputs themselves), on the GPU:
states whose function has no finite value at the lower end of the bracket."""
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
