"""The tile kernels at the edges of their tiles, on the GPU: blocks of one
tile, just over and under one, with remainders in every direction, under each
refresh rule.  Reading halos through the rule equals reading stored ghosts
bitwise, and the stored-ghost result meets the oracle's parity gate."""
import numpy as np
import pytest

import oracle as O
from parity import assert_parity, compare, report
from paper_2311_04989_amd import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

# tiles are 8 x 8 x 4 points; a rule needs n >= ng (3 at order 4, 4 at order 6)
SHAPES = [(6, (4, 4, 4)), (6, (8, 8, 4)), (6, (9, 7, 5)), (6, (17, 8, 11)), (6, (5, 16, 9)),
          (4, (3, 3, 3)), (4, (9, 15, 7))]


def _blocks(order, n, matter):
    """2 x 2 x 2 blocks of n points each, smooth data plus noise, unrelated
    values in every ghost point and in the frozen array."""
    ng = order // 2 + 1
    rng = np.random.default_rng(W.SEED_BASE + 4000 + sum(n))
    h = (0.11, 0.13, 0.17)
    bt = W.Batch([W.Block(*n, ng, *h, *(h[a] * n[a] * ((b >> a) & 1) for a in range(3)))
                  for b in range(8)], with_matter=matter)
    k = rng.uniform(0.5, 2.0, size=(W.NF, 3))
    for b, blk in enumerate(bt.blocks):
        X, Y, Z = blk.coords()
        for f, name in enumerate(W.FIELDS):
            one = 1.0 if name in ("chi", "gxx", "gyy", "gzz", "alpha") else 0.0
            v = bt.view(bt.u, b, f)
            v[...] = rng.uniform(0.9, 1.1, size=v.shape) if one else rng.uniform(-0.1, 0.1, v.shape)
            s = np.sin(k[f, 0] * X + k[f, 1] * Y + k[f, 2] * Z + f)
            bt.interior(bt.u, b, f)[...] = (one + 1e-2 * s)[ng:-ng, ng:-ng, ng:-ng]
        if matter:
            for f in range(W.NM):
                bt.view(bt.matter, b, f, W.NM)[...] = 1e-3 * np.cos(X - Y + 2 * Z + f)
    bt.frozen = np.zeros_like(bt.u)
    for b in range(8):
        for f, name in enumerate(W.FIELDS):
            one = 1.0 if name in ("chi", "gxx", "gyy", "gzz", "alpha") else 0.0
            v = bt.view(bt.frozen, b, f)
            v[...] = one + rng.uniform(-1e-2, 1e-2, size=v.shape)
    nbr = np.full((8, 27), -1, dtype=np.int32)
    for b in range(8):
        for d in range(27):
            q = [((b >> a) & 1) + (d % 3 - 1, (d // 3) % 3 - 1, d // 9 - 1)[a] for a in range(3)]
            if all(0 <= v < 2 for v in q):
                nbr[b, d] = q[0] + 2 * q[1] + 4 * q[2]
    bt.neighbours = nbr
    bt.params = W.Params(fd_order=order, ko_sigma=0.3)
    return bt


@pytest.mark.parametrize("order,n", SHAPES)
@pytest.mark.parametrize("rule", ["periodic", "neighbour", "neighbour stored outside", "frozen"])
def test_tile_edges(order, n, rule):
    from paper_2311_04989_amd import z4c as Z
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    O.build(force=False)
    print(f"tile edges: order {order}, {n}, {rule}", flush=True)
    bt = _blocks(order, n, matter=rule == "neighbour")
    policy = {"periodic": Z.GHOST_PERIODIC, "frozen": Z.GHOST_FROZEN}.get(rule, Z.GHOST_NEIGHBOUR)
    if rule in ("periodic", "neighbour stored outside"):
        bt.frozen = None
    dev = lambda a: None if a is None else torch.from_numpy(a).to("cuda:0")  # noqa: E731
    filled = bt.u.copy()
    O.ghost_fill(bt, filled, policy)
    got = {}
    for read in ("rule", "stored"):
        plan = Z.plan_for(bt)
        if read == "rule":
            plan.set_halo(policy, frozen := dev(bt.frozen))
        u = dev(bt.u if read == "rule" else filled)
        rhs, out, acc = (torch.zeros(bt.total_u, dtype=torch.float64, device="cuda:0")
                         for _ in range(3))
        m = dev(bt.matter)
        plan.rhs(u, m, rhs)
        plan.rk_stage(u, out, acc, u, m, Z.RK4[1], 0.01)
        cons = torch.zeros(bt.total_c, dtype=torch.float64, device="cuda:0")
        norms = torch.zeros(16 * len(bt.blocks), dtype=torch.float64, device="cuda:0")
        plan.constraints(u, m, cons, norms)
        torch.cuda.synchronize()
        got[read] = [x.cpu().numpy() for x in (rhs, out, acc, cons, norms)]
        plan.close()
    for a, b in zip(got["rule"], got["stored"]):
        assert np.array_equal(a, b)
    bt.u = filled
    rows = compare(bt, got["stored"][0], O.rhs(bt), O.rhs(bt, ext=True))
    assert_parity(rows, f"tile edges {order} {n} {rule}\n" + report(rows))
    c80, n80 = O.constraints(bt, ext=True)
    rows = compare(bt, got["stored"][3], O.constraints(bt)[0], c80, nfields=W.NC)
    assert_parity(rows, f"tile edges {order} {n} {rule} constraints\n" + report(rows))
    np.testing.assert_allclose(got["stored"][4].reshape(-1, 8, 2), n80, rtol=1e-10, atol=1e-300)


# Tile rows along x of over 8 tiles: slabs of 4 rows (17 tiles) and of one (66)
@pytest.mark.parametrize("n", [(130, 43, 5), (521, 9, 5)])
def test_tile_slabs(n):
    from paper_2311_04989_amd import z4c as Z
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    O.build(force=False)
    print(f"tile slabs: {n}", flush=True)
    bt = _blocks(6, n, matter=False)
    plan = Z.plan_for(bt)
    u = torch.from_numpy(bt.u).to("cuda:0")
    rhs = torch.full_like(u, np.nan)
    cons = torch.zeros(bt.total_c, dtype=torch.float64, device="cuda:0")
    norms = torch.zeros(16 * len(bt.blocks), dtype=torch.float64, device="cuda:0")
    plan.rhs(u, None, rhs)
    plan.constraints(u, None, cons, norms)
    torch.cuda.synchronize()
    plan.close()
    rows = compare(bt, rhs.cpu().numpy(), O.rhs(bt), O.rhs(bt, ext=True))
    assert_parity(rows, f"tile slabs {n}\n" + report(rows))
    c80, n80 = O.constraints(bt, ext=True)
    rows = compare(bt, cons.cpu().numpy(), O.constraints(bt)[0], c80, nfields=W.NC)
    assert_parity(rows, f"tile slabs {n} constraints\n" + report(rows))
    np.testing.assert_allclose(norms.cpu().numpy().reshape(-1, 8, 2), n80, rtol=1e-10, atol=1e-300)
