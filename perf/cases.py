"""The work that programs have this library do, as cases that can be timed.

Every case goes through the public binding (`paper_2311_04989_amd.z4c`) on
arrays that live on the GPU.  A case is a dict with the kind of work
("kind") and its sizes; the kinds and the ranges of their sizes are those of
the repository's workload configurations, tests and benchmark:

  step         one Runge-Kutta step of a level set, captured in a HIP graph
  stage        one fused right-hand side + Runge-Kutta stage
  rhs          the right-hand side alone
  constraints  constraint fields and per-block norms
  matter       metric to cells, GRMHD sources, sources to vertices
  recovery     primitive recovery of every cell
  exchange     restriction and prolongation across a level jump

`exact` evaluates the same quantities with plain torch operations in 64 bits.
"""
import math
import os
import shutil
import tempfile

import numpy as np
import torch

from paper_2311_04989_amd import workloads as W
from paper_2311_04989_amd import z4c as Z

DEV = "cuda:0"
NF, NM, NC = W.NF, W.NM, W.NC
CHI, G0, KHAT, A0, THETA, GAM0, ALPHA, B0 = 0, 1, 7, 8, 14, 15, 18, 19
ONES = (CHI, G0, G0 + 3, G0 + 5, ALPHA)   # fields that are 1 in flat space
RK4_STAGE2 = Z.RK4[1]
POLICY = {"none": Z.GHOST_NONE, "periodic": Z.GHOST_PERIODIC, "neighbour": Z.GHOST_NEIGHBOUR,
          "frozen": Z.GHOST_FROZEN, "radiative": Z.GHOST_NEIGHBOUR}


def listed():
    return [
        # one small block, order 4, stored 3 ghosts deep: the smallest step a
        # program takes, where the launches and their latency are the cost
        dict(name="gauge wave step 16^3", kind="step", data="gauge", order=4, ng=3, sizes="16",
             counts="1", nz=0, halo="periodic", matter=False, arith="fp64", advection=0,
             monitor=False, tuned=False),
        # right-hand side of one ordinary block with matter sources, frozen
        # outer ghosts, the plan's default launch: a method-of-lines driver
        # with an integrator of its own
        dict(name="star rhs 64^3", kind="rhs", data="star", order=6, ng=4, sizes="64",
             counts="1", nz=0, halo="frozen", matter=True, arith="fp64", advection=0,
             monitor=False, tuned=False),
        # one stage of a level set of equal 16^3 blocks, stored ghosts: the
        # shape that mesh codes run most
        dict(name="level set stage 512x16^3", kind="stage", data="gauge", order=6, ng=4,
             sizes="16", counts="512", nz=0, halo="none", matter=False, arith="fp64",
             advection=0, monitor=False, tuned=True),
        # the benchmark: a whole step of 1,024 blocks of four sizes
        dict(name="uneven level set step", kind="step", data="flat", order=6, ng=4,
             sizes="8/16/24/32", counts="410/307/205/102", nz=0, halo="periodic", matter=False,
             arith="fp64", advection=0, monitor=False, tuned=True),
        # a whole step of the star on 8 large blocks that share faces: the
        # largest call
        dict(name="star step 8x128^3", kind="step", data="star", order=6, ng=4, sizes="128",
             counts="8", nz=0, halo="neighbour", matter=True, arith="fp64", advection=0,
             monitor=False, tuned=True),
        # the same physics with single-precision arithmetic
        dict(name="star step fp32 8x64^3", kind="step", data="star", order=6, ng=4, sizes="64",
             counts="8", nz=0, halo="neighbour", matter=True, arith="fp32", advection=0,
             monitor=False, tuned=True),
        # the radiative outer boundary and the constraint monitor inside a step
        dict(name="radiative monitor step 8x40^3", kind="step", data="star", order=6, ng=4,
             sizes="40", counts="8", nz=0, halo="radiative", matter=False, arith="fp64",
             advection=0, monitor=True, tuned=True),
        # upwind-biased advection on ragged blocks, the plan's default launch
        dict(name="lopsided stage ragged", kind="stage", data="smooth", order=6, ng=4,
             sizes="20/13/33", counts="24/40/12", nz=19, halo="none", matter=False,
             arith="fp64", advection=1, monitor=False, tuned=False),
        # constraints of a set at an output time, the plan's default launch
        dict(name="constraints 96x24^3", kind="constraints", data="smooth", order=6, ng=4,
             sizes="24", counts="96", nz=0, halo="none", matter=True, arith="fp64", advection=0,
             monitor=False, tuned=False),
        # matter coupling of every stage of a run with a fluid
        dict(name="matter coupling 8x128^3 cells", kind="matter", nc=128, blocks=8, ext=3,
             order_cc=4, order_vc=6),
        # primitive recovery of a magnetised star and its atmosphere
        dict(name="primitive recovery 8x96^3", kind="recovery", nc=96, blocks=8, ext=3, mhd=True),
        # ghosts across a level jump: octants restricted, face slabs prolongated
        dict(name="level jump 64+512 blocks", kind="exchange", ncoarse=64, n=16, order=6),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["step", "step", "stage", "stage", "rhs", "constraints", "matter",
                       "recovery", "exchange"])
    if kind == "matter":
        return dict(kind=kind, nc=_log(rng, 12, 128), blocks=8, ext=rng.randint(0, 3),
                    order_cc=rng.choice([2, 4]), order_vc=rng.choice([4, 6]))
    if kind == "recovery":
        return dict(kind=kind, nc=_log(rng, 12, 96), blocks=8, ext=rng.randint(0, 3),
                    mhd=rng.random() < 0.7)
    if kind == "exchange":
        return dict(kind=kind, ncoarse=_log(rng, 2, 64), n=rng.choice([12, 14, 16]),
                    order=rng.choice([4, 6]))
    c = dict(kind=kind, order=6, ng=4, nz=0, matter=rng.random() < 0.3, arith="fp64",
             advection=0, monitor=False, tuned=rng.random() < 0.7)
    if kind == "step":
        c["halo"] = rng.choice(["periodic", "neighbour", "radiative"])
        if c["halo"] == "periodic":
            c["data"] = rng.choice(["gauge", "flat"])
            if rng.random() < 0.3:   # small order-4 runs
                c.update(order=4, ng=3, data="gauge", tuned=False)
                c["sizes"], c["counts"] = str(rng.randint(12, 32)), str(_log(rng, 1, 16))
            else:
                s = sorted(rng.sample(range(8, 34), 3))
                c["sizes"] = "/".join(map(str, s))
                c["counts"] = "/".join(str(_log(rng, 2, 200)) for _ in s)
            c["matter"] = False
        else:
            c["data"], c["counts"] = "star", "8"
            c["sizes"] = str(_log(rng, 12, 96))
            if c["halo"] == "neighbour" and rng.random() < 0.5:
                c["arith"] = "fp32"
            c["monitor"] = c["halo"] == "radiative" and rng.random() < 0.5
    else:
        c["halo"] = "none"
        c["data"] = rng.choice(["gauge", "smooth"])
        s = rng.sample(range(8, 49), 2)
        c["sizes"] = "/".join(map(str, s))
        c["counts"] = "/".join(str(_log(rng, 1, 128)) for _ in s)
        if rng.random() < 0.5:
            c["nz"] = rng.randint(5, 40)
        if kind == "rhs" and rng.random() < 0.5:
            c.update(halo="frozen", data="star", sizes=str(_log(rng, 16, 80)), counts="1", nz=0)
        if kind == "stage" and rng.random() < 0.4:
            c["advection"] = 1
    return c


# --- blocks and their arrays -------------------------------------------------------


class Blocks:
    """The MeshBlocks of a case (shuffled by the seed, as a mesh numbers
    them) in the block-major layout of the workloads."""

    def __init__(self, c, seed):
        sizes = [int(v) for v in c["sizes"].split("/")]
        counts = [int(v) for v in c["counts"].split("/")]
        rng = np.random.default_rng(seed)
        ns = np.concatenate([np.full(k, s) for k, s in zip(counts, sizes)])
        rng.shuffle(ns)
        nb = len(ns)
        self.ng = c["ng"]
        self.dims = [(int(n), int(n), c["nz"] or int(n)) for n in ns]   # nx, ny, nz
        if c["data"] == "star":
            # the blocks tile [-16, 16]^3 (2 x 2 x 2 of them, or one)
            side = 2 if nb == 8 else 1
            d = 32.0 / (side * self.dims[0][0])
            self.dx = np.full(nb, d)
            self.x0 = [tuple(-16.0 + 32.0 / side * ((b >> a) & 1) + 0.5 * d for a in range(3))
                       for b in range(nb)]
        elif c["order"] == 4:   # periodic unit box
            self.dx = 1.0 / np.array([d[0] for d in self.dims], dtype=np.float64)
            self.x0 = [(0.0, 0.0, 0.0)] * nb
        else:
            self.dx = 0.5 / 2.0 ** rng.integers(0, 7, size=nb)
            self.x0 = [tuple(v) for v in rng.uniform(0.0, 1.0, size=(nb, 3))]
        g = 2 * self.ng
        self.shape = [(nz + g, ny + g, nx + g) for nx, ny, nz in self.dims]
        self.npts = [a * b * d for a, b, d in self.shape]
        self.stride = np.array([n + (n & 1) for n in self.npts], dtype=np.int64)
        self.start = np.concatenate([[0], np.cumsum(self.stride)])
        self.nb = nb
        self.classes = {}
        for b, d in enumerate(self.dims):
            self.classes.setdefault(d, []).append(b)
        self.interior = sum(a * b * d for a, b, d in self.dims)

    def zeros(self, nf):
        return torch.zeros(nf * int(self.start[-1]), dtype=torch.float64, device=DEV)

    def view(self, arr, b, nf):
        """(nf, sz, sy, sx) view of block b of an array of nf fields."""
        o, s, n = nf * int(self.start[b]), int(self.stride[b]), self.npts[b]
        return arr[o:o + nf * s].view(nf, s)[:, :n].unflatten(1, self.shape[b])

    def table(self):
        t = np.zeros(self.nb, dtype=W.BLOCK_DTYPE)
        for b, (nx, ny, nz) in enumerate(self.dims):
            s, d = int(self.start[b]), self.dx[b]
            t[b] = (NF * s, NM * s, NC * s, self.stride[b], nx, ny, nz, self.ng, d, d, d)
        return t

    def coords(self, b):
        """x, y, z of the stored points of block b, each shaped to broadcast."""
        out = []
        for a, n in enumerate(self.dims[b]):
            v = torch.arange(-self.ng, n + self.ng, dtype=torch.float64, device=DEV)
            shp = [1, 1, 1]
            shp[2 - a] = -1
            out.append((self.x0[b][a] + v * float(self.dx[b])).view(shp))
        return out


def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(int(seed))


def _state(c, L, seed, g):
    """The 22 state fields, ghosts included."""
    noise = {"gauge": 1e-10, "flat": 1e-8, "star": 1e-6, "smooth": 1e-6}[c["data"]]
    u = torch.empty(NF * int(L.start[-1]), dtype=torch.float64, device=DEV)
    u.uniform_(-noise, noise, generator=g)
    rng = np.random.default_rng(seed + 1)
    for b in range(L.nb):
        v = L.view(u, b, NF)
        if c["data"] == "flat":
            for f in ONES:
                v[f] += 1.0
        elif c["data"] == "gauge":   # varies along x only
            x = L.x0[b][0] + np.arange(-L.ng, L.dims[b][0] + L.ng) * L.dx[b]
            w = W.gauge_wave(x, x, x, amp=0.01, wavelength=1.0)
            v += torch.from_numpy(np.stack([w[n] for n in W.FIELDS])).to(DEV)[:, None, None, :]
        elif c["data"] == "star":
            x, y, z = L.coords(b)
            psi = 1.0 + 0.7 / torch.sqrt(x * x + y * y + z * z + 4.0)
            v[CHI] += psi ** -4.0
            v[ALPHA] += psi ** -2.0
            for f in (G0, G0 + 3, G0 + 5):
                v[f] += 1.0
        else:   # smooth perturbation of flat space, shift of both signs
            x, y, z = L.coords(b)
            h = 4.0 * float(L.dx[b])
            k, ph = rng.uniform(0.5, 2.0, size=(NF, 3)) / h, rng.uniform(0, 2 * math.pi, NF)
            for f in range(NF):
                v[f] += 1e-3 * torch.sin(k[f, 0] * x + k[f, 1] * y + k[f, 2] * z + ph[f])
            for f in ONES:
                v[f] += 1.0
    return u


def _matter(L, seed):
    """ADM projections: one Gaussian blob per field."""
    m = L.zeros(NM)
    centres, amps, w = W.matter_blobs(np.random.default_rng(seed + 2))
    for b in range(L.nb):
        x, y, z = L.coords(b)
        v = L.view(m, b, NM)
        for f in range(NM):
            d2 = (x - centres[f, 0]) ** 2 + (y - centres[f, 1]) ** 2 + (z - centres[f, 2]) ** 2
            v[f] = amps[f] * torch.exp(-d2 / (2.0 * w * w))
    return m


def _params(c):
    return W.Params(fd_order=c["order"], ko_sigma=0.02 if c["order"] == 4 else 0.5,
                    advection=c["advection"])


def _neighbours(nb):
    """2 x 2 x 2 blocks tiling a cube: -1 beyond its faces."""
    t = np.full((nb, 27), -1, dtype=np.int32)
    for b in range(nb):
        p = (b & 1, (b >> 1) & 1, (b >> 2) & 1)
        for d in range(27):
            q = [p[0] + d % 3 - 1, p[1] + (d // 3) % 3 - 1, p[2] + d // 9 - 1]
            if all(0 <= v < 2 for v in q):
                t[b, d] = q[0] + 2 * q[1] + 4 * q[2]
    return t


def _dt(L):
    return 0.25 * float(min(L.dx))


_cache = None


def _tune_cache():
    """A copy of the committed launch-shape cache that this program may add to."""
    global _cache
    if _cache is None:
        _cache = os.path.join(tempfile.mkdtemp(prefix="z4c_tune_"), "tune.txt")
        shutil.copy(os.path.join(os.path.dirname(Z.__file__), "tune_gfx950.txt"), _cache)
    return _cache


def _stream():
    return torch.cuda.current_stream()


# --- what a program has in hand, and one pass ---------------------------------------


def prepare(case, seed):
    kind = case["kind"]
    if kind == "matter":
        return _prepare_matter(case, seed)
    if kind == "recovery":
        return _prepare_recovery(case, seed)
    if kind == "exchange":
        return _prepare_exchange(case, seed)
    L = Blocks(case, seed)
    g = _gen(seed)
    s = dict(case=case, kind=kind, L=L, dt=_dt(L), u=_state(case, L, seed, g))
    s["matter"] = _matter(L, seed) if case["matter"] else None
    plan = Z.Plan(Z.make_params(_params(case), Z.ARITH_FP32 if case["arith"] == "fp32"
                                else Z.ARITH_FP64), Z.make_blocks(L.table()))
    s["plan"] = plan
    halo = case["halo"]
    s["frozen"] = s["u"].clone() if halo in ("frozen", "neighbour") else None
    if halo in ("neighbour", "radiative"):
        plan.set_neighbours(_neighbours(L.nb))
    if halo == "radiative":
        plan.set_sommerfeld(np.array(L.x0))
    plan.set_halo(POLICY[halo], s["frozen"])
    if kind == "rhs":
        s["out"] = L.zeros(NF)
    elif kind == "stage":
        s["out"] = L.zeros(NF)
        s["acc"] = s["u"] * 0.25
        s["y"] = s["u"] * (1.0 + 1e-9)
    elif kind == "step":
        s["regs"] = [s["u"]] + [L.zeros(NF) for _ in range(3)]
        s["flags"] = ((Z.STEP_MONITOR if case["monitor"] else 0)
                      | (Z.STEP_SOMMERFELD if halo == "radiative" else 0))
    if kind == "constraints" or case["monitor"]:
        s["cons"] = L.zeros(NC)
        s["norms"] = torch.zeros(16 * L.nb, dtype=torch.float64, device=DEV)
    if case["tuned"]:
        Z.set_tune_cache(_tune_cache())
        b = [L.zeros(NF) for _ in range(2)]
        plan.autotune(s["u"], b[0], b[1], s["matter"], reps=3, stream=_stream())
    return s


def run(s):
    kind, plan, st = s["kind"], s.get("plan"), _stream()
    if kind == "step":
        c = s["case"]
        r = plan.step(s["regs"], s["matter"], Z.RK4, s["dt"], POLICY[c["halo"]],
                      frozen=s["frozen"], stream=st, graph=True, flags=s["flags"],
                      cons=s.get("cons"), norms=s.get("norms"))
        out = [s["regs"][r]]
        return out + [s["cons"], s["norms"]] if c["monitor"] else out
    if kind == "stage":
        plan.rk_stage(s["u"], s["out"], s["acc"], s["y"], s["matter"], RK4_STAGE2, s["dt"],
                      stream=st)
        return [s["out"], s["acc"]]
    if kind == "rhs":
        plan.rhs(s["u"], s["matter"], s["out"], stream=st)
        return [s["out"]]
    if kind == "constraints":
        plan.constraints(s["u"], s["matter"], s["cons"], s["norms"], stream=st)
        return [s["cons"], s["norms"]]
    if kind == "matter":
        c, mp = s["case"], s["mplan"]
        mp.metric_to_cc(c["order_cc"], c["ext"], s["u"], s["geom"], stream=st)
        mp.adm_sources(1, 2.0, 1e-6, c["ext"], s["geom"], s["prim"], s["adm"], stream=st)
        mp.sources_to_vc(c["order_vc"], s["adm"], s["matter"], stream=st)
        return [s["geom"], s["adm"], s["matter"]]
    if kind == "recovery":
        s["mplan"].c2p(s["par"], s["case"]["ext"], s["geom"], s["cons"], s["prim"], s["status"],
                       stream=st)
        return [s["prim"], s["cons"], s["status"]]
    s["xplan"].restrict(s["u"], stream=st)
    s["xplan"].prolongate(s["u"], stream=st)
    return [s["u"]]


def work(case):
    """Each input read once and each output written once; the operations of
    the equations (derivatives in separable form, algebra, combination)."""
    kind = case["kind"]
    if kind in ("matter", "recovery"):
        n = case["nc"] + 2 * case["ext"]
        cells, v = 8 * n ** 3, 8 * (case["nc"] + 1) ** 3
        if kind == "recovery":
            q = 8 if case["mhd"] else 5
            return dict(bytes=cells * (7 * 8 + 2 * 8 * q + 4), flops=cells * 2000.0)
        return dict(bytes=8.0 * (7 * v + 7 * cells + 15 * cells + 10 * cells + 10 * cells + 10 * v),
                    flops=cells * (7 * 36 + 150.0) + v * 10 * 51.0)
    if kind == "exchange":
        n, k = case["n"], 8 * case["ncoarse"]
        fine, coarse = k * 6 * 4 * n * n, k * (n // 2) ** 3
        return dict(bytes=176.0 * (fine + fine / 8 + 2 * coarse), flops=22.0 * fine * 20)
    pts = Blocks(case, 0).interior
    m = 80 * pts if case["matter"] else 0
    flops = {6: 4400.0, 4: 3300.0}[case["order"]]
    if kind == "rhs":
        return dict(bytes=352.0 * pts + m, flops=flops * pts)
    if kind == "stage":
        return dict(bytes=880.0 * pts + m, flops=(flops + 160) * pts)
    if kind == "constraints":
        return dict(bytes=8.0 * (18 + 8) * pts + m, flops=0.6 * flops * pts)
    return dict(bytes=4 * (704.0 * pts + m) + (64 * pts if case["monitor"] else 0),
                flops=4 * (flops + 160) * pts)


# --- matter, recovery, exchange ------------------------------------------------------


class Cells:
    """2 x 2 x 2 blocks of nc^3 cells tiling [-16, 16]^3 (4 ghost vertices,
    3 ghost cells), block-major."""

    def __init__(self, nc):
        self.nc, self.nb, self.ngv, self.ngc = nc, 8, 4, 3
        self.sv, self.sc = nc + 9, nc + 6
        self.nv, self.ncell = self.sv ** 3, self.sc ** 3
        self.vs, self.cs = self.nv + (self.nv & 1), self.ncell + (self.ncell & 1)
        t = np.zeros(8, dtype=W.MBLOCK_DTYPE)
        for b in range(8):
            t[b] = (NF * self.vs * b, NM * self.vs * b, self.vs, 7 * self.cs * b, 8 * self.cs * b,
                    10 * self.cs * b, 8 * self.cs * b, self.cs * b, self.cs, nc, nc, nc, 4, 3, 0)
        self.table = t

    def zeros(self, nf, cells=True):
        return torch.zeros(8 * nf * (self.cs if cells else self.vs), dtype=torch.float64,
                           device=DEV)

    def view(self, arr, nf, cells=True):
        """(8, nf, s, s, s) view."""
        st, n, s = (self.cs, self.ncell, self.sc) if cells else (self.vs, self.nv, self.sv)
        return arr.view(8, nf, st)[:, :, :n].unflatten(2, (s, s, s))

    def coords(self, cells=True):
        s, ng, h = (self.sc, self.ngc, 0.5) if cells else (self.sv, self.ngv, 0.0)
        d = 16.0 / self.nc
        v = (torch.arange(s, dtype=torch.float64, device=DEV) - ng + h) * d
        out = []
        for a in range(3):
            o = torch.tensor([-16.0 + 16.0 * ((b >> a) & 1) for b in range(8)],
                             dtype=torch.float64, device=DEV)
            shp = [8, 1, 1, 1]
            shp[3 - a] = s
            out.append((o[:, None] + v[None, :]).view(shp))
        return out


def _metric(v, x, y, z):
    """chi and gt_ij of a star, slightly anisotropic, into v[:, 0..6]."""
    psi = 1.0 + 0.7 / torch.sqrt(x * x + y * y + z * z + 4.0)
    h = 0.02 * torch.sin(0.3 * x + 0.2 * y) * torch.cos(0.25 * z)
    v[:, 0] += psi ** -4.0
    for q, (i, j) in enumerate(W.SYM):
        v[:, 1 + q] += (1.0 if i == j else 0.0) + h * (1.0 if i == j else 0.5) * (1 + q) / 6.0


def _fluid(M, g, seed, noise=1e-6):
    """Primitives of a rotating magnetised star: density blobs in a thin
    atmosphere, polytropic pressure, a field that follows the density."""
    rng = np.random.default_rng(seed + 3)
    x, y, z = M.coords()
    rho = torch.zeros_like(x + y + z)
    for ctr in rng.uniform(-4.0, 4.0, size=(4, 3)):
        rho += 1e-3 * torch.exp(-((x - ctr[0]) ** 2 + (y - ctr[1]) ** 2 + (z - ctr[2]) ** 2) / 8.0)
    tilt = rng.normal(size=3)
    tilt /= np.linalg.norm(tilt)
    rho = rho * (1.0 + noise * torch.empty_like(rho).uniform_(-1.0, 1.0, generator=g))
    prim = M.zeros(8)
    v = M.view(prim, 8)
    v[:, 0] = rho
    v[:, 1] = -0.02 * y
    v[:, 2] = 0.02 * x
    v[:, 3] = float(rng.uniform(-0.05, 0.05))
    v[:, 4] = 100.0 * rho * rho
    for a in range(3):
        v[:, 5 + a] = 1e-3 * tilt[a] * torch.sqrt(rho / 1e-3)
    v[:, 7] += 2e-4 * torch.sin(0.3 * x) * torch.sqrt(rho / 1e-3)
    return prim


def _prepare_matter(c, seed):
    M, g = Cells(c["nc"]), _gen(seed)
    u = M.zeros(NF, cells=False).uniform_(-1e-6, 1e-6, generator=g)
    _metric(M.view(u, NF, cells=False), *M.coords(cells=False))
    return dict(case=c, kind="matter", M=M, mplan=Z.MPlan(M.table), u=u, prim=_fluid(M, g, seed),
                geom=M.zeros(7), adm=M.zeros(10), matter=M.zeros(NM, cells=False))


def _atm():
    return dict(rho_atm=1e-10, gamma_ad=2.0, p_atm=100.0 * 1e-20)


def _conserved(M, geom, prim, mhd):
    """Densitised conservatives of the primitives, and sqrt(gamma)."""
    gv, w = M.view(geom, 7), M.view(prim, 8)
    gam = [gv[:, 1 + q] / gv[:, 0].clamp(min=1e-6) for q in range(6)]
    G = [[gam[S(i, j)] for j in range(3)] for i in range(3)]
    sg = torch.sqrt(_det(gam))
    low = lambda a: [sum(G[i][j] * a[j] for j in range(3)) for i in range(3)]  # noqa: E731
    ut, rho, p = [w[:, 1 + i] for i in range(3)], w[:, 0], w[:, 4]
    ul = low(ut)
    W2 = 1.0 + sum(a * b for a, b in zip(ut, ul))
    Wl = torch.sqrt(W2)
    e, b2, ab0, bl = rho + 2.0 * p, 0.0, 0.0, [0.0] * 3
    if mhd:
        Bu = [w[:, 5 + i] for i in range(3)]
        Bl = low(Bu)
        ab0 = sum(a * b for a, b in zip(Bu, ul))
        b2 = (ab0 * ab0 + sum(a * b for a, b in zip(Bu, Bl))) / W2
        bl = [Bl[i] / Wl + ab0 * ul[i] / Wl for i in range(3)]
    cons = M.zeros(8)
    q = M.view(cons, 8)
    q[:, 0] = sg * rho * Wl
    for i in range(3):
        q[:, 1 + i] = sg * ((e + b2) * Wl * ul[i] - ab0 * bl[i])
    q[:, 4] = sg * ((e + b2) * W2 - rho * Wl - (p + 0.5 * b2) - ab0 * ab0)
    if mhd:
        for i in range(3):
            q[:, 5 + i] = sg * Bu[i]
    return cons


def _recovery_data(c, seed):
    M, g = Cells(c["nc"]), _gen(seed)
    geom = M.zeros(7)
    _metric(M.view(geom, 7), *M.coords())
    prim = _fluid(M, g, seed)
    return M, geom, prim, _conserved(M, geom, prim, c["mhd"])


def _prepare_recovery(c, seed):
    M, geom, prim, cons = _recovery_data(c, seed)
    a = _atm()
    par = Z.c2p_params(mhd=int(c["mhd"]), gamma_ad=a["gamma_ad"], rho_atm=a["rho_atm"],
                       p_atm=a["p_atm"])
    del prim
    return dict(case=c, kind="recovery", M=M, mplan=Z.MPlan(M.table), geom=geom, cons=cons,
                par=par, prim=M.zeros(8),
                status=torch.zeros(8 * M.cs, dtype=torch.int32, device=DEV))


def _exchange_parts(c, seed):
    """Blocks of n^3 + 4 ghosts: coarse ones, then 8 fine ones per coarse
    one; every fine block receives its six face slabs from a coarse block
    drawn by the seed and injects its even vertices into its octant."""
    n, nco, ng = c["n"], c["ncoarse"], 4
    npts = (n + 8) ** 3
    st = npts + (npts & 1)
    nb = 9 * nco
    t = np.zeros(nb, dtype=W.BLOCK_DTYPE)
    for b in range(nb):
        d = 1.0 if b < nco else 0.5
        t[b] = (NF * st * b, NM * st * b, NC * st * b, st, n, n, n, ng, d, d, d)
    src = np.random.default_rng(seed).integers(0, nco, size=(8 * nco, 6))
    h, pro, res = n // 2, [], []
    for k in range(8 * nco):
        s = 0
        for d in range(3):
            for lo, hi in ((-ng, 0), (n, n + ng)):
                bl, bh = [0] * 3, [n] * 3
                bl[d], bh[d] = lo, hi
                pro.append(dict(coarse=int(src[k, s]), fine=nco + k, c0=[4, 4, 4], lo=bl, hi=bh))
                s += 1
        c0 = [h * ((k >> d) & 1) for d in range(3)]
        res.append(dict(coarse=k // 8, fine=nco + k, c0=c0, lo=c0, hi=[v + h for v in c0]))
    u = torch.empty(NF * st * nb, dtype=torch.float64, device=DEV)
    u.uniform_(-1.0, 1.0, generator=_gen(seed))
    return t, u, pro, res, src, st, npts


def _prepare_exchange(c, seed):
    t, u, pro, res, _, _, _ = _exchange_parts(c, seed)
    plan = Z.Plan(Z.make_params(W.Params()), Z.make_blocks(t))
    return dict(case=c, kind="exchange", u=u, plan=plan, xplan=Z.XPlan(plan, pro, res, c["order"]))


# --- the same in plain torch, 64 bits --------------------------------------------------

S = lambda i, j: ((0, 1, 2), (1, 3, 4), (2, 4, 5))[i][j]  # noqa: E731


def _det(g):
    return (g[0] * (g[3] * g[5] - g[4] * g[4]) - g[1] * (g[1] * g[5] - g[4] * g[2])
            + g[2] * (g[1] * g[4] - g[3] * g[2]))


def _inverse(g):
    d = 1.0 / _det(g)
    return [(g[3] * g[5] - g[4] * g[4]) * d, (g[2] * g[4] - g[1] * g[5]) * d,
            (g[1] * g[4] - g[2] * g[3]) * d, (g[0] * g[5] - g[2] * g[2]) * d,
            (g[2] * g[1] - g[0] * g[4]) * d, (g[0] * g[3] - g[1] * g[1]) * d]


D1W = {4: (8.0, -1.0), 6: (45.0, -9.0, 1.0)}
D1N = {4: 12.0, 6: 60.0}
D2W = {4: (16.0, -1.0), 6: (270.0, -27.0, 2.0)}
D2N = {4: 12.0, 6: 180.0}
KOW = {4: (15.0, -6.0, 1.0), 6: (-56.0, 28.0, -8.0, 1.0)}
LOPW = {4: ((-1, -3.0), (1, 18.0), (2, -6.0), (3, 1.0)),
        6: ((-2, 2.0), (-1, -24.0), (1, 80.0), (2, -30.0), (3, 8.0), (4, -1.0))}


class Grid:
    """Stencils on arrays (blocks, z, y, x) that hold ng ghosts; h: spacing
    per block.  Results live on the interior points."""

    def __init__(self, dims, ng, order, h, sigma):
        self.n, self.ng, self.p, self.sigma = dims, ng, order, sigma   # dims: nx, ny, nz
        self.h = torch.as_tensor(np.asarray(h), dtype=torch.float64, device=DEV).view(-1, 1, 1, 1)

    def at(self, u, off, grow=(0, 0, 0)):
        """u shifted by off per direction on the interior grown by `grow`."""
        idx = [slice(None)]
        for a in (2, 1, 0):
            o = self.ng - grow[a] + off[a]
            idx.append(slice(o, o + self.n[a] + 2 * grow[a]))
        return u[tuple(idx)]

    def _pair(self, u, a, m, grow=(0, 0, 0)):
        o = [0, 0, 0]
        o[a] = m
        return self.at(u, o, grow), self.at(u, [-v for v in o], grow)

    def d1(self, u, a):
        s = 0.0
        for m, w in enumerate(D1W[self.p], 1):
            p, q = self._pair(u, a, m)
            s = s + w * (p - q)
        return s / (D1N[self.p] * self.h)

    def d2(self, u, a, b):
        if a == b:
            c, s = self.at(u, (0, 0, 0)), 0.0
            for m, w in enumerate(D2W[self.p], 1):
                p, q = self._pair(u, a, m)
                s = s + w * ((p - c) + (q - c))
            return s / (D2N[self.p] * self.h * self.h)
        s = 0.0
        for m, w in enumerate(D1W[self.p], 1):
            for k, x in enumerate(D1W[self.p], 1):
                o = [[0, 0, 0] for _ in range(4)]
                for t, (i, j) in enumerate(((1, 1), (1, -1), (-1, 1), (-1, -1))):
                    o[t][a], o[t][b] = i * m, j * k
                v = [self.at(u, q) for q in o]
                s = s + w * x * ((v[0] - v[1]) - (v[2] - v[3]))
        return s / ((D1N[self.p] * self.h) ** 2)

    def ko(self, u):
        c, s = self.at(u, (0, 0, 0)), 0.0
        for a in range(3):
            for m, w in enumerate(KOW[self.p], 1):
                p, q = self._pair(u, a, m)
                s = s + w * ((p - c) + (q - c))
        return s * ((self.sigma / 64.0 if self.p == 4 else -self.sigma / 256.0) / self.h)

    def lop(self, u, a, beta):
        """beta d_a u on the points shifted by one towards the sign of beta."""
        c = self.at(u, (0, 0, 0))
        v = []
        for side in (1, -1):
            s = 0.0
            for m, w in LOPW[self.p]:
                o = [0, 0, 0]
                o[a] = side * m
                s = s + w * (self.at(u, o) - c)
            v.append(side * s)
        return beta * torch.where(beta > 0, v[0], v[1]) / (D1N[self.p] * self.h)


def _evaluate(G, u, m, par, constraints=False):
    """d_t u (22 interior arrays) or the 8 constraints of u[f] (ghosts
    included); m: 10 interior matter arrays or None."""
    R3 = range(3)
    c = [G.at(u[f], (0, 0, 0)) for f in range(NF)]
    g, A = c[G0:G0 + 6], c[A0:A0 + 6]
    gi = _inverse(g)
    tr = lambda t: sum((1 if i == j else 2) * gi[S(i, j)] * t[S(i, j)]  # noqa: E731
                       for i in R3 for j in range(i, 3))
    chi, al, be = c[CHI], c[ALPHA], c[B0:B0 + 3]
    chis = chi.clamp(min=par.chi_floor)
    K = c[KHAT] + 2.0 * c[THETA]
    adv = ((lambda f, d: sum(G.lop(u[f], k, be[k]) for k in R3)) if par.advection
           else (lambda f, d: sum(be[k] * d[k] for k in R3)))
    dd = lambda f: [G.d2(u[f], i, j) for i in R3 for j in range(i, 3)]  # noqa: E731
    d1 = lambda f: [G.d1(u[f], a) for a in R3]  # noqa: E731
    dg = [d1(G0 + q) for q in range(6)]   # dg[q][k]
    Ric = [-0.5 * tr(dd(G0 + q)) for q in range(6)]
    Gl = [[0.5 * (dg[S(j, k)][i] + dg[S(i, k)][j] - dg[S(i, j)][k]) for i in R3
           for j in range(i, 3)] for k in R3]
    Gu = [[sum(gi[S(k, l)] * Gl[l][q] for l in R3) for q in range(6)] for k in R3]
    Gd = [tr(Gu[k]) for k in R3]
    # T[a][b][l] = gt^{lm} Gt_{a bm}
    T = [[[sum(gi[S(l, m2)] * Gl[a][S(b, m2)] for m2 in R3) for l in R3] for b in R3] for a in R3]
    dG = [d1(GAM0 + k) for k in R3]
    for i in R3:
        for j in range(i, 3):
            s = 0.0
            for k in R3:
                s = s + 0.5 * (g[S(k, i)] * dG[k][j] + g[S(k, j)] * dG[k][i])
                s = s + 0.5 * Gd[k] * (Gl[i][S(j, k)] + Gl[j][S(i, k)])
                for l in R3:
                    s = s + (Gu[k][S(l, i)] * T[j][k][l] + Gu[k][S(l, j)] * T[i][k][l]
                             + Gu[k][S(i, l)] * T[k][j][l])
            Ric[S(i, j)] = Ric[S(i, j)] + s
    dchi, ddc = d1(CHI), dd(CHI)
    DD = [ddc[q] - sum(Gu[k][q] * dchi[k] for k in R3) for q in range(6)]
    dc2 = [dchi[i] * dchi[j] for i in R3 for j in range(i, 3)]
    tD, t2 = tr(DD), tr(dc2)
    for q in range(6):
        Ric[q] = Ric[q] + (DD[q] + g[q] * tD) / (2 * chis) - (dc2[q] + 3 * g[q] * t2) / (4 * chis ** 2)
    Am = [[sum(gi[S(i, k)] * A[S(k, j)] for k in R3) for j in R3] for i in R3]   # At^i_j
    Au = [sum(Am[i][k] * gi[S(k, j)] for k in R3) for i in R3 for j in range(i, 3)]
    AA = sum((1 if i == j else 2) * A[S(i, j)] * Au[S(i, j)] for i in R3 for j in range(i, 3))
    rho, Si, Sij = (m[0], m[1:4], m[4:10]) if m is not None else (0.0, [0.0] * 3, [0.0] * 6)
    Rs = chi * tr(Ric)
    pi = math.pi
    if constraints:
        dK, dT = d1(KHAT), d1(THETA)
        dA = [d1(A0 + q) for q in range(6)]
        out = [Rs + 2.0 / 3.0 * K * K - AA - 16 * pi * rho]
        for i in R3:
            s = -2.0 / 3.0 * (dK[i] + 2.0 * dT[i]) - 8 * pi * Si[i]
            for j in R3:
                s = s - 1.5 / chis * Am[j][i] * dchi[j]
                for k in R3:
                    t = dA[S(i, j)][k]
                    for l in R3:
                        t = t - Gu[l][S(j, k)] * A[S(l, i)] - Gu[l][S(j, i)] * A[S(k, l)]
                    s = s + gi[S(j, k)] * t
            out.append(s)
        return out + [c[THETA]] + [0.5 * (c[GAM0 + k] - Gd[k]) for k in R3]
    dal, dda = d1(ALPHA), dd(ALPHA)
    ca = sum(gi[S(i, j)] * dchi[i] * dal[j] for i in R3 for j in R3)
    DA = [dda[S(i, j)] - sum(Gu[k][S(i, j)] * dal[k] for k in R3)
          + (dchi[i] * dal[j] + dchi[j] * dal[i] - g[S(i, j)] * ca) / (2 * chis)
          for i in R3 for j in range(i, 3)]
    db = [d1(B0 + k) for k in R3]   # db[k][j]
    divb = db[0][0] + db[1][1] + db[2][2]
    ddb = [dd(B0 + k) for k in R3]
    dK, dT = d1(KHAT), d1(THETA)
    X = [-DA[q] + al * (Ric[q] - 8 * pi * Sij[q]) for q in range(6)]
    tX = tr(X)
    trS = chi * tr(Sij) if m is not None else 0.0
    k1, k2 = par.kappa1, par.kappa2
    r = [None] * NF
    r[CHI] = 2.0 / 3.0 * chi * (al * K - divb) + adv(CHI, dchi) + G.ko(u[CHI])
    for i in R3:
        for j in range(i, 3):
            q = S(i, j)
            lie = lambda t: sum(t[S(i, k)] * db[k][j] + t[S(j, k)] * db[k][i]  # noqa: E731
                                for k in R3) - 2.0 / 3.0 * t[q] * divb
            r[G0 + q] = -2 * al * A[q] + lie(g) + adv(G0 + q, dg[q]) + G.ko(u[G0 + q])
            r[A0 + q] = (chi * (X[q] - g[q] * tX / 3.0)
                         + al * (K * A[q] - 2 * sum(A[S(i, k)] * Am[k][j] for k in R3)) + lie(A)
                         + adv(A0 + q, d1(A0 + q)) + G.ko(u[A0 + q]))
    r[KHAT] = (-chi * tr(DA) + al * (AA + K * K / 3.0) + 4 * pi * al * (trS + rho)
               + al * k1 * (1 - k2) * c[THETA] + adv(KHAT, dK) + G.ko(u[KHAT]))
    r[THETA] = (0.5 * al * (Rs - AA + 2.0 / 3.0 * K * K)
                - al * (8 * pi * rho + k1 * (2 + k2) * c[THETA]) + adv(THETA, dT) + G.ko(u[THETA]))
    for i in R3:
        s = adv(GAM0 + i, dG[i]) + G.ko(u[GAM0 + i]) - 2 * al * k1 * (c[GAM0 + i] - Gd[i])
        s = s + tr(ddb[i]) + 2.0 / 3.0 * Gd[i] * divb
        for j in R3:
            s = s - Gd[j] * db[i][j] - 2 * Au[S(i, j)] * dal[j] - 3 * al / chis * Au[S(i, j)] * dchi[j]
            s = s - 2.0 / 3.0 * al * gi[S(i, j)] * (2 * dK[j] + dT[j]) - 16 * pi * al * gi[S(i, j)] * Si[j]
            for k in R3:
                s = s + gi[S(i, j)] * ddb[k][S(j, k)] / 3.0 + 2 * al * Gu[i][S(j, k)] * Au[S(j, k)]
        r[GAM0 + i] = s
        r[B0 + i] = c[GAM0 + i] - par.eta * be[i] + adv(B0 + i, db[i]) + G.ko(u[B0 + i])
    r[ALPHA] = -2 * al * c[KHAT] + adv(ALPHA, dal) + G.ko(u[ALPHA])
    return r


def _enforce(v, par):
    f = _det(v[G0:G0 + 6]) ** (-1.0 / 3.0)
    for q in range(6):
        v[G0 + q] = v[G0 + q] * f
    gi = _inverse(v[G0:G0 + 6])
    tr = sum((1 if i == j else 2) * gi[S(i, j)] * v[A0 + S(i, j)]
             for i in range(3) for j in range(i, 3))
    for q in range(6):
        v[A0 + q] = v[A0 + q] - v[G0 + q] * tr / 3.0
    v[CHI] = v[CHI].clamp(min=par.chi_floor)
    v[ALPHA] = v[ALPHA].clamp(min=par.alpha_floor)
    return v


def _combine(k, u0, u1, u2, co, dt):
    delta, eps, g1, g2, g3, beta, read, write = co
    n1 = (u1 if read else 0.0) + delta * u0 + eps * dt * k
    return n1, g1 * u0 + g2 * n1 + (g3 * u2 if g3 else 0.0) + beta * dt * k


def _radiative_rhs(u, n, ng, dx, x0):
    """The radiative law at every stored point of equal blocks (u: 22 x blocks
    x s^3); only its outer ghost points are used."""
    s = u.shape[-1]
    r2, adv = 0.0, 0.0
    idx = torch.arange(s, device=DEV)
    lo_i, hi_i = idx < ng, idx >= ng + n
    for a in range(3):
        ax = 4 - a   # axis of direction a
        shp = [1] * 5
        shp[ax] = s
        x = torch.stack([x0[b][a] + (idx.double() - ng) * dx for b in range(u.shape[1])])
        shp[1] = u.shape[1]
        x = x.view(shp)
        shp[1] = 1
        r2 = r2 + x * x
        sh = lambda k: u.index_select(ax, (idx + k).clamp(0, s - 1))  # noqa: E731
        d = torch.where(lo_i.view(shp), 4 * (sh(1) - u) - (sh(2) - u),
                        torch.where(hi_i.view(shp), -4 * (sh(-1) - u) + (sh(-2) - u),
                                    sh(1) - sh(-1)))
        adv = adv + x * d / (2.0 * dx)
    flat = torch.zeros(NF, dtype=torch.float64, device=DEV)
    flat[list(ONES)] = 1.0
    return -(adv + (u - flat.view(-1, 1, 1, 1, 1))) / torch.sqrt(r2)


def _fill_from_neighbours(cur, keep, n, ng):
    """Ghosts of the 2 x 2 x 2 blocks: the neighbour's points where there is
    one, `keep` beyond the outer faces."""
    i = slice(ng, ng + n)
    cube = torch.empty(cur.shape[0], 2 * n, 2 * n, 2 * n, dtype=torch.float64, device=DEV)
    for b in range(8):
        o = [n * ((b >> a) & 1) for a in (2, 1, 0)]
        cube[:, o[0]:o[0] + n, o[1]:o[1] + n, o[2]:o[2] + n] = cur[:, b, i, i, i]
    out = keep.clone()
    for b in range(8):
        hi = [(b >> a) & 1 for a in (2, 1, 0)]
        src = [slice(n - ng, 2 * n) if h else slice(0, n + ng) for h in hi]
        dst = [slice(0, n + ng) if h else slice(ng, n + 2 * ng) for h in hi]
        out[:, b, dst[0], dst[1], dst[2]] = cube[:, src[0], src[1], src[2]]
    return out


def _exact_evolution(case, seed):
    L = Blocks(case, seed)
    u = _state(case, L, seed, _gen(seed))
    m = _matter(L, seed) if case["matter"] else None
    par, kind, halo, ng, dt = _params(case), case["kind"], case["halo"], L.ng, _dt(L)
    inner = (Ellipsis, slice(ng, -ng), slice(ng, -ng), slice(ng, -ng))
    outs = {"state": L.zeros(NF), "acc": (u * 0.25 if kind == "stage" else None)}
    if kind == "constraints" or case["monitor"]:
        outs["cons"], outs["norms"] = L.zeros(NC), torch.zeros(L.nb, 8, 2, dtype=torch.float64,
                                                               device=DEV)

    def put_constraints(bl, q, dx):
        q = torch.stack(q, 1)
        for k, b in enumerate(bl):
            L.view(outs["cons"], b, NC)[inner] = q[k]
            dv = float(dx[k]) ** 3
            outs["norms"][b, :, 0] = q[k].abs().sum((1, 2, 3)) * dv
            outs["norms"][b, :, 1] = (q[k] ** 2).sum((1, 2, 3)) * dv

    if halo in ("neighbour", "radiative"):
        n = L.dims[0][0]
        y = torch.stack([L.view(u, b, NF) for b in range(8)], 1)
        mm = (list(torch.stack([L.view(m, b, NM)[inner] for b in range(8)], 1))
              if m is not None else None)
        G = Grid(L.dims[0], ng, par.fd_order, L.dx, par.ko_sigma)
        acc, cur = torch.zeros_like(y), _fill_from_neighbours(y, y, n, ng)
        y0 = cur
        if case["monitor"]:
            put_constraints(range(8), _evaluate(G, cur, mm, par, constraints=True), L.dx)
        for co in Z.RK4:
            k = (_radiative_rhs(cur, n, ng, float(L.dx[0]), L.x0) if halo == "radiative"
                 else torch.zeros_like(cur))
            k[inner] = torch.stack(_evaluate(G, cur, mm, par))
            acc, new = _combine(k, cur, acc, y0, co, dt)
            new = torch.stack(_enforce(list(new), par))
            cur = _fill_from_neighbours(new, new if halo == "radiative" else y, n, ng)
        for b in range(8):
            L.view(outs["state"], b, NF)[...] = cur[:, b]
        return ([outs["state"]] + ([outs["cons"], outs["norms"].reshape(-1)] if case["monitor"]
                                   else []))

    for dims, bl in L.classes.items():
        G = Grid(dims, ng, par.fd_order, [L.dx[b] for b in bl], par.ko_sigma)
        cur = torch.stack([L.view(u, b, NF) for b in bl], 1)
        mm = (list(torch.stack([L.view(m, b, NM)[inner] for b in bl], 1)) if m is not None
              else None)
        if kind == "constraints":
            put_constraints(bl, _evaluate(G, cur, mm, par, constraints=True),
                            [L.dx[b] for b in bl])
            continue
        if kind == "rhs":
            r = torch.stack(_evaluate(G, cur, mm, par))
            for k, b in enumerate(bl):
                L.view(outs["state"], b, NF)[inner] = r[:, k]
            continue
        if kind == "stage":
            u0 = cur[inner]
            k = torch.stack(_evaluate(G, cur, mm, par))
            acc, new = _combine(k, u0, 0.25 * u0, u0 * (1.0 + 1e-9), RK4_STAGE2, dt)
            new = torch.stack(_enforce(list(new), par))
            for q, b in enumerate(bl):
                L.view(outs["state"], b, NF)[inner] = new[:, q]
                L.view(outs["acc"], b, NF)[inner] = acc[:, q]
            continue

        def wrap(v):   # every block periodic on itself
            for ax, nn in ((4, dims[0]), (3, dims[1]), (2, dims[2])):
                i = torch.arange(-ng, nn + ng, device=DEV) % nn
                v = v.index_select(ax, i)
            return v

        y = cur[inner].clone()
        acc, st = torch.zeros_like(y), y
        for co in Z.RK4:
            k = torch.stack(_evaluate(G, wrap(st), mm, par))
            acc, new = _combine(k, st, acc, y, co, dt)
            st = torch.stack(_enforce(list(new), par))
        st = wrap(st)
        for q, b in enumerate(bl):
            L.view(outs["state"], b, NF)[...] = st[:, q]
    if kind == "constraints":
        return [outs["cons"], outs["norms"].reshape(-1)]
    return [outs["state"], outs["acc"]] if kind == "stage" else [outs["state"]]


MIDW = {2: (0.5, 0.5), 4: (-1 / 16, 9 / 16, 9 / 16, -1 / 16),
        6: (3 / 256, -25 / 256, 150 / 256, 150 / 256, -25 / 256, 3 / 256)}


def _midpoints(v, order):
    """Lagrange values midway between points, along the last three axes."""
    for ax in (-1, -2, -3):
        n = v.shape[ax] - order + 1
        v = sum(w * v.narrow(ax, k, n) for k, w in enumerate(MIDW[order]))
    return v


def _exact_matter(c, seed):
    M, g = Cells(c["nc"]), _gen(seed)
    u = M.zeros(NF, cells=False).uniform_(-1e-6, 1e-6, generator=g)
    _metric(M.view(u, NF, cells=False), *M.coords(cells=False))
    prim = _fluid(M, g, seed)
    nc, ext = c["nc"], c["ext"]
    geom, adm, matter = M.zeros(7), M.zeros(10), M.zeros(NM, cells=False)
    cells = slice(3 - ext, 3 + nc + ext)
    box = (slice(None), slice(None), cells, cells, cells)
    o = c["order_cc"]
    lo = 4 - ext - (o // 2 - 1)
    src = M.view(u, NF, cells=False)[:, :7, lo:lo + nc + 2 * ext + o - 1,
                                     lo:lo + nc + 2 * ext + o - 1, lo:lo + nc + 2 * ext + o - 1]
    M.view(geom, 7)[box] = _midpoints(src, o)
    gv, w = M.view(geom, 7)[box], M.view(prim, 8)[box]
    gam = [gv[:, 1 + q] / gv[:, 0].clamp(min=1e-6) for q in range(6)]
    low = lambda a: [sum(gam[S(i, j)] * a[j] for j in range(3)) for i in range(3)]  # noqa: E731
    ut, Bu = [w[:, 1 + i] for i in range(3)], [w[:, 5 + i] for i in range(3)]
    ul, Bl = low(ut), low(Bu)
    Wl = torch.sqrt(1.0 + sum(a * b for a, b in zip(ut, ul)))
    v = [x / Wl for x in ul]
    ab0 = Wl * sum(a * b for a, b in zip(Bu, v))
    b2 = (ab0 * ab0 + sum(a * b for a, b in zip(Bu, Bl))) / Wl ** 2
    bl = [Bl[i] / Wl + ab0 * v[i] for i in range(3)]
    E, P = (w[:, 0] + 2.0 * w[:, 4] + b2) * Wl ** 2, w[:, 4] + 0.5 * b2
    out = [E - P - ab0 * ab0] + [E * v[i] - ab0 * bl[i] for i in range(3)]
    out += [E * v[i] * v[j] + P * gam[S(i, j)] - bl[i] * bl[j] for i in range(3)
            for j in range(i, 3)]
    M.view(adm, 10)[box] = torch.stack(out, 1)
    o = c["order_vc"]
    lo, n = 3 - o // 2, nc + 1 + o - 1
    a = M.view(adm, 10)[:, :, lo:lo + n, lo:lo + n, lo:lo + n]
    verts = slice(4, 4 + nc + 1)
    M.view(matter, NM, cells=False)[:, :, verts, verts, verts] = _midpoints(a, o)
    return [geom, adm, matter]


def _exact_recovery(c, seed):
    M, geom, prim, cons = _recovery_data(c, seed)
    a, nc, ext = _atm(), c["nc"], c["ext"]
    cells = slice(3 - ext, 3 + nc + ext)
    box = (slice(None), slice(None), cells, cells, cells)
    v = M.view(prim, 8)
    atm = v.clone()
    atm[:, 0], atm[:, 1:4], atm[:, 4] = a["rho_atm"], 0.0, a["p_atm"]
    # every velocity of the data is far below the ceiling, so D or rho below
    # the threshold is what makes a cell atmosphere
    is_atm = (v[:, 0] < a["rho_atm"])[:, None]
    want = torch.where(is_atm, atm, v)
    p = M.zeros(8)
    M.view(p, 8)[box] = want[box]
    if not c["mhd"]:
        M.view(p, 8)[:, 5:] = 0.0
    full = M.zeros(8)
    M.view(full, 8)[...] = want
    new, q = _conserved(M, geom, full, c["mhd"]), cons.clone()
    M.view(q, 8)[box] = torch.where(is_atm, M.view(new, 8), M.view(cons, 8))[box]
    return [p, q, None]


def _exact_exchange(c, seed):
    t, u, pro, res, src, st, npts = _exchange_parts(c, seed)
    n, nco, o = c["n"], c["ncoarse"], c["order"]
    s = n + 8
    v = u.view(9 * nco, NF, st)[:, :, :npts].unflatten(2, (s, s, s))
    h = n // 2
    even = slice(4, 4 + n, 2)
    for k in range(8):
        b = [slice(4 + h * ((k >> d) & 1), 4 + h * ((k >> d) & 1) + h) for d in (2, 1, 0)]
        v[:nco, :, b[0], b[1], b[2]] = v[nco + k::8][:, :, even, even, even]
    # interpolation matrix of fine index i (rows) from coarse index - 4 (columns)
    mat = torch.zeros(s, s, dtype=torch.float64, device=DEV)
    for i in range(-4, n + 4):
        if i % 2 == 0:
            mat[i + 4, 4 + 4 + i // 2] = 1.0
        else:
            first = 4 + (i - 1) // 2 - (o // 2 - 1)
            for k, w in enumerate(MIDW[o]):
                if 0 <= 4 + first + k < s:
                    mat[i + 4, 4 + first + k] = w
    src = torch.from_numpy(src).to(DEV)
    for q in range(6):
        rng = [slice(4, 4 + n)] * 3
        rng[q // 2] = slice(0, 4) if q % 2 == 0 else slice(4 + n, 8 + n)
        for lo in range(0, 8 * nco, 64):
            w = v[src[lo:lo + 64, q]]
            w = torch.tensordot(w, mat[rng[0]], dims=([4], [1]))             # x
            w = torch.tensordot(w, mat[rng[1]], dims=([3], [1])).transpose(3, 4)   # y
            w = torch.tensordot(w, mat[rng[2]], dims=([2], [1])).permute(0, 1, 4, 2, 3)
            v[nco + lo:nco + lo + 64, :, rng[2], rng[1], rng[0]] = w
    return [u]


def exact(case, seed):
    if case["kind"] == "matter":
        return _exact_matter(case, seed)
    if case["kind"] == "recovery":
        return _exact_recovery(case, seed)
    if case["kind"] == "exchange":
        return _exact_exchange(case, seed)
    return _exact_evolution(case, seed)
