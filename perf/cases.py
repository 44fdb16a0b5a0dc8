"""Performance cases of the FMM solver: what a program calls, over the range it calls it in.

A case names one kind of pass through the public entry points of
``paper_1712_10116_amd.fmm`` and its sizes:

forces   one complete Poisson solve (``Solver.forces``)
kicks    one tree over an active subset and two evaluations of it, the masses
         of the fast particles zeroed in the first (``build``, ``evaluate``)
grad     the forces with their gradient, then the field of the vector sources
         m_j a_j on the same tree (``forces_grad``, ``evaluate_dipole``): what
         one modified kick of the fourth-order integrator evaluates
hhs      one top-level step of the hierarchical integrator of one system from
         a snapshot (``HHS.init``, ``HHS.step``)
serve    a batch of simulation requests handed to the request server as host
         arrays and run to their end (``Server``)

Solver parameters are those of the repository's workloads (``workloads.PARAMS``),
of the benchmark's tuned configuration, or of the paper's cold collapse.
"""
import math

import numpy as np
import torch

import paper_1712_10116_amd.fmm as F
from paper_1712_10116_amd import workloads as W

# softening of each particle distribution
EPS = {"plummer": 0.01, "sphere": 0.005, "disk": 0.02, "zoom": 0.001}
LEAVES = (16, 24, 32, 48, 64, 96, 128)
# Integrator parameters: those of the serving ensemble at the opening angle of the
# paper's cold collapse.  At 0.5 every pair of equal cells two cells apart lies
# exactly on the threshold of the opening test, where the last bit of a position
# decides it, so that trajectories could only be compared bit for bit; at 0.45 no
# pair of cells does.
RUN = dict(eps=0.01, theta=0.45, p=4, eta=0.0025, max_levels=10)
DT_TOP = 1.0 / 16
# force particles of one top-level step per particle of the system, measured
# on the ensemble's systems (an estimate for work(): it depends on the rungs)
STEP_EVALS = 130


def _forces(n, dist, kernel, mixed, p, theta, leaf, predict=False, eps=None, **more):
    return dict(kind="forces", n=n, dist=dist, kernel=kernel, mixed=mixed, p=p, theta=theta,
                leaf=leaf, eps=EPS[dist] if eps is None else eps, predict=predict, **more)


def listed():
    return [
        # the smallest systems: one deep rung's active set, or a small cluster
        _forces(1000, "plummer", "plummer", False, 4, 0.5, 16, name="forces 1000 fp64"),
        # the 4096-particle Plummer workload
        _forces(4096, "plummer", "plummer", False, 4, 0.5, 16, name="forces 4096 fp64"),
        # a middle-sized system of the serving ensemble
        _forces(12526, "plummer", "wendland", True, 4, 0.5, 64, name="forces 12526 mixed"),
        # the paper's cold collapse: theta 0.45, p 5, 64 per leaf, softening
        # 0.01 (N / 10^4)^(-1/3); an odd size
        _forces(100003, "sphere", "wendland", False, 5, 0.45, 64, eps=0.00464,
                name="forces 100003 fp64"),
        # a reference-quality double-precision solve of a few 10^5 particles
        _forces(300007, "plummer", "wendland", False, 6, 0.5, 96, name="forces 300007 fp64"),
        # the benchmark's headline: a steady loop over 2^20 particles
        _forces(1 << 20, "sphere", "wendland", True, 6, 0.5, 96, predict=True,
                name="forces 2^20 mixed"),
        # the disk-galaxy workload
        _forces(1 << 22, "disk", "wendland", True, 6, 0.4, 96, name="forces disk 2^22 mixed"),
        # the clustered-zoom workload, the largest solve
        _forces(1 << 24, "zoom", "wendland", True, 6, 0.4, 64, name="forces zoom 2^24 mixed"),
        # one rung of a large run: an eighth of the particles is active
        dict(kind="kicks", n=1 << 20, active=131073, dist="sphere", kernel="wendland",
             mixed=True, p=6, theta=0.5, leaf=96, eps=0.005, name="kicks 131073 of 2^20 mixed"),
        # the fourth-order integrator's Plummer sphere
        dict(kind="grad", n=65536, dist="plummer", kernel="plummer", mixed=False, p=6,
             theta=0.4, leaf=64, eps=0.1, name="grad 65536 fp64"),
        # a single small system integrated alone
        dict(kind="hhs", n=12526, mixed=True, leaf=64, name="hhs 12526 mixed"),
        # a batch of ensemble simulations, each one top-level step long
        dict(kind="serve", requests=24, n_min=1024, n_max=131072, mixed=True, leaf=64,
             name="serve 24 requests mixed"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(("forces",) * 6 + ("kicks", "grad", "hhs", "serve"))
    if kind == "hhs":
        return dict(kind="hhs", n=_log_int(rng, 1024, 100000), mixed=rng.random() < 0.75,
                    leaf=rng.choice((32, 64)))
    if kind == "serve":
        return dict(kind="serve", requests=rng.randint(4, 24), n_min=1024,
                    n_max=_log_int(rng, 4096, 100000), mixed=True, leaf=64)
    if kind == "grad":
        return dict(kind="grad", n=_log_int(rng, 2000, 131072), dist="plummer",
                    kernel=rng.choice(("plummer", "wendland")), mixed=rng.random() < 0.25,
                    p=rng.choice((4, 5, 6)), theta=rng.choice((0.4, 0.45, 0.5)),
                    leaf=rng.choice((32, 64)), eps=rng.choice((0.01, 0.1)))
    dist = rng.choice(("plummer", "sphere", "sphere", "disk", "zoom"))
    c = dict(dist=dist, kernel=rng.choice(("wendland", "wendland", "plummer")),
             mixed=rng.random() < 0.6, p=rng.choice((4, 5, 6)),
             theta=rng.choice((0.4, 0.45, 0.5, 0.55, 0.6)), leaf=rng.choice(LEAVES),
             eps=EPS[dist])
    if kind == "kicks":
        n = _log_int(rng, 20000, 1 << 21)
        return dict(kind="kicks", n=n, active=_log_int(rng, 1000, n // 2), **c)
    return dict(kind="forces", n=_log_int(rng, 1000, 1 << 21), predict=rng.random() < 0.25, **c)


# ---------------------------------------------------------------------------
# inputs, drawn on the GPU (the numpy generators of the workloads take seconds
# at the large sizes)
# ---------------------------------------------------------------------------
def _uniform(g, *shape):
    return torch.rand(*shape, dtype=torch.float64, device="cuda", generator=g)


def _directions(g, n):
    cz = 2.0 * _uniform(g, n) - 1.0
    ph = 2.0 * math.pi * _uniform(g, n)
    sz = (1.0 - cz * cz).clamp_(min=0.0).sqrt_()
    return torch.stack([sz * ph.cos(), sz * ph.sin(), cz])


def _inverse(cdf, x_hi, u):
    """x in [0, x_hi] with cdf(x) / cdf(x_hi) = u, linear between 20000 nodes."""
    x = torch.linspace(0.0, x_hi, 20000, dtype=torch.float64, device="cuda")
    c = cdf(x)
    c = c / c[-1].clone()
    k = torch.searchsorted(c, u, right=True).clamp_(1, 19999)
    f = (u - c[k - 1]) / (c[k] - c[k - 1])
    return x[k - 1] + f * (x[k] - x[k - 1])


def _nfw(x):
    return torch.log1p(x) - x / (1.0 + x)


def _particles(dist, n, seed):
    """(pos (3, n), mass (n)) of one of the workloads' distributions."""
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    if dist == "plummer":
        x = (0.999 * _uniform(g, n)).clamp_(min=1e-12)
        pos = _directions(g, n) / (x.pow(-2.0 / 3.0) - 1.0).sqrt_()
        w = torch.ones(n, dtype=torch.float64, device="cuda")
    elif dist == "sphere":
        pos = _uniform(g, n).pow(1.0 / 3.0) * _directions(g, n)
        w = torch.ones(n, dtype=torch.float64, device="cuda")
    elif dist == "disk":
        nd, nb = n // 4, n // 8
        nh = n - nd - nb
        r = _inverse(lambda x: 1.0 - (1.0 + x) * torch.exp(-x), 10.0, _uniform(g, nd))
        ph = 2.0 * math.pi * _uniform(g, nd)
        z = 0.1 * torch.atanh((2.0 * _uniform(g, nd) - 1.0).clamp_(-0.999999, 0.999999))
        s = (0.999 * _uniform(g, nb)).sqrt_()
        pos = torch.cat([torch.stack([r * ph.cos(), r * ph.sin(), z]),
                         0.2 * s / (1.0 - s) * _directions(g, nb),
                         6.0 * _inverse(_nfw, 20.0, _uniform(g, nh)) * _directions(g, nh)], 1)
        w = torch.ones(n, dtype=torch.float64, device="cuda")
        w[nd + nb:] = 8.0
    else:  # zoom: 2000 halos, dN/dM ~ M^-1.9 on [1, 1e3], and a uniform background
        rng = np.random.default_rng(seed)
        nbg = n // 5
        nh = n - nbg
        mh = (1.0 + rng.uniform(0, 1, 2000) * (1e3 ** -0.9 - 1.0)) ** (1.0 / -0.9)
        cnt = np.floor(mh / mh.sum() * nh).astype(np.int64)
        cnt[np.argmax(mh)] += nh - cnt.sum()
        r200 = 0.05 * (mh / mh.max()) ** (1.0 / 3.0)
        ctr = torch.from_numpy(rng.uniform(0.25, 0.75, (3, 2000))).cuda()
        h = torch.repeat_interleave(torch.arange(2000, device="cuda"),
                                    torch.from_numpy(cnt).cuda(), output_size=nh)
        r = torch.from_numpy(r200 / 10.0).cuda()[h] * _inverse(_nfw, 10.0, _uniform(g, nh))
        pos = torch.cat([ctr[:, h] + r * _directions(g, nh), _uniform(g, 3, nbg)], 1)
        w = torch.ones(n, dtype=torch.float64, device="cuda")
        w[nh:] = 8.0
    return pos.contiguous(), w / w.sum()


def _system(i, n, seed):
    """(pos, vel, mass) host arrays: Plummer spheres and King models in turn."""
    if i % 2 == 0:
        return W.plummer(n, seed=seed, a=3.0 * np.pi / 16.0)
    return W.king(n, seed=seed, henon=True)


def _request_sizes(case):
    """Sizes of a serving batch, even in the logarithm from n_min to n_max."""
    k = case["requests"]
    lo, hi = math.log(case["n_min"]), math.log(case["n_max"])
    return [int(math.exp(lo + (hi - lo) * (i + 0.5) / k)) for i in range(k)]


def _solver(case, n, p_max):
    return F.Solver(n, p_max=p_max, leaf_size=case["leaf"],
                    kernel=F.PLUMMER if case.get("kernel") == "plummer" else F.WENDLAND,
                    precision=F.MIXED if case["mixed"] else F.FP64)


def _fast_active(case, seed):
    """The active subset (sorted indices) and the half of it that is fast."""
    g = torch.Generator(device="cuda")
    g.manual_seed(seed + 77)
    act = torch.randperm(case["n"], device="cuda", generator=g)[:case["active"]]
    act = act.sort().values
    return act, act[torch.rand(case["active"], device="cuda", generator=g) < 0.5]


def prepare(case, seed):
    s = dict(case=case)
    if case["kind"] == "serve":
        sizes = _request_sizes(case)
        s["requests"] = [_system(i, n, 100 * seed + i) for i, n in enumerate(sizes)]
        s["solver"] = _solver(case, max(1 << 18, sum(sizes)), RUN["p"])
        foot = sum(F.Server.footprint(n, RUN["max_levels"]) + 4096 for n in sizes)
        s["server"] = F.Server(s["solver"], arena_bytes=foot, max_slots=case["requests"],
                               dt_max=DT_TOP, **RUN)
        return s
    if case["kind"] == "hhs":
        pos, vel, mass = (torch.from_numpy(a).cuda() for a in _system(0, case["n"], seed))
        s["solver"] = _solver(case, case["n"], RUN["p"])
        s["start"] = (pos, vel)
        s["hhs"] = F.HHS(s["solver"], pos.clone(), vel.clone(), mass, **RUN)
        return s
    pos, mass = _particles(case["dist"], case["n"], seed)
    n = case.get("active", case["n"])
    s.update(pos=pos, mass=mass, solver=_solver(case, n, case["p"]))
    if case.get("predict"):
        s["solver"].set_level_prediction(True)
    if case["kind"] == "kicks":
        act, fast = _fast_active(case, seed)
        masked = mass.clone()
        masked[fast] = 0.0
        s.update(active=act.to(torch.int32), masked=masked)
    if case["kind"] != "grad":
        s["out"] = [(torch.empty((3, n), dtype=torch.float64, device="cuda"),
                     torch.empty(n, dtype=torch.float64, device="cuda")) for _ in range(2)]
    return s


def run(s):
    case, solver = s["case"], s["solver"]
    kind = case["kind"]
    if kind == "forces":
        acc, pot = s["out"][0]
        return solver.forces(s["pos"], s["mass"], eps=case["eps"], theta=case["theta"],
                             p=case["p"], acc=acc, pot=pot)
    if kind == "kicks":
        solver.build(s["pos"], s["active"], eps=case["eps"], theta=case["theta"])
        return [solver.evaluate(s["pos"], m, s["active"], p=case["p"], acc=acc, pot=pot)
                for m, (acc, pot) in zip((s["masked"], s["mass"]), s["out"])]
    if kind == "grad":
        acc, pot, grad = solver.forces_grad(s["pos"], s["mass"], eps=case["eps"],
                                            theta=case["theta"], p=case["p"])
        u, phi = solver.evaluate_dipole(s["pos"], s["mass"], acc, p=case["p"])
        return acc, pot, grad, u, phi
    if kind == "hhs":
        h = s["hhs"]
        h.pos.copy_(s["start"][0])
        h.vel.copy_(s["start"][1])
        h.init()
        h.step(DT_TOP)
        return h.pos, h.vel, h.a_cur, h.rung
    srv = s["server"]
    ids = [srv.submit(pos, vel, mass, DT_TOP) for pos, vel, mass in s["requests"]]
    got = {}
    while len(got) < len(ids):
        srv.step()
        for r in srv.poll():
            got[r["id"]] = r
    return (np.concatenate([got[i]["pos"] for i in ids], axis=1),
            np.concatenate([got[i]["vel"] for i in ids], axis=1))


# ---------------------------------------------------------------------------
# the work a pass cannot do without
# ---------------------------------------------------------------------------
def _solve_flops(n, p, theta, leaf):
    """Multiply-adds (as two operations) of one force solve.

    A leaf's neighbours are the cells within its side / theta, about
    4 pi / (3 theta^3) of them, and each cell's M2L partners the children of
    its parent's neighbours that are not its own, about 7 times as many.  Leaves
    hold about 0.55 of the leaf size.  30 operations per unordered particle
    pair, 4 C(p+6, 6) + 2 C(p+3, 3) (p + 1) per unordered cell pair."""
    per = max(1.0, 0.55 * leaf)
    cells = n / per
    near = 4.0 * math.pi / (3.0 * theta ** 3)
    pairs = 0.5 * n * min(n, near * per)
    far = 0.5 * (8.0 / 7.0) * cells * min(cells, 7.0 * near)
    m2l = 4 * math.comb(p + 6, 6) + 2 * math.comb(p + 3, 3) * (p + 1)
    return 30.0 * pairs + m2l * far + 2.0 * 5 * math.comb(p + 3, 3) * n


def work(case):
    kind = case["kind"]
    if kind in ("hhs", "serve"):
        sizes = [case["n"]] if kind == "hhs" else _request_sizes(case)
        n = sum(sizes)
        flops = sum(_solve_flops(k, RUN["p"], RUN["theta"], case["leaf"]) for k in sizes)
        # pos, vel, mass in, pos and vel out; hhs also gives |a| and the rungs
        return dict(bytes=n * (56 + 48 + (12 if kind == "hhs" else 0)), flops=STEP_EVALS * flops)
    flops = _solve_flops(case.get("active", case["n"]), case["p"], case["theta"], case["leaf"])
    n = case["n"]
    if kind == "forces":
        return dict(bytes=64 * n, flops=flops)
    if kind == "kicks":  # positions, two sets of masses and indices in, two results out
        return dict(bytes=case["active"] * (24 + 16 + 4 + 64), flops=2 * flops)
    # forces, their gradient and the vector pass: positions, masses, then acc,
    # pot, the six gradient terms, u and phi
    return dict(bytes=n * (32 + 32 + 48 + 32), flops=3 * flops)


# ---------------------------------------------------------------------------
# direct summation in 64 bits
# ---------------------------------------------------------------------------
def _direct(pos, mass, eps, kernel, vec=None):
    """Forces and potentials of all pairs, and with vec (a function of the
    accelerations) the force gradient and the field of the sources m_j vec_j."""
    n = pos.shape[1]
    rows = max(1, (1 << 27) // n)
    acc = torch.empty((3, n), dtype=torch.float64, device="cuda")
    pot = torch.empty(n, dtype=torch.float64, device="cuda")
    grad = torch.empty((6, n), dtype=torch.float64, device="cuda")

    def chunk(a, b, second):
        """d = x_j - x_i, psi, g = psi'/r and (second) h = (dg/dr)/r, 0 for the self pairs."""
        d = [pos[k, None, :] - pos[k, a:b, None] for k in range(3)]
        r2 = d[0] * d[0]
        r2.addcmul_(d[1], d[1]).addcmul_(d[2], d[2])
        i = torch.arange(b - a, device="cuda")
        if kernel == "plummer":
            r2.add_(eps * eps)
        else:
            ins = (r2 < eps * eps).nonzero(as_tuple=True)
            u = r2[ins].sqrt() / eps
            r2[ins] = eps * eps
        ri = r2.rsqrt_()
        g = ri * ri
        h = -3.0 * g * g * ri if second else None
        g.mul_(ri)
        psi = ri.neg_()
        if kernel != "plummer":
            psi[ins] = _psi_in(u) / eps
            g[ins] = _g_in(u) / eps ** 3
            if second:
                h[ins] = _h_in(u) / eps ** 5
        for w in (psi, g, h):
            if w is not None:
                w[i, a + i] = 0.0
        return d, psi, g, h

    for a in range(0, n, rows):
        b = min(n, a + rows)
        d, psi, g, h = chunk(a, b, vec is not None)
        pot[a:b] = psi @ mass
        gm = g * mass
        for k in range(3):
            acc[k, a:b] = (gm * d[k]).sum(1)
        if vec is not None:
            tr = gm.sum(1)
            hm = h.mul_(mass)
            for q, (i, j) in enumerate(((0, 0), (1, 1), (2, 2), (0, 1), (0, 2), (1, 2))):
                grad[q, a:b] = -(hm * d[i] * d[j]).sum(1) - (tr if i == j else 0.0)
    if vec is None:
        return acc, pot
    v = vec(acc)
    u = torch.empty_like(acc)
    phi = torch.empty_like(pot)
    for a in range(0, n, rows):
        b = min(n, a + rows)
        d, psi, g, h = chunk(a, b, True)
        dv = d[0] * v[0]
        dv.addcmul_(d[1], v[1].expand_as(dv)).addcmul_(d[2], v[2].expand_as(dv))
        dv.mul_(mass)
        phi[a:b] = -(dv * g).sum(1)
        dv.mul_(h)
        for k in range(3):
            u[k, a:b] = (g @ (mass * v[k])) + (dv * d[k]).sum(1)
    return acc, pot, grad, u, phi


# Wendland C2 inside the radius, u = r / eps: psi, (dpsi/dr)/r, (dg/dr)/r
def _psi_in(u):
    u2 = u * u
    return -(3.0 + u2 * (-7.0 + u2 * (21.0 + u * (-28.0 + u * (15.0 - 3.0 * u)))))


def _g_in(u):
    u2 = u * u
    return 14.0 + u2 * (-84.0 + u * (140.0 + u * (-90.0 + 21.0 * u)))


def _h_in(u):
    return -168.0 + u * (420.0 + u * (-360.0 + 105.0 * u))


def exact(case, seed):
    n = case.get("active", case.get("n", 0))
    if case["kind"] in ("hhs", "serve") or n > 320000:
        return None  # a trajectory, or more pairs than direct summation takes in seconds
    pos, mass = _particles(case["dist"], case["n"], seed)
    eps, kernel = case["eps"], case["kernel"]
    if case["kind"] == "forces":
        return _direct(pos, mass, eps, kernel)
    if case["kind"] == "grad":
        return _direct(pos, mass, eps, kernel, vec=lambda acc: acc)
    act, fast = _fast_active(case, seed)
    masked = mass.clone()
    masked[fast] = 0.0
    sub = pos[:, act].contiguous()
    return [_direct(sub, m[act], eps, kernel) for m in (masked, mass)]
