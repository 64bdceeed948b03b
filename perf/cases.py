"""Timing cases of the public entry points: what a program using this package
has it do, over the sizes it is used at.

A case is one pass through the Python entry points (``md.Simulation``,
``md.Batch``, ``adjoint.trajectory_observables``) as a program calls them.
Kinds:

  run    leapfrog steps of one system with neighbor lists (tiled pipeline,
         slots reordered at every rebuild): the main use of the package, from
         500 atoms, where launches and latency count, to 2.048 million.
         Soft spheres (WCA) and Lennard-Jones, FP64 and FP32-mixed
  cells  leapfrog steps of a small soft-sphere system straight from its cells
         (no list, cells rebuilt every step)
  frame  a new configuration evaluated: positions in, cells, list, forces in
         the caller's order and the observables out (external integrators,
         trajectory re-analysis)
  batch  many independent soft-sphere replicas of mixed sizes and densities
         advanced together (FP32-mixed, one graph launch per call)
  melt   leapfrog steps of a bonded polymer melt (FENE bonds, bending)
  grad   the gradient of a trajectory's observables (mean energy, soft g(r))
         with respect to the initial state and the potential parameters,
         forward and backward through torch.autograd

Initial states are seeded: jittered FCC sites (a random subset of them when
the atom count is not 4 m^3) with thermal velocities; the steps of repeated
passes melt them.
"""
import math

import numpy as np
import torch

from paper_2003_14061_amd import adjoint, md

WCA_CUT = 2.0 ** (1.0 / 6.0)
SKIN = 0.3
# state points of the workloads: cutoff, density, temperature, time step, and the
# jitter of the starting lattice
POINTS = {
    "wca": dict(r_cut=WCA_CUT, rho=0.8, T=1.0, dt=0.005, jitter=0.05),
    "lj": dict(r_cut=2.5, rho=0.8442, T=0.72, dt=0.004, jitter=0.03),
}
GRAD_RHO, GRAD_T, GRAD_DT, GRAD_BINS, GRAD_RMAX = 0.8, 1.0, 0.004, 50, 2.5
MELT_RHO, MELT_DT, FENE_K, FENE_R0, BEND_K = 0.85, 0.005, 30.0, 1.5, 1.5


# ---- the cases ----

def listed():
    return [
        # the smallest replica of the ensemble workload on its own, sampled: launches
        # and latency are all there is
        dict(name="run_wca_500", kind="run", model="wca", n=500, steps=50, every=10,
             precision="fp64"),
        # the 4000-atom cells-only workload
        dict(name="cells_wca_4000", kind="cells", n=4000, rho=0.8, steps=50, precision="fp64"),
        # an ordinary small liquid, an odd atom count
        dict(name="run_lj_10007", kind="run", model="lj", n=10007, steps=50, every=10,
             precision="fp64"),
        # a mid-sized liquid in mixed precision
        dict(name="run_lj_32k_fp32", kind="run", model="lj", n=32000, steps=20, every=0,
             precision="fp32"),
        # the 256 000-atom soft-sphere workload
        dict(name="run_wca_256k", kind="run", model="wca", n=256000, steps=20, every=0,
             precision="fp64"),
        # the 2.048 million atom Lennard-Jones workload, both precisions
        dict(name="run_lj_2048k", kind="run", model="lj", n=2048000, steps=20, every=0,
             precision="fp64"),
        dict(name="run_lj_2048k_fp32", kind="run", model="lj", n=2048000, steps=20, every=0,
             precision="fp32"),
        # one configuration evaluated, a ragged size
        dict(name="frame_lj_100003", kind="frame", model="lj", n=100003, precision="fp64"),
        # the 64-replica ensemble workload
        dict(name="batch_64", kind="batch", replicas=64, n_lo=500, n_hi=32000, steps=20,
             precision="fp32"),
        # the 262 144-atom polymer melt workload
        dict(name="melt_256k", kind="melt", side=64, chain=64, steps=20, precision="fp64"),
        # the differentiable 32 000-atom workload (fewer steps), and a small one
        dict(name="grad_lj_32k", kind="grad", n=32000, steps=40, checkpoint=20,
             precision="fp64"),
        dict(name="grad_lj_4000", kind="grad", n=4000, steps=40, checkpoint=20,
             precision="fp64"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """A case of the listed ones' ranges; sizes over their logarithm."""
    kind = rng.choice(["run", "run", "run", "run", "cells", "frame", "batch", "melt", "grad"])
    precision = rng.choice(["fp64", "fp64", "fp32"])
    if kind == "run":
        model = rng.choice(["wca", "lj"])
        n = _log_int(rng, 500 if model == "wca" else 640, 2048000)
        steps = rng.randint(20, 50) if n < 100000 else rng.randint(10, 20)
        return dict(kind=kind, model=model, n=n, steps=steps, every=rng.choice([0, 1, 10]),
                    precision=precision)
    if kind == "cells":
        return dict(kind=kind, n=_log_int(rng, 500, 30000), rho=rng.uniform(0.6, 0.9),
                    steps=rng.randint(20, 50), precision=precision)
    if kind == "frame":
        model = rng.choice(["wca", "lj"])
        return dict(kind=kind, model=model, n=_log_int(rng, 1000, 400000), precision=precision)
    if kind == "batch":
        lo = rng.randint(500, 2000)
        return dict(kind=kind, replicas=rng.randint(4, 64), n_lo=lo,
                    n_hi=lo + _log_int(rng, 500, 30000), steps=rng.randint(10, 20),
                    precision=rng.choice(["fp32", "fp32", "fp64"]))
    if kind == "melt":
        side = rng.choice([12, 16, 20, 24, 32, 40, 48, 64])
        chain = rng.choice([m for m in (4, 8, 16, 32, 64) if side ** 3 % m == 0])
        return dict(kind=kind, side=side, chain=chain, steps=rng.randint(10, 20),
                    precision=precision)
    return dict(kind=kind, n=_log_int(rng, 1000, 32000), steps=rng.randint(10, 40),
                checkpoint=rng.choice([10, 20]), precision=precision)


# ---- inputs (numpy, from the seed alone) ----

def _lattice(n, L, rng):
    m = 1
    while 4 * m ** 3 < n:
        m += 1
    g = np.arange(m, dtype=np.float64)
    cells = np.stack(np.meshgrid(g, g, g, indexing="ij"), -1)[..., ::-1].reshape(-1, 1, 3)
    basis = np.array([[0, 0, 0], [.5, .5, 0], [.5, 0, .5], [0, .5, .5]]) + 0.25
    sites = ((cells + basis) * (L / m)).reshape(-1, 3)
    if len(sites) > n:
        sites = sites[np.sort(rng.choice(len(sites), size=n, replace=False))]
    return sites


def _thermal(n, T, rng):
    v = rng.standard_normal((n, 3))
    v -= v.mean(0)
    return v * math.sqrt(T * 3.0 * (n - 1) / float((v * v).sum()))


def _jittered(pos, L, amp, rng):
    p = np.mod(pos + amp * rng.standard_normal(pos.shape), L)
    p[p >= L] = 0.0
    return p


def _system(n, rho, T, jitter, rng):
    L = (n / rho) ** (1.0 / 3.0)
    pos = _jittered(_lattice(n, L, rng), L, jitter, rng)
    return pos, _thermal(n, T, rng), L


def _snake(side, L):
    """Simple-cubic sites along a path whose consecutive sites are neighbors."""
    x = np.arange(side)
    out = []
    for z in range(side):
        ys = x if z % 2 == 0 else x[::-1]
        for k, y in enumerate(ys):
            fwd = (z * side + k) % 2 == 0
            xs = x if fwd else x[::-1]
            out.append(np.stack([xs, np.full(side, y), np.full(side, z)], 1))
    return (np.concatenate(out) + 0.5) * (L / side)


def _single(case, seed):
    """pos, vel, L and the method parameters of a one-system case."""
    rng = np.random.default_rng([int(seed), 11])
    if case["kind"] == "melt":
        n = case["side"] ** 3
        L = (n / MELT_RHO) ** (1.0 / 3.0)
        # a cool start: the lattice's bonds are stretched and release about 3 eps per
        # atom, after which the melt is near T = 1 (hotter ones break bonds)
        pos = _jittered(_snake(case["side"], L), L, 0.01, rng)
        return pos, _thermal(n, 0.1, rng), L, dict(r_cut=WCA_CUT, dt=MELT_DT)
    if case["kind"] == "grad":
        pos, vel, L = _system(case["n"], GRAD_RHO, GRAD_T, 0.03, rng)
        return pos, vel, L, dict(r_cut=2.5, dt=GRAD_DT)
    pt = dict(POINTS[case.get("model", "wca")])
    if "rho" in case:
        pt["rho"] = case["rho"]
    pos, vel, L = _system(case["n"], pt["rho"], pt["T"], pt["jitter"], rng)
    return pos, vel, L, dict(r_cut=pt["r_cut"], dt=pt["dt"])


def _replicas(case, seed):
    rng = np.random.default_rng([int(seed), 12])
    # sizes and densities are the case's, states the seed's
    spec = np.random.default_rng([4, case["replicas"], case["n_lo"], case["n_hi"]])
    out = []
    for _ in range(case["replicas"]):
        n = int(spec.integers(case["n_lo"], case["n_hi"] + 1))
        pos, vel, L = _system(n, float(spec.uniform(0.6, 0.9)), 1.0, 0.02, rng)
        out.append(dict(pos=pos, vel=vel, L=L, r_cut=WCA_CUT, dt=0.005, skin=SKIN))
    return out


def _target(seed):
    """The g(r) a gradient case fits to."""
    g = torch.Generator().manual_seed(int(seed))
    return 1.0 + 0.1 * torch.randn(GRAD_BINS, generator=g, dtype=torch.float64)


# ---- what a program holds before the call ----

def prepare(case, seed):
    kind = case["kind"]
    st = dict(case=case)
    if kind == "batch":
        b = md.Batch(_replicas(case, seed), precision=case["precision"])
        b.prepare()
        st["batch"] = b
        return st
    pos, vel, L, kw = _single(case, seed)
    if kind == "grad":
        st["x0"] = torch.tensor(pos, device="cuda")
        st["v0"] = torch.tensor(vel, device="cuda")
        st["target"] = _target(seed).cuda()
        st["spec"] = adjoint.TrajectorySpec(
            L=L, n_steps=case["steps"], dt=kw["dt"], skin=SKIN, precision=case["precision"],
            checkpoint_every=case["checkpoint"], n_bins=GRAD_BINS, gr_rmax=GRAD_RMAX)
        return st
    if kind == "melt":
        kw["bonded"] = dict(chain_length=case["chain"], fene_k=FENE_K, fene_r0=FENE_R0,
                            bend_k=BEND_K)
    if kind == "frame":
        kw["reorder"] = False  # forces in the caller's order
    sim = md.Simulation(pos, vel, L, skin=SKIN, precision=case["precision"],
                        neighbor_list=kind != "cells", **kw)
    st["sim"] = sim
    if kind == "frame":
        st["frame"] = [torch.tensor(np.ascontiguousarray(pos[:, k]), device="cuda")
                       for k in range(3)]
    else:
        sim.prepare()
    return st


def run(state):
    case, kind = state["case"], state["case"]["kind"]
    if kind == "batch":
        b = state["batch"]
        b.run(case["steps"])
        torch.cuda.current_stream().wait_stream(b.stream)
        return dict(x=b.x, y=b.y, z=b.z, vx=b.vx, vy=b.vy, vz=b.vz, fx=b.fx, fy=b.fy, fz=b.fz,
                    id=b.id)
    if kind == "grad":
        x0 = state["x0"].detach().requires_grad_(True)
        v0 = state["v0"].detach().requires_grad_(True)
        eps = torch.tensor(1.0, dtype=torch.float64, requires_grad=True)
        sigma = torch.tensor(1.0, dtype=torch.float64, requires_grad=True)
        ubar, g = adjoint.trajectory_observables(x0, v0, eps, sigma, state["spec"])
        loss = ubar + ((g - state["target"]) ** 2).sum()
        loss.backward()
        return dict(ubar=ubar.detach(), g=g.detach(), x0=x0.grad, v0=v0.grad, eps=eps.grad,
                    sigma=sigma.grad)
    sim = state["sim"]
    if kind == "frame":
        for dst, src in zip((sim.x, sim.y, sim.z), state["frame"]):
            dst.copy_(src)
        sim.prepare()
        o = sim.reduce()
        return dict(fx=sim.fx, fy=sim.fy, fz=sim.fz, U=o["U"], W=o["W"], K=o["K"])
    sim.step(case["steps"], record_every=case.get("every", 0))
    return dict(x=sim.x, y=sim.y, z=sim.z, vx=sim.vx, vy=sim.vy, vz=sim.vz, fx=sim.fx, fy=sim.fy,
                fz=sim.fz, id=sim.id)


# ---- what a pass cannot do without ----

def work(case):
    """Bytes: per step every position and velocity read and written once, and per
    pass the forces written.  Operations: per step, 27 for each pair inside the
    cutoff met once (separation and its square 8, force, energy and virial 16,
    and the partner's sum 3); a gradient's backward walk takes twice that."""
    kind = case["kind"]
    fsz = 8 if case["precision"] == "fp64" else 4
    if kind == "batch":
        spec = np.random.default_rng([4, case["replicas"], case["n_lo"], case["n_hi"]])
        systems = [(int(spec.integers(case["n_lo"], case["n_hi"] + 1)),
                    float(spec.uniform(0.6, 0.9)), WCA_CUT) for _ in range(case["replicas"])]
    elif kind == "melt":
        systems = [(case["side"] ** 3, MELT_RHO, WCA_CUT)]
    elif kind == "grad":
        systems = [(case["n"], GRAD_RHO, 2.5)]
    else:
        pt = POINTS[case.get("model", "wca")]
        systems = [(case["n"], case.get("rho", pt["rho"]), pt["r_cut"])]
    nbytes = flops = 0.0
    for n, rho, rc in systems:
        pairs = 0.5 * n * 4.0 / 3.0 * math.pi * rc ** 3 * rho
        if kind == "frame":
            nbytes += n * (24 + 3 * fsz)
            flops += 27 * pairs
            continue
        s = case["steps"]
        nbytes += n * (96 * s + 3 * fsz)
        flops += 27 * pairs * s
        if kind == "grad":
            nbytes += n * 96 * s
            flops += 2 * 27 * pairs * s
        if kind == "melt":
            flops += 150 * n * s
    return dict(bytes=nbytes, flops=flops)


# ---- the same results in 64 bits, by plain torch ----

def _device():
    return torch.device("cuda" if torch.cuda.is_available() else "cpu")


def _near(pos, L, R):
    """Every pair i < j closer than R (minimum image), by cells of width >= R."""
    n, dev = len(pos), pos.device
    p = torch.remainder(pos, L)
    nc = min(int(L / R), 200)
    if nc < 3:
        pi, pj = [], []
        for i0 in range(0, n, 2048):
            d = p[i0:i0 + 2048, None] - p[None]
            d = d - L * torch.round(d / L)
            i, j = torch.nonzero((d * d).sum(-1) < R * R, as_tuple=True)
            i = i + i0
            pi.append(i[i < j])
            pj.append(j[i < j])
        return torch.cat(pi), torch.cat(pj)
    c3 = torch.clamp((p * (nc / L)).long(), max=nc - 1)
    cell = (c3[:, 2] * nc + c3[:, 1]) * nc + c3[:, 0]
    order = torch.argsort(cell)
    sc = cell[order]
    start = torch.searchsorted(sc, torch.arange(nc ** 3 + 1, device=dev))
    rank = torch.arange(n, device=dev) - start[sc]
    occ = int(rank.max()) + 1
    table = torch.full((nc ** 3, occ), -1, dtype=torch.long, device=dev)
    table[sc, rank] = order
    pi, pj = [], []
    step = 1 << 19
    for i0 in range(0, n, step):
        ii = torch.arange(i0, min(n, i0 + step), device=dev)
        for o in range(27):
            dz, dy, dx = o // 9 - 1, o // 3 % 3 - 1, o % 3 - 1
            q = c3[ii] + torch.tensor([dx, dy, dz], device=dev)
            q = torch.remainder(q, nc)
            cand = table[(q[:, 2] * nc + q[:, 1]) * nc + q[:, 0]]
            d2 = torch.zeros(cand.shape, dtype=torch.float64, device=dev)
            for k in range(3):
                d = p[ii, k][:, None] - p[:, k][cand.clamp(min=0)]
                d = d - L * torch.round(d / L)
                d2 += d * d
            a, b = torch.nonzero((d2 < R * R) & (cand > ii[:, None]), as_tuple=True)
            pi.append(ii[a])
            pj.append(cand[a, b])
    return torch.cat(pi), torch.cat(pj)


class _Pairs:
    """Pair lists good until some atom has moved half their margin."""

    def __init__(self, L, r_cut, margin=0.5):
        self.L, self.rc, self.margin, self.ref = L, r_cut, margin, None

    def get(self, pos):
        p = pos.detach()
        if self.ref is not None:
            d = p - self.ref
            d = d - self.L * torch.round(d / self.L)
            if float((d * d).sum(-1).max()) < (0.5 * self.margin) ** 2:
                return self.ij
        self.ref = p.clone()
        self.ij = _near(p, self.L, self.rc + self.margin)
        return self.ij


def _separations(pos, i, j, L):
    d = pos[i] - pos[j]
    return d - L * torch.round(d / L).detach()


def _lj(pos, pairs, L, r_cut, eps=1.0, sigma=1.0):
    """Forces [n, 3], energy and virial of the cut and shifted 12-6 potential;
    the cutoff is r_cut as given (it moves with sigma through the caller)."""
    i, j = pairs.get(pos)
    d = _separations(pos, i, j, L)
    inside = (d * d).sum(-1) < r_cut * r_cut
    i, j, d = i[inside], j[inside], d[inside]
    r2 = (d * d).sum(-1)
    s6 = (sigma * sigma / r2) ** 3
    w = 48.0 * eps * s6 * (s6 - 0.5)
    f = (w / r2)[:, None] * d
    force = torch.zeros_like(pos).index_add(0, i, f).index_add(0, j, -f)
    c6 = (1.0 / (r_cut / float(torch.as_tensor(sigma).detach()))) ** 6
    return force, (4.0 * eps * (s6 * (s6 - 1.0) - c6 * (c6 - 1.0))).sum(), w.sum()


def _bonded(pos, L, chain):
    """Forces of the FENE bonds and the bond angles (by differentiation)."""
    with torch.enable_grad():
        x = pos.detach().requires_grad_(True)
        c = x.view(-1, chain, 3)
        b = c[:, 1:] - c[:, :-1]
        b = b - L * torch.round(b / L).detach()
        r2 = (b * b).sum(-1)
        u = (-0.5 * FENE_K * FENE_R0 ** 2 * torch.log(1.0 - r2 / FENE_R0 ** 2)).sum()
        dots = (b[:, 1:] * b[:, :-1]).sum(-1)
        u = u + (BEND_K * (1.0 - dots / torch.sqrt(r2[:, 1:] * r2[:, :-1]))).sum()
        return -torch.autograd.grad(u, x)[0]


class _Order:
    """Cells, the storage order and the displacement rule of one system."""

    def __init__(self, L, r_cut, lists, reorder):
        self.L, self.lists, self.reorder = L, lists, reorder
        w = r_cut + (SKIN if lists else 0.0)
        self.nc = int(math.floor(L / w))
        if L / self.nc < w:
            self.nc -= 1
        self.ids = None

    def rebuild(self, x):
        """Folded positions; the slots in order of (cell, id)."""
        x = torch.where(x >= self.L, x - self.L, torch.where(x < 0, x + self.L, x))
        x = torch.where(x >= self.L, torch.zeros_like(x), x)
        if self.reorder:
            c = torch.clamp(torch.floor(x * (self.nc / self.L)).long(), 0, self.nc - 1)
            cell = (c[:, 2] * self.nc + c[:, 1]) * self.nc + c[:, 0]
            self.ids = torch.argsort(cell, stable=True)
        self.ref = x.clone()
        return x

    def after_drift(self, x):
        if self.lists:
            d = x - self.ref
            d = d - self.L * torch.round(d / self.L)
            if float((d * d).sum(-1).max()) <= (0.5 * SKIN) ** 2:
                return x
        return self.rebuild(x)


def _steps(pos, vel, L, r_cut, dt, steps, lists, reorder, chain=0):
    """x, v, f (in storage order) and the ids after leapfrog steps."""
    dev = _device()
    x, v = torch.tensor(pos, device=dev), torch.tensor(vel, device=dev)
    pairs, order = _Pairs(L, r_cut), _Order(L, r_cut, lists, reorder)

    def force(x):
        f = _lj(x, pairs, L, r_cut)[0]
        return f + _bonded(x, L, chain) if chain else f

    x = order.rebuild(x)
    f = force(x)
    for _ in range(steps):
        v = v + 0.5 * dt * f
        x = order.after_drift(x + dt * v)
        f = force(x)
        v = v + 0.5 * dt * f
    ids = order.ids if reorder else torch.arange(len(x), device=dev)
    return x[ids], v[ids], f[ids], ids.to(torch.int32)


def _state_dict(x, v, f, ids):
    out = dict(id=ids)
    for name, a in (("", x), ("v", v), ("f", f)):
        for k, axis in enumerate("xyz"):
            out[name + axis] = a[:, k].contiguous()
    return out


def _gradient(case, seed):
    pos, vel, L, kw = _single(case, seed)
    dev = _device()
    x0 = torch.tensor(pos, device=dev, requires_grad=True)
    v0 = torch.tensor(vel, device=dev, requires_grad=True)
    eps = torch.tensor(1.0, dtype=torch.float64, device=dev, requires_grad=True)
    sigma = torch.tensor(1.0, dtype=torch.float64, device=dev, requires_grad=True)
    S, n, dt, rc = case["steps"], case["n"], kw["dt"], kw["r_cut"]
    pairs = _Pairs(L, rc)
    x, v = x0, v0
    f, _, _ = _lj(x, pairs, L, rc, eps, sigma)
    ubar = 0.0
    for _ in range(S):
        v = v + 0.5 * dt * f
        x = x + dt * v
        f, u, _ = _lj(x, pairs, L, rc, eps, sigma)
        v = v + 0.5 * dt * f
        ubar = ubar + u / (S * n)
    # soft g(r): a Gaussian per ordered pair, lowered by its value at 3 widths
    w = GRAD_RMAX / GRAD_BINS
    i, j = _near(x.detach(), L, GRAD_RMAX + 3.0 * w)
    r = torch.sqrt((_separations(x, i, j, L) ** 2).sum(-1))
    g = []
    for b in range(GRAD_BINS):
        rb = (b + 0.5) * GRAD_RMAX / GRAD_BINS
        t = r[(r.detach() - rb).abs() < 3.0 * w] - rb
        k = (torch.exp(-0.5 * (t / w) ** 2) - math.exp(-4.5)) / (w * math.sqrt(2.0 * math.pi))
        g.append(2.0 * k.sum() / (n * (n / L ** 3) * 4.0 * math.pi * rb * rb))
    g = torch.stack(g)
    loss = ubar + ((g - _target(seed).to(dev)) ** 2).sum()
    loss.backward()
    return dict(ubar=ubar.detach(), g=g.detach(), x0=x0.grad, v0=v0.grad, eps=eps.grad,
                sigma=sigma.grad)


def exact(case, seed):
    kind = case["kind"]
    if kind == "grad":
        return _gradient(case, seed)
    if kind == "batch":
        parts = [_steps(s["pos"], s["vel"], s["L"], s["r_cut"], s["dt"], case["steps"], True, True)
                 for s in _replicas(case, seed)]
        return _state_dict(*(torch.cat(p) for p in zip(*parts)))
    pos, vel, L, kw = _single(case, seed)
    if kind == "frame":
        x = torch.tensor(pos, device=_device())
        f, u, w = _lj(x, _Pairs(L, kw["r_cut"]), L, kw["r_cut"])
        return dict(fx=f[:, 0].contiguous(), fy=f[:, 1].contiguous(), fz=f[:, 2].contiguous(),
                    U=float(u), W=float(w), K=0.5 * float((vel * vel).sum()))
    return _state_dict(*_steps(pos, vel, L, kw["r_cut"], kw["dt"], case["steps"],
                               kind != "cells", kind != "cells",
                               case.get("chain", 0)))
