"""Timed cases of the framework: what its users have it do, over the sizes they use.

The inputs are the repository's own synthetic workloads, made on the GPU from a seed: the
dense Lennard-Jones liquid (fcc at 0.8442, T = 1.44, cutoff 2.5, skin 0.3, one or two
types, atoms taken out at random for sizes that are no multiple of anything), the same
liquid with unit charges (SPME, alpha 1.2, order 4, spacing <= 0.7), and the jittered
simple-cubic SPH fluid (h = 1.3, skin 0.4).

Kinds of a case:
  md       LJSim.step: one window of velocity-Verlet steps with its re-sort and list build
  charged  ChargedLJSim.step: the same with Ewald real space and SPME
  sph      SPHSim.step: density, pressure acceleration, integration, re-sort, list build
  resort   ops.bin + ops.build_neighbors for a program with its own integrator
  csr      a compressed list (from the cells, or from the tiled list) and forces over it
  match    one force-matching training step: forces, loss, gradients (x, eps, sigma)
  traj     gradients through a checkpointed trajectory (x0, v0, eps, sigma)
"""
import math

import torch
import torch.utils.checkpoint

from paper_2109_09056_amd import autograd, md, ops, sph, trajectory
from paper_2109_09056_amd.electrostatics import ChargedLJSim

DENSITY, TEMPERATURE, JITTER = 0.8442, 1.44, 0.05
RC, SKIN, DT, WINDOW = 2.5, 0.3, 0.005, 20
ALPHA, ORDER = 1.2, 4
SPH_H, SPH_C0, SPH_RHO0, SPH_SKIN, SPH_DT, SPH_WINDOW = 1.3, 10.0, 1.0, 0.4, 0.01, 10
PRECISION = {"fp64": ops.FP64, "mixed": ops.MIXED}
KIND = {"full": ops.FULL, "half": ops.HALF}


def _lj(kind, cells, drop=0, types=1, precision="mixed", **more):
    return dict(kind=kind, nx=cells[0], ny=cells[1], nz=cells[2], drop=drop, types=types,
                precision=precision, **more)


def listed():
    cube = lambda c: (c, c, c)  # noqa: E731
    return [
        # the smallest system: launch latency and the host's share of a step
        _lj("md", cube(4), precision="fp64", list="full") | {"name": "md-256-fp64"},
        # the 32,000-atom liquid, both list kinds
        _lj("md", cube(20), precision="mixed", list="full") | {"name": "md-32000-mixed"},
        _lj("md", cube(20), precision="fp64", list="half") | {"name": "md-32000-half-fp64"},
        # an ordinary production size: ragged box, odd atom count, two types
        _lj("md", (31, 27, 33), drop=37, types=2, precision="fp64", list="full")
        | {"name": "md-110447-2types-fp64"},
        # the benchmark liquid
        _lj("md", cube(50), precision="mixed", list="full") | {"name": "md-500000-mixed"},
        # sorting and lists for a caller's own integrator
        _lj("resort", cube(50), list="full") | {"name": "resort-500000"},
        # compressed lists, built straight from the cells, four lanes per atom
        _lj("csr", cube(32), precision="mixed", source="cells", team=4)
        | {"name": "csr-131072"},
        # force matching: forward and backward of one training step
        _lj("match", cube(20), types=2, precision="mixed") | {"name": "match-32000"},
        # backpropagation through 20 steps with checkpoints every 5
        _lj("traj", cube(40), types=2, precision="fp64") | {"name": "traj-256000"},
        # the SPH fluid
        dict(name="sph-512000", kind="sph", nx=80, ny=80, nz=80, drop=0),
        # charged liquids: 64^3 and 128^3 grids
        _lj("charged", cube(20), precision="mixed") | {"name": "charged-32000"},
        _lj("charged", cube(50), precision="mixed") | {"name": "charged-500000"},
    ]


# largest particle number of a drawn case of each kind (the listed one's)
LARGEST = {"md": 500000, "resort": 500000, "csr": 500000, "match": 256000, "traj": 256000,
           "sph": 512000, "charged": 500000}


def draw(rng):
    kind = rng.choice(["md", "md", "md", "resort", "csr", "match", "traj", "sph", "charged",
                       "charged"])
    per = 1 if kind == "sph" else 4
    low = 8 if kind == "sph" else 4
    n = math.exp(rng.uniform(math.log(per * low ** 3 * 1.5), math.log(LARGEST[kind])))
    edge = (n / per) ** (1.0 / 3.0)
    cells = [max(low, round(edge * rng.uniform(0.85, 1.18))) for _ in range(3)]
    while per * cells[0] * cells[1] * cells[2] > LARGEST[kind]:
        cells[cells.index(max(cells))] -= 1
    drop = rng.randrange(0, min(64, per * cells[0] * cells[1] * cells[2] // 16))
    if kind == "sph":
        return dict(kind=kind, nx=cells[0], ny=cells[1], nz=cells[2], drop=drop)
    if kind == "charged":
        drop -= drop % 2  # neutral
    case = _lj(kind, cells, drop=drop, precision=rng.choice(["fp64", "mixed"]))
    if kind in ("md", "match", "traj"):
        case["types"] = rng.choice([1, 2])
    if kind in ("md", "resort"):
        case["list"] = rng.choice(["full", "full", "half"])
    if kind == "csr":
        case["source"] = rng.choice(["cells", "tiled"])
        case["team"] = rng.choice([1, 2, 4, 8])
    return case


# ------------------------------------------------------------------ inputs --


class _Draws:
    """Seeded draws on the GPU."""

    def __init__(self, seed):
        self.dev = torch.device("cuda")
        self.g = torch.Generator(device=self.dev)
        self.g.manual_seed(20210919 + 7919 * int(seed))

    def uniform(self, lo, hi, shape):
        return lo + (hi - lo) * torch.rand(shape, generator=self.g, device=self.dev,
                                           dtype=torch.float64)

    def normal(self, shape):
        return torch.randn(shape, generator=self.g, device=self.dev, dtype=torch.float64)

    def perm(self, n):
        return torch.randperm(n, generator=self.g, device=self.dev)


def _wrap(x, L):
    x = torch.where(x < 0.0, x + L, x)
    x = torch.where(x >= L, x - L, x)
    return torch.where(x >= L, x - L, x)


def _lattice(case, basis, a, d, jitter):
    """Jittered lattice with `drop` atoms taken out, in lattice order, and its box."""
    n3 = [torch.arange(case[k], device=d.dev, dtype=torch.float64) for k in ("nx", "ny", "nz")]
    o = torch.stack(torch.meshgrid(*n3, indexing="ij"), dim=-1).reshape(-1, 1, 3)
    x = ((o + torch.tensor(basis, device=d.dev, dtype=torch.float64)) * a).reshape(-1, 3)
    L = torch.tensor([case["nx"] * a, case["ny"] * a, case["nz"] * a], device=d.dev,
                     dtype=torch.float64)
    x = _wrap(x + d.uniform(-jitter, jitter, x.shape), L)
    if case["drop"]:
        keep = torch.ones(x.shape[0], dtype=torch.bool, device=d.dev)
        keep[d.perm(x.shape[0])[:case["drop"]]] = False
        x = x[keep]
    return x.contiguous(), L


def _system(case, seed):
    """x, v, types, eps, sigma, charges, L (list of floats) of a liquid, and its draws."""
    d = _Draws(seed)
    fcc = [[0.0, 0.0, 0.0], [0.5, 0.5, 0.0], [0.5, 0.0, 0.5], [0.0, 0.5, 0.5]]
    x, L = _lattice(case, fcc, (4.0 / DENSITY) ** (1.0 / 3.0), d, JITTER)
    n = x.shape[0]
    v = d.normal(x.shape) * math.sqrt(TEMPERATURE)
    v = v - v.mean(dim=0)
    v = v * torch.sqrt(TEMPERATURE * (3 * n - 3) / (v * v).sum())
    types = torch.zeros(n, dtype=torch.int32, device=d.dev)
    eps = torch.ones(1, dtype=torch.float64, device=d.dev)
    sigma = torch.ones(1, dtype=torch.float64, device=d.dev)
    if case["types"] == 2:
        types[d.perm(n)[:n // 2]] = 1
        eps, sigma = d.uniform(0.8, 1.2, (3,)), d.uniform(0.9, 1.1, (3,))
    q = -torch.ones(n, dtype=torch.float64, device=d.dev)
    q[d.perm(n)[:n // 2]] = 1.0
    return dict(x=x, v=v, types=types, eps=eps, sigma=sigma, q=q, L=L.tolist(), n=n, draws=d)


def _fluid(case, seed):
    d = _Draws(seed)
    x, L = _lattice(case, [[0.5, 0.5, 0.5]], 1.0, d, 0.1)
    v = 0.2 * d.normal(x.shape)
    return dict(x=x, v=v - v.mean(dim=0), L=L.tolist(), n=x.shape[0])


def _charge_grid(L):
    out = []
    for edge in L:
        k = 8
        while edge / k > 0.7:
            k *= 2
        out.append(k)
    return tuple(out)


def _drifted(case, seed):
    """A liquid in the sorted order of its last re-sort, after the moves of one window:
    what a program hands to its next re-sort (x, v, types, ids)."""
    s = _system(case, seed)
    order = _sorted_order(s["x"], s["L"], RC + SKIN)
    L = torch.tensor(s["L"], device=s["x"].device, dtype=torch.float64)
    x = _wrap((s["x"] + 0.5 * WINDOW * DT * s["v"])[order], L)
    return dict(s, x=x.contiguous(), v=s["v"][order].contiguous(),
                types=s["types"][order].contiguous(), ids=order.contiguous())


def _matching(case, seed):
    """Positions, parameters and the target forces of a force-matching step (sorted order)."""
    s = _system(case, seed)
    order = _sorted_order(s["x"], s["L"], RC + SKIN)
    target = 10.0 * s["draws"].normal(s["x"].shape)
    return dict(s, order=order, target=target)


def _window(case, seed):
    """A trajectory's start, parameters and observed end positions."""
    s = _system(case, seed)
    L = torch.tensor(s["L"], device=s["x"].device, dtype=torch.float64)
    end = s["x"] + WINDOW * DT * 0.5 * s["v"] + 0.02 * s["draws"].normal(s["x"].shape)
    return dict(s, xref=_wrap(end, L).contiguous())


def prepare(case, seed):
    kind = case["kind"]
    if kind == "sph":
        s = _fluid(case, seed)
        sim = sph.SPHSim(s["L"], SPH_H, c0=SPH_C0, rho0=SPH_RHO0, skin=SPH_SKIN, dt=SPH_DT,
                         rebuild_every=SPH_WINDOW)
        return dict(kind=kind, sim=sim.load(s["x"], s["v"]))
    prec = PRECISION[case["precision"]]
    if kind == "md":
        s = _system(case, seed)
        sim = md.LJSim(s["L"], rc=RC, skin=SKIN, eps=s["eps"], sigma=s["sigma"], precision=prec,
                       kind=KIND[case["list"]], dt=DT, rebuild_every=WINDOW)
        return dict(kind=kind, sim=sim.load(s["x"], s["v"], s["types"]))
    if kind == "charged":
        s = _system(case, seed)
        sim = ChargedLJSim(s["L"], alpha=ALPHA, order=ORDER, grid=_charge_grid(s["L"]), rc=RC,
                           skin=SKIN, precision=prec, dt=DT, rebuild_every=WINDOW)
        return dict(kind=kind, sim=sim.load(s["x"], s["v"], s["q"]))
    if kind == "resort":
        s = _drifted(case, seed)
        n, dev = s["n"], s["x"].device
        nc = ops.grid(s["L"], RC + SKIN)
        cells = nc[0] * nc[1] * nc[2]
        maxn = md.initial_maxn(n, s["L"], RC + SKIN, ops.FULL)  # half rows reach full length
        i32 = dict(dtype=torch.int32, device=dev)
        return dict(
            kind=kind, s=s, maxn=maxn, list=KIND[case["list"]],
            out=(torch.empty_like(s["x"]), torch.empty_like(s["v"]), torch.empty(n, **i32),
                 torch.empty(n, dtype=torch.int64, device=dev)),
            cell_start=torch.empty(cells + 1, **i32),
            ws=torch.empty(max(ops.workspace_bytes(ops.OP_BIN, n, ncells=cells), 8),
                           dtype=torch.uint8, device=dev),
            nbr=torch.zeros(ops.list_shape(n, maxn), **i32), nnbr=torch.empty(n, **i32),
            max_count=torch.empty(1, **i32))
    if kind == "csr":
        s = _system(case, seed)
        n, dev, rl = s["n"], s["x"].device, RC + SKIN
        x, _, types, _, cs = ops.bin(s["L"], rl, s["x"], None, s["types"])
        cap = int((4.0 / 3.0 * math.pi * rl ** 3 * DENSITY * 1.1 + 8) * n) + 64
        st = dict(kind=kind, s=s, x=x, types=types, cell_start=cs, precision=prec,
                  source=case["source"], team=case["team"], cap=cap,
                  offsets=torch.empty(n + 1, dtype=torch.int64, device=dev),
                  csr=torch.zeros(cap, dtype=torch.int32, device=dev))
        if case["source"] == "tiled":
            nl = md.NeighborList(s["L"], rl).build(x, cs)
            st.update(nbr=nl.nbr, nnbr=nl.nnbr, maxn=nl.maxn)
        return st
    if kind == "match":
        s = _matching(case, seed)
        fc = autograd.ForceContext(s["L"], s["x"], s["types"], rc=RC, skin=SKIN, precision=prec)
        return dict(kind=kind, fc=fc, x=fc.x.clone().requires_grad_(True),
                    eps=s["eps"].requires_grad_(True), sigma=s["sigma"].requires_grad_(True),
                    target=s["target"])
    s = _window(case, seed)
    return dict(kind=kind, s=s, precision=prec)


# --------------------------------------------------------------------- run --


def run(state):
    kind = state["kind"]
    if kind == "sph":
        sim = state["sim"].step(SPH_WINDOW, energy=True)
        return dict(x=sim.x, v=sim.v, acc=sim.acc, rho=sim.rho, u=sim.u, ke=sim.ke, ids=sim.ids)
    if kind in ("md", "charged"):
        sim = state["sim"].step(WINDOW)
        out = dict(x=sim.x, v=sim.v, F=sim.F, ids=sim.ids, e=sim.e_atom, ev=sim.ev)
        if kind == "charged":
            out.update(ec=sim.ec)
        return out
    if kind == "resort":
        s, rl = state["s"], RC + SKIN
        x, v, types, ids, cs = ops.bin(s["L"], rl, s["x"], s["v"], s["types"], s["ids"],
                                       out=state["out"], cell_start=state["cell_start"],
                                       ws=state["ws"])
        nbr, nnbr, most = ops.build_neighbors(s["L"], rl, state["list"], x, cs, state["maxn"],
                                              state["nbr"], state["nnbr"], state["max_count"])
        return dict(x=x, v=v, types=types, ids=ids, cell_start=cs, nbr=nbr, nnbr=nnbr,
                    max_count=most)
    if kind == "csr":
        s = state["s"]
        if state["source"] == "cells":
            off, csr = ops.build_neighbors_csr(s["L"], RC + SKIN, ops.FULL, state["x"],
                                               state["cell_start"], cap=state["cap"],
                                               offsets=state["offsets"], csr=state["csr"])
        else:
            off, csr = ops.list_to_csr(state["nbr"], state["nnbr"], state["maxn"],
                                       cap=state["cap"], offsets=state["offsets"],
                                       csr=state["csr"])
        F, e, ev = ops.compute_forces_csr(s["L"], state["precision"], RC, s["eps"], s["sigma"],
                                          state["x"], state["types"], off, csr,
                                          team=state["team"])
        return dict(offsets=off, csr=csr, F=F, e=e, ev=ev)
    if kind == "match":
        F = autograd.lj_forces(state["x"], state["eps"], state["sigma"], state["fc"])
        loss = ((F - state["target"]) ** 2).sum()
        gx, ge, gs = torch.autograd.grad(loss, (state["x"], state["eps"], state["sigma"]))
        return dict(F=F, loss=loss, gx=gx, geps=ge, gsigma=gs)
    s = state["s"]
    r = trajectory.backprop_trajectory(s["L"], s["x"], s["v"], s["types"], s["eps"], s["sigma"],
                                       s["xref"], steps=WINDOW, checkpoint_every=5, rc=RC,
                                       skin=SKIN, dt=DT, precision=state["precision"])
    return dict(loss=r.loss, gx0=r.gx0, gv0=r.gv0, geps=r.geps, gsigma=r.gsigma, xT=r.xT)


# -------------------------------------------------------------------- work --


def work(case):
    """Bytes and operations a pass cannot do without: per step each list entry's index, the
    particle's own arrays in and out, and ~25 operations per entry inside the list; per
    re-sort the arrays moved and the list written; per grid pass the grid in and out."""
    cells = case["nx"] * case["ny"] * case["nz"]
    if case["kind"] == "sph":
        n, rl = cells - case["drop"], 2.0 * SPH_H + SPH_SKIN
        m = 4.0 / 3.0 * math.pi * rl ** 3
        step = n * (2 * 4 * m + 36 + 60 + 96)
        return {"bytes": SPH_WINDOW * step + n * (4 * m + 160),
                "flops": SPH_WINDOW * n * m * 60 + n * m * 10}
    n = 4 * cells - case["drop"]
    m = 4.0 / 3.0 * math.pi * (RC + SKIN) ** 3 * DENSITY
    kind = case["kind"]
    rebuild = n * (4 * m * (0.5 if case.get("list") == "half" else 1.0) + 28 + 140)
    if kind == "resort":
        return {"bytes": rebuild, "flops": n * m * 10}
    if kind == "md":
        rows = 0.5 if case["list"] == "half" else 1.0
        return {"bytes": WINDOW * n * (4 * m * rows + 132) + rebuild,
                "flops": WINDOW * n * m * rows * 25 + n * m * 10}
    if kind == "charged":
        K = _charge_grid([case[k] * (4.0 / DENSITY) ** (1.0 / 3.0) for k in ("nx", "ny", "nz")])
        grid = K[0] * K[1] * K[2]
        step = n * (2 * 4 * m + 132 + 64 + 112) + grid * (5 * 8 + 8 * 8)
        fft = 2 * 2.5 * grid * math.log2(grid)
        return {"bytes": WINDOW * step + rebuild,
                "flops": WINDOW * (n * m * 75 + n * 4 ** 3 * 8 + fft) + n * m * 10}
    if kind == "csr":
        return {"bytes": n * (2 * 4 * m + 24 + 8 + 60), "flops": n * m * 35}
    if kind == "match":
        return {"bytes": n * (2 * 4 * m + 24 + 24 + 24 + 24 + 24 + 12), "flops": n * m * 85}
    # forward, recomputation and reverse
    return {"bytes": WINDOW * n * (2 * (4 * m + 132) + 4 * m + 172) + rebuild,
            "flops": WINDOW * n * m * (2 * 25 + 60) + n * m * 10}


# ------------------------------------------------------- 64-bit references --


def _cells(x, L, rlist):
    """Cell of every particle and the grid, by the binning rule (edges >= rlist)."""
    nc, idx = [], []
    for k in range(3):
        m = max(int(math.floor(L[k] / rlist)), 1)
        while m > 1 and L[k] / m < rlist * (1.0 + 1e-10):
            m -= 1
        nc.append(m)
        idx.append(torch.floor(x[:, k] / (L[k] / m)).long().clamp(0, m - 1))
    return nc, idx


def _sorted_order(x, L, rlist):
    """Particles by cell (x fastest), then by id."""
    nc, (cx, cy, cz) = _cells(x, L, rlist)
    return torch.sort((cz * nc[1] + cy) * nc[0] + cx, stable=True).indices


def _image(d, Lt):
    return d - Lt * torch.round(d / Lt)


def _pairs(x, L, rlist):
    """All unordered pairs (i, j) closer than rlist."""
    n, dev = x.shape[0], x.device
    Lt = torch.tensor(L, device=dev, dtype=torch.float64)
    nc, idx = _cells(x, L, rlist)
    cell = (idx[2] * nc[1] + idx[1]) * nc[0] + idx[0]
    ncell = nc[0] * nc[1] * nc[2]
    order = torch.sort(cell, stable=True).indices
    count = torch.bincount(cell, minlength=ncell)
    start = torch.cumsum(count, 0) - count
    width = int(count.max())
    slot = torch.arange(n, device=dev) - start[cell[order]]
    table = torch.full((ncell, width), -1, dtype=torch.int64, device=dev)
    table[cell[order], slot] = order
    # distinct neighbour cells per dimension (fewer than three cells: each once)
    off = [[-1, 0, 1] if m >= 3 else list(range(m)) for m in nc]
    out_i, out_j = [], []
    chunk = max(1, 40_000_000 // max(width, 1))
    for oz in off[2]:
        for oy in off[1]:
            for ox in off[0]:
                other = [(idx[k] + o) % nc[k] if nc[k] >= 3 else torch.full_like(idx[k], o)
                         for k, o in enumerate((ox, oy, oz))]
                cand = (other[2] * nc[1] + other[1]) * nc[0] + other[0]
                for a in range(0, n, chunk):
                    b = min(n, a + chunk)
                    j = table[cand[a:b]]
                    i = torch.arange(a, b, device=dev).unsqueeze(1).expand_as(j)
                    keep = j > i
                    i, j = i[keep], j[keep]
                    d = _image(x[i] - x[j], Lt)
                    near = (d * d).sum(1) < rlist * rlist
                    out_i.append(i[near])
                    out_j.append(j[near])
    return torch.cat(out_i), torch.cat(out_j)


def _scatter_pairs(n, i, j, f):
    out = torch.zeros((n, f.shape[1]), dtype=torch.float64, device=f.device)
    return out.index_add(0, i, f).index_add(0, j, -f)


def _packed(t, i, j):
    """Packed upper-triangle index of the pairs' types (one or two types)."""
    return (t[i] + t[j]).long()


def _lj_forces(x, Lt, pairs, types, eps, sigma):
    """F, per-atom energy and [E, Wxx, Wyy, Wzz, Wxy, Wxz, Wyz] over the listed pairs."""
    i, j = pairs
    with torch.no_grad():
        d = _image(x[i] - x[j], Lt)
        near = (d * d).sum(1) < RC * RC
        i, j = i[near], j[near]
        shift = Lt * torch.round((x[i] - x[j]) / Lt)
    d = x[i] - x[j] - shift
    r2 = (d * d).sum(1)
    p = _packed(types, i, j)
    e4, sr6 = 4.0 * eps[p], (sigma[p] * sigma[p] / r2) ** 3
    s = 6.0 * e4 * (2.0 * sr6 * sr6 - sr6) / r2
    f = s.unsqueeze(1) * d
    F = _scatter_pairs(x.shape[0], i, j, f)
    with torch.no_grad():
        u = e4 * (sr6 * sr6 - sr6)
        e = torch.zeros(x.shape[0], dtype=torch.float64, device=x.device)
        e = e.index_add(0, i, 0.5 * u).index_add(0, j, 0.5 * u)
        w = [(d[:, a] * f[:, b]).sum() for a, b in ((0, 0), (1, 1), (2, 2), (0, 1), (0, 2), (1, 2))]
        ev = torch.stack([u.sum()] + w)
    return F, e, ev


def _spline(u, K):
    """Order-4 B-spline weights and derivatives (4, n) at the points floor(u) - j, mod K."""
    w = u - torch.floor(u)
    k = torch.stack([(torch.floor(u).long() - a) % K for a in range(4)])
    m2 = [w, 1.0 - w, torch.zeros_like(w), torch.zeros_like(w)]

    def up(m, order):
        return [((w + a) * m[a] + (order - w - a) * (m[a - 1] if a else 0.0)) / (order - 1)
                for a in range(4)]

    m3 = up(m2, 3)
    m4 = up(m3, 4)
    dm = [m3[a] - (m3[a - 1] if a else 0.0) for a in range(4)]
    return k, torch.stack(m4), torch.stack(dm)


def _coulomb(x, q, L, pairs):
    """Ewald forces, E_dir and E_rec + E_self (SPME of order 4 on the case's grid)."""
    dev, n = x.device, x.shape[0]
    Lt = torch.tensor(L, device=dev, dtype=torch.float64)
    i, j = pairs
    d = _image(x[i] - x[j], Lt)
    r2 = (d * d).sum(1)
    near = r2 < RC * RC
    i, j, d, r = i[near], j[near], d[near], torch.sqrt(r2[near])
    qq, er = q[i] * q[j], torch.special.erfc(ALPHA * r) / r
    gauss = 2.0 * ALPHA / math.sqrt(math.pi) * torch.exp(-(ALPHA * r) ** 2)
    F = _scatter_pairs(n, i, j, (qq * (er + gauss) / (r * r)).unsqueeze(1) * d)
    e_dir = (qq * er).sum()
    K = _charge_grid(L)
    sp = [_spline(x[:, a] * (K[a] / L[a]), K[a]) for a in range(3)]
    grid = torch.zeros(K[2] * K[1] * K[0], dtype=torch.float64, device=dev)
    for c in range(4):
        for b in range(4):
            for a in range(4):
                at = (sp[2][0][c] * K[1] + sp[1][0][b]) * K[0] + sp[0][0][a]
                grid.index_add_(0, at, q * sp[2][1][c] * sp[1][1][b] * sp[0][1][a])
    fq = torch.fft.fftn(grid.view(K[2], K[1], K[0]))
    m, bm = [], []
    for a in range(3):
        k = torch.arange(K[a], device=dev, dtype=torch.float64)
        m.append(torch.where(k <= K[a] // 2, k, k - K[a]) / L[a])
        arg = 2.0 * math.pi * k / K[a]
        den = (1.0 / 6.0 + 4.0 / 6.0 * torch.exp(1j * arg) + 1.0 / 6.0 * torch.exp(2j * arg)).abs()
        bm.append(1.0 / (den * den))
    msq = m[2].view(-1, 1, 1) ** 2 + m[1].view(1, -1, 1) ** 2 + m[0].view(1, 1, -1) ** 2
    msq[0, 0, 0] = 1.0
    V = L[0] * L[1] * L[2]
    G = torch.exp(-math.pi ** 2 * msq / ALPHA ** 2) / (math.pi * V * msq)
    G = G * bm[2].view(-1, 1, 1) * bm[1].view(1, -1, 1) * bm[0].view(1, 1, -1)
    G[0, 0, 0] = 0.0
    e_rec = 0.5 * (G * fq.abs() ** 2).sum()
    phi = (torch.fft.ifftn(G * fq) * (K[0] * K[1] * K[2])).real.reshape(-1)
    g = [torch.zeros(n, dtype=torch.float64, device=dev) for _ in range(3)]
    for c in range(4):
        for b in range(4):
            for a in range(4):
                at = (sp[2][0][c] * K[1] + sp[1][0][b]) * K[0] + sp[0][0][a]
                ph = phi[at]
                g[0] += ph * sp[0][2][a] * sp[1][1][b] * sp[2][1][c]
                g[1] += ph * sp[0][1][a] * sp[1][2][b] * sp[2][1][c]
                g[2] += ph * sp[0][1][a] * sp[1][1][b] * sp[2][2][c]
    F = F - torch.stack([q * g[a] * (K[a] / L[a]) for a in range(3)], dim=1)
    e_self = -ALPHA / math.sqrt(math.pi) * (q * q).sum()
    return F, torch.stack([e_dir, e_rec + e_self])


def _exact_md(case, seed):
    s = _system(case, seed)
    L, Lt = s["L"], torch.tensor(s["L"], device=s["x"].device, dtype=torch.float64)
    x, v, q = s["x"], s["v"], s["q"]
    charged = case["kind"] == "charged"
    pairs = _pairs(x, L, RC + SKIN)
    order = None

    def forces():
        F, e, ev = _lj_forces(x, Lt, pairs, s["types"], s["eps"], s["sigma"])
        ec = None
        if charged:
            Fc, ec = _coulomb(x, q, L, pairs)
            F = F + Fc
        return F, e, ev, ec

    F, e, ev, ec = forces()
    for k in range(1, WINDOW + 1):
        v = v + 0.5 * DT * F
        x = _wrap(x + DT * v, Lt)
        if k % WINDOW == 0:
            pairs = _pairs(x, L, RC + SKIN)
            order = _sorted_order(x, L, RC + SKIN)
        F, e, ev, ec = forces()
        v = v + 0.5 * DT * F
    ke = 0.5 * (v * v).sum()
    out = dict(x=x[order], v=v[order], F=F[order], ids=None, e=e[order],
               ev=torch.cat([ev, ke.reshape(1)]))
    if charged:
        out.update(ec=ec)
    return out


def _exact_sph(case, seed):
    s = _fluid(case, seed)
    L, Lt = s["L"], torch.tensor(s["L"], device=s["x"].device, dtype=torch.float64)
    x, v, n, h = s["x"], s["v"], s["n"], SPH_H
    rlist = 2.0 * h + SPH_SKIN
    pairs, order = _pairs(x, L, rlist), None

    def accel():
        i, j = pairs
        d = _image(x[i] - x[j], Lt)
        r = torch.sqrt((d * d).sum(1))
        near = r < 2.0 * h
        i, j, d, r = i[near], j[near], d[near], r[near]
        q = r / h
        w = torch.where(q < 1.0, 1.0 - 1.5 * q ** 2 + 0.75 * q ** 3, 0.25 * (2.0 - q) ** 3)
        g = torch.where(q < 1.0, -3.0 + 2.25 * q, -0.75 * (2.0 - q) ** 2 / q)
        rho = torch.ones(n, dtype=torch.float64, device=x.device).index_add(0, i, w)
        rho = rho.index_add(0, j, w) / (math.pi * h ** 3)
        P = SPH_C0 ** 2 * (rho - SPH_RHO0) / rho ** 2
        f = (-(P[i] + P[j]) * g / (math.pi * h ** 5)).unsqueeze(1) * d
        return _scatter_pairs(n, i, j, f), rho

    a, rho = accel()
    for k in range(1, SPH_WINDOW + 1):
        v = v + 0.5 * SPH_DT * a
        x = _wrap(x + SPH_DT * v, Lt)
        if k % SPH_WINDOW == 0:
            pairs, order = _pairs(x, L, rlist), _sorted_order(x, L, rlist)
        a, rho = accel()
        v = v + 0.5 * SPH_DT * a
    u = (SPH_C0 ** 2 * (torch.log(rho / SPH_RHO0) + SPH_RHO0 / rho - 1.0)).sum()
    return dict(x=x[order], v=v[order], acc=a[order], rho=rho[order], u=u.reshape(1),
                ke=0.5 * (v * v).sum().reshape(1), ids=None)


def _exact_traj(case, seed):
    s = _window(case, seed)
    L, Lt = s["L"], torch.tensor(s["L"], device=s["x"].device, dtype=torch.float64)
    leaf = [t.clone().requires_grad_(True) for t in (s["x"], s["v"], s["eps"], s["sigma"])]
    x, v, eps, sigma = leaf
    pairs = _pairs(s["x"], L, RC + SKIN)

    def step(x, v, F, eps, sigma):
        v = v + 0.5 * DT * F
        x = _wrap(x + DT * v, Lt)
        F = _lj_forces(x, Lt, pairs, s["types"], eps, sigma)[0]
        return x, v + 0.5 * DT * F, F

    again = torch.utils.checkpoint.checkpoint
    F = again(lambda *a: _lj_forces(a[0], Lt, pairs, s["types"], a[1], a[2])[0], x, eps, sigma,
              use_reentrant=False)
    for _ in range(WINDOW):
        x, v, F = again(step, x, v, F, eps, sigma, use_reentrant=False)
    d = x - s["xref"]
    d = d - (Lt * torch.round(d / Lt)).detach()
    loss = 0.5 * (d * d).sum()
    gx, gv, ge, gs = torch.autograd.grad(loss, leaf)
    return dict(loss=loss.reshape(1), gx0=gx, gv0=gv, geps=ge, gsigma=gs, xT=x)


def exact(case, seed):
    kind = case["kind"]
    if kind in ("md", "charged"):
        return _exact_md(case, seed)
    if kind == "sph":
        return _exact_sph(case, seed)
    if kind == "traj":
        return _exact_traj(case, seed)
    if kind == "resort":
        s = _drifted(case, seed)
        by_id = torch.argsort(s["ids"])
        order = by_id[_sorted_order(s["x"][by_id], s["L"], RC + SKIN)]
        return dict(x=s["x"][order], v=s["v"][order], types=None, ids=None, cell_start=None,
                    nbr=None, nnbr=None, max_count=None)
    s = _system(case, seed) if kind == "csr" else _matching(case, seed)
    Lt = torch.tensor(s["L"], device=s["x"].device, dtype=torch.float64)
    order = _sorted_order(s["x"], s["L"], RC + SKIN)
    x, types = s["x"][order], s["types"][order]
    pairs = _pairs(x, s["L"], RC + SKIN)
    if kind == "csr":
        F, e, ev = _lj_forces(x, Lt, pairs, types, s["eps"], s["sigma"])
        return dict(offsets=None, csr=None, F=F, e=e, ev=ev)
    leaf = [t.clone().requires_grad_(True) for t in (x, s["eps"], s["sigma"])]
    F = _lj_forces(leaf[0], Lt, pairs, types, leaf[1], leaf[2])[0]
    loss = ((F - s["target"]) ** 2).sum()
    gx, ge, gs = torch.autograd.grad(loss, leaf)
    return dict(F=F, loss=loss, gx=gx, geps=ge, gsigma=gs)
