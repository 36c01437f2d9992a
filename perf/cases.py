"""Workloads that the performance of this package is followed on.

Every case is one call sequence of a user's program through
``paper_1210_3450_amd.binding``: load a state, evaluate or step it, and take the
results out.  Sizes, densities and parameters are those of ``bench.py``, the tests
and ``inputs.py`` (FCC boxes at density 0.5 and cutoff 2.5 from 4000 to 32 million
particles, the cavitation liquid at density 0.7 and cutoff 3.0, the uneven 256-box
ensemble), with ragged particle counts and non-cubic boxes between them.

States are FCC blocks with some sites removed and every particle displaced by a
uniform jitter, as disordered as a fluid a few hundred steps after the lattice, with
Maxwell-Boltzmann velocities.  They are drawn on the GPU from the seed alone.

FP64 cases return what the library hands out, in FP64.  The FP32-mixed path computes
its forces in FP32 (a choice the caller makes at creation), so its velocities, forces
and energies are returned as the FP32 values a trajectory file of such a run holds;
its positions, integrated in FP64, are returned in FP64.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_1210_3450_amd import binding as B
from paper_1210_3450_amd import inputs

FP64, MIXED = B.MD_PREC_FP64, B.MD_PREC_FP32_MIXED
DT = 0.005
JITTER = 0.1      # of the nearest-neighbour distance, uniform per coordinate
EXACT_MAX = 3_000_000  # particles; a 64-bit reference of more takes minutes

_BASE = dict(kind="nve", cx=10, cy=10, cz=10, holes=0, rho=0.5, T=1.0, rc=2.5, skin=0.3, precision=FP64,
             policy=B.MD_REBUILD_DUTC, flags=0, calls=1, steps=20, energy_every=0)


def _case(name=None, **kw):
    c = dict(_BASE)
    if name is not None:
        c["name"] = name
    c.update(kw)
    return c


def listed():
    return [
        # the small box of the tests and the benchmark: 4000 particles, 100 steps in captured
        # graphs with the energy sampled every 10; launches and latency are what it costs
        _case("nve_fp64_4k", steps=100, energy_every=10, flags=B.MD_F_GRAPH),
        # the smallest calls: an odd-sized dense box advanced 5 steps per call, as a program
        # that looks at the state in between does; no graphs
        _case("nve_mixed_10k_calls", cx=14, cy=14, cz=13, holes=185, rho=0.7, precision=MIXED, calls=5, steps=5),
        # the million-particle box in both precisions, graphs on
        _case("nve_fp64_1m", cx=64, cy=64, cz=64, steps=50, flags=B.MD_F_GRAPH),
        _case("nve_mixed_1m", cx=64, cy=64, cz=64, steps=50, precision=MIXED, flags=B.MD_F_GRAPH),
        # a ragged, elongated box of ordinary size with the displacement rebuild rule
        _case("nve_mixed_250k_slab", cx=61, cy=33, cz=31, holes=1237, rho=0.6, precision=MIXED,
              policy=B.MD_REBUILD_DISPLACEMENT, steps=50),
        # the headline box in both precisions
        _case("nve_fp64_32m", cx=200, cy=200, cz=200, steps=20),
        _case("nve_mixed_32m", cx=200, cy=200, cz=200, steps=20, precision=MIXED),
        # equilibration of the cavitation liquid: Nose-Hoover at cutoff 3.0
        _case("thermostat_mixed_2m", kind="thermostat", cx=81, cy=81, cz=80, holes=2368, rho=0.7, T=0.9, rc=3.0,
              precision=MIXED, steps=20, energy_every=10),
        # the uneven ensemble: 256 boxes of 2000 to 65536 particles, densities 0.3 to 0.8
        _case("ensemble_mixed_256", kind="ensemble", boxes=256, precision=MIXED, flags=B.MD_F_GRAPH, steps=20),
        # one evaluation of new positions: pair list, forces, energies and pressure
        _case("static_fp64_100k", kind="static", cx=30, cy=29, cz=29, holes=917, rho=0.6),
        # the pair list itself, taken out in caller order
        _case("neighbors_fp64_32k", kind="neighbors", cx=20, cy=20, cz=20, holes=31),
        # bubble analysis of an expanded box: subcells of edge 3, gas below density 0.2
        _case("bubbles_2m", kind="bubbles", cx=81, cy=81, cz=81, holes=28612, rho=0.526, precision=MIXED, p_gas=0.12),
    ]


def draw(rng):
    def cells(lo, hi, limit=200 ** 3):
        """FCC cells per axis for about lo..hi particles, sides up to 1.5 apart, and some holes."""
        n = math.exp(rng.uniform(math.log(lo), math.log(hi)))
        side = (n / 4.0) ** (1.0 / 3.0)
        cx, cy, cz = (max(7, round(side * rng.uniform(0.8, 1.25))) for _ in range(3))
        while cx * cy * cz > limit:
            cx -= 1
            cy -= 1
        return dict(cx=cx, cy=cy, cz=cz, holes=rng.randrange(max(1, cx * cy * cz // 8)))

    state = dict(rho=round(rng.uniform(0.45, 0.75), 3), T=round(rng.uniform(0.7, 1.2), 3))
    prec = rng.choice([FP64, MIXED])
    kind = rng.choice(["nve", "nve", "nve", "nve", "thermostat", "ensemble", "static", "neighbors", "bubbles"])
    graph = rng.choice([0, B.MD_F_GRAPH])
    if kind == "nve":
        size = cells(3000, 24_000_000)
        fl = graph
        if prec == FP64:
            fl |= rng.choice([0, 0, 0, B.MD_F_FAST_RCP])
        c = _case(**size, **state, precision=prec, flags=fl, rc=rng.choice([2.5, 2.5, 3.0]),
                  policy=rng.choice([B.MD_REBUILD_DUTC, B.MD_REBUILD_DUTC, B.MD_REBUILD_DISPLACEMENT]),
                  steps=rng.randrange(4, 21), calls=rng.choice([1, 1, 2]))
        most = max(work(x)["bytes"] for x in listed())
        while work(c)["bytes"] > most:  # no dearer than the headline box
            c["calls"], c["steps"] = 1, c["steps"] - 1
        return c
    if kind == "thermostat":
        return _case(kind=kind, **cells(3000, 3_000_000), **state, rc=rng.choice([2.5, 3.0]), precision=prec,
                     steps=rng.randrange(4, 21), energy_every=rng.choice([0, 5, 10]))
    if kind == "ensemble":
        return _case(kind=kind, boxes=rng.randrange(3, 257), precision=prec, flags=graph, steps=rng.randrange(4, 21))
    if kind == "static":
        return _case(kind=kind, **cells(3000, 4_000_000), **state, rc=rng.choice([2.5, 3.0]), precision=prec)
    if kind == "neighbors":
        return _case(kind=kind, **cells(3000, 300_000), **state, precision=prec)
    return _case(kind="bubbles", **cells(30_000, 8_000_000), rho=round(rng.uniform(0.45, 0.6), 3), precision=prec,
                 p_gas=round(rng.uniform(0.02, 0.4), 3))


# ---------------------------------------------------------------- states

def _fcc_state(cx, cy, cz, holes, rho, T, gen):
    """Jittered FCC block with `holes` sites removed, at density rho; returns
    (positions, velocities, box) with the arrays on the GPU."""
    dev = gen.device
    n = 4 * cx * cy * cz - holes
    a = (n / (rho * cx * cy * cz)) ** (1.0 / 3.0)
    ix = torch.arange(cx, device=dev, dtype=torch.float64)
    iy = torch.arange(cy, device=dev, dtype=torch.float64)
    iz = torch.arange(cz, device=dev, dtype=torch.float64)
    z, y, x = torch.meshgrid(iz, iy, ix, indexing="ij")
    cell = torch.stack([x, y, z], dim=-1).reshape(-1, 1, 3)
    basis = torch.tensor([[0.0, 0.0, 0.0], [0.5, 0.5, 0.0], [0.5, 0.0, 0.5], [0.0, 0.5, 0.5]], device=dev,
                         dtype=torch.float64)
    q = ((cell + basis) * a).reshape(-1, 3)
    del cell, x, y, z
    if holes:
        keep = torch.ones(q.shape[0], dtype=torch.bool, device=dev)
        keep[torch.randperm(q.shape[0], generator=gen, device=dev)[:holes]] = False
        q = q[keep]
    box = torch.tensor([cx * a, cy * a, cz * a], dtype=torch.float64, device=dev)
    j = torch.rand(q.shape, generator=gen, device=dev, dtype=torch.float64)
    q += (2.0 * j - 1.0) * (JITTER * a / math.sqrt(2.0))
    del j
    q = torch.where(q < 0.0, q + box, torch.where(q >= box, q - box, q))
    v = torch.randn(q.shape, generator=gen, device=dev, dtype=torch.float64) * math.sqrt(T)
    v -= v.mean(dim=0)
    return q.contiguous(), v, (cx * a, cy * a, cz * a)


def _bubble_state(case, gen):
    """The expanded liquid with a gas fraction: the particles of randomly chosen subcells
    (edge 3) are moved onto others, so that those hold none or few."""
    q, v, box = _fcc_state(case["cx"], case["cy"], case["cz"], case["holes"], case["rho"], case["T"], gen)
    L = torch.tensor(box, dtype=torch.float64, device=q.device)
    ns = torch.floor(L / 3.0)
    at = torch.minimum((q * (ns / L)).long(), (ns - 1).long())
    nx, ny, nz = (int(k) for k in ns.tolist())
    sub = (at[:, 2] * ny + at[:, 1]) * nx + at[:, 0]
    gas = torch.rand(nx * ny * nz, generator=gen, device=q.device) < case["p_gas"]
    out = gas[sub] & (torch.rand(q.shape[0], generator=gen, device=q.device) < 0.85)
    into = (~gas).nonzero().flatten()
    to = into[torch.randint(into.numel(), (q.shape[0],), generator=gen, device=q.device)]
    there = torch.stack([to % nx, (to // nx) % ny, to // (nx * ny)], dim=1).double()
    there = (there + 0.01 + 0.98 * torch.rand(q.shape, generator=gen, device=q.device, dtype=torch.float64)) * (L / ns)
    return torch.where(out[:, None], there, q).contiguous(), v, box


def _ensemble_boxes(case, seed):
    """(cx, cy, cz, holes, rho, T) of each box: the sizes of inputs.batch_spec, every site
    count made up to a whole FCC block."""
    spec = inputs.batch_spec(case["boxes"], seed=5)
    got = []
    for n, rho, T in zip(spec.n.tolist(), spec.rho.tolist(), spec.T.tolist()):
        nc = math.ceil((n / 4.0) ** (1.0 / 3.0) - 1e-12)
        nz = max(1, math.ceil(n / (4.0 * nc * nc)))
        got.append((nc, nc, nz, 4 * nc * nc * nz - n, rho, T))
    return got


def _states(case, seed):
    """[(positions, velocities, box)] of the case's boxes."""
    gen = torch.Generator(device="cuda").manual_seed(seed)
    if case["kind"] == "ensemble":
        return [_fcc_state(*b, gen) for b in _ensemble_boxes(case, seed)]
    if case["kind"] == "bubbles":
        return [_bubble_state(case, gen)]
    return [_fcc_state(case["cx"], case["cy"], case["cz"], case["holes"], case["rho"], case["T"], gen)]


def prepare(case, seed):
    st = _states(case, seed)
    params = [B.make_params(q.shape[0], box, rc=case["rc"], skin=case["skin"], dt=DT, precision=case["precision"],
                            rebuild=case["policy"], flags=case["flags"]) for q, _, box in st]
    ctx = B.Context(params if case["kind"] == "ensemble" else params[0])
    if case["kind"] == "thermostat":
        ctx.set_thermostat(case["T"], 0.5)
    s = {"case": case, "ctx": ctx}
    if len(st) == 1:
        s["pos"], s["vel"] = st[0][0], st[0][1]
    else:
        s["pos"], s["vel"] = torch.cat([x[0] for x in st]), torch.cat([x[1] for x in st])
    if case["kind"] == "bubbles":  # the analysis looks at a run's current state
        ctx.set_state(s["pos"], s["vel"])
        nsub = math.prod(int(math.floor(x / 3.0)) for x in st[0][2])
        s["roots"], s["sizes"] = np.full(nsub, -1), np.full(nsub, -1)  # room for every number of bubbles
    if case["kind"] == "neighbors":
        s["partners"] = torch.full((64 * s["pos"].shape[0],), -1, dtype=torch.int32, device="cuda")
    return s


# ---------------------------------------------------------------- one pass

def run(state):
    case, ctx = state["case"], state["ctx"]
    kind = case["kind"]
    mixed = case["precision"] == MIXED
    low = (lambda t: t.float()) if mixed else (lambda t: t)
    num = (lambda a: np.asarray(a, dtype=np.float32 if mixed else np.float64))
    if kind == "bubbles":
        r = ctx.bubbles(side=3.0, rho_gas=0.2, fields=True)
        for k in ("roots", "sizes"):  # a program's own buffer, as long for every state
            state[k][:r[k].size] = r[k]
            state[k][r[k].size:] = -1
        return {"counts": r["counts"], "labels": r["labels"], "roots": state["roots"], "sizes": state["sizes"],
                "nbubbles": int(r["nbubbles"]), "ngas": int(r["ngas"]), "largest": int(r["largest"])}
    ctx.set_state(state["pos"], state["vel"])
    if kind == "neighbors":
        ctx.build_neighbors()
        cells, ncell = ctx.get_cells()
        ptr, partners = ctx.get_neighbors()
        all_partners = state["partners"]
        all_partners[:partners.numel()] = partners
        all_partners[partners.numel():] = -1
        return {"cells": cells, "key_ptr": ptr, "partners": all_partners}
    if kind == "static":
        f = ctx.compute_forces()
        ke, pe = ctx.energy()
        return {"force": low(f), "energy": num([ke, pe]), "pressure": num(ctx.pressure())}
    for _ in range(case["calls"]):
        ctx.step(case["steps"], energy_every=case["energy_every"])
    q, v = ctx.get_state()
    out = {"pos": q, "vel": low(v)}
    if case["energy_every"]:
        ke, pe = ctx.energy_series()
        out["ke"], out["pe"] = num(ke), num(pe)
    if kind == "thermostat":
        xi, eta = ctx.get_thermostat()
        out["xi"] = num(xi)
    return out


# ---------------------------------------------------------------- what a pass cannot do without

def _boxes_of(case):
    if case["kind"] == "ensemble":
        return [(4 * b[0] * b[1] * b[2] - b[3], b[4]) for b in _ensemble_boxes(case, 0)]
    return [(4 * case["cx"] * case["cy"] * case["cz"] - case["holes"], case["rho"])]


def work(case):
    """Per particle and step: position and velocity read and written (96 bytes) and the half
    pair list read (4 bytes an entry); 25 flops for a pair within the cutoff.  Static calls:
    inputs read, outputs written."""
    kind, rl, rc = case["kind"], case["rc"] + case["skin"], case["rc"]
    by = fl = 0.0
    for n, rho in _boxes_of(case):
        half = rho * 2.0 * math.pi / 3.0 * rl ** 3
        pairs = rho * 2.0 * math.pi / 3.0 * rc ** 3
        if kind == "bubbles":
            vol = n / rho / 27.0
            by += 24.0 * n + 5.0 * vol
            fl += 6.0 * n
        elif kind == "neighbors":
            by += 48.0 * n + 12.0 * n + 8.0 * n * half
            fl += 8.0 * n * half
        elif kind == "static":
            by += 48.0 * n + 24.0 * n + 4.0 * n * half
            fl += 30.0 * n * pairs
        else:
            k = case["steps"] * case["calls"]
            by += k * n * (96.0 + 4.0 * half)
            fl += k * n * 25.0 * pairs
    return {"bytes": by, "flops": fl}


# ---------------------------------------------------------------- 64-bit reference

def _pairs(q, L, r):
    """All pairs i < j within r (minimum image), from padded tables of cells of side >= r
    (at least three to an axis)."""
    dev = q.device
    nb = [max(3, int(math.floor(float(x) / r))) for x in L]
    nc = nb[0] * nb[1] * nb[2]
    qw = q - L * torch.floor(q / L)
    n3 = torch.tensor(nb, device=dev)
    c = torch.minimum((qw * (n3 / L)).long().clamp_(min=0), n3 - 1)
    cid = (c[:, 2] * nb[1] + c[:, 1]) * nb[0] + c[:, 0]
    order = torch.argsort(cid)
    cnt = torch.bincount(cid, minlength=nc)
    start = torch.cumsum(cnt, 0) - cnt
    M = int(cnt.max())
    tab = torch.full((nc, M), -1, dtype=torch.long, device=dev)
    sc = cid[order]
    tab[sc, torch.arange(q.shape[0], device=dev) - start[sc]] = order
    ids = torch.arange(nc, device=dev)
    x, y, z = ids % nb[0], (ids // nb[0]) % nb[1], ids // (nb[0] * nb[1])
    fwd = [(dx, dy, dz) for dz in (-1, 0, 1) for dy in (-1, 0, 1) for dx in (-1, 0, 1) if (dz, dy, dx) >= (0, 0, 0)]
    step = max(1, (1 << 24) // (M * M))
    gi, gj = [], []
    for dx, dy, dz in fwd:
        other = (((z + dz) % nb[2]) * nb[1] + (y + dy) % nb[1]) * nb[0] + (x + dx) % nb[0]
        for c0 in range(0, nc, step):
            a, b = tab[c0:c0 + step, :, None], tab[other[c0:c0 + step]][:, None, :]
            ok = (a >= 0) & (b >= 0)
            if (dx, dy, dz) == (0, 0, 0):
                ok &= a < b
            k = ok.nonzero()
            i, j = tab[c0 + k[:, 0], k[:, 1]], tab[other[c0 + k[:, 0]], k[:, 2]]
            d = q[j] - q[i]
            d -= L * torch.round(d / L)
            near = (d * d).sum(1) < r * r
            gi.append(i[near])
            gj.append(j[near])
    return torch.cat(gi), torch.cat(gj)


class _Exact:
    """Truncated LJ (Eq. 1), velocity Verlet and the list-rebuild rule of the run, plainly."""

    def __init__(self, case, q, v, box):
        self.case, self.q, self.v = case, q.clone(), v.clone()
        self.L = torch.tensor(box, dtype=torch.float64, device=q.device)
        self.rc2 = case["rc"] ** 2
        s = 1.0 / self.rc2
        self.c2, self.c0 = 6.0 * s ** 7 - 3.0 * s ** 4, -7.0 * s ** 6 + 4.0 * s ** 3
        # margin of this function's own list; a box may be as small as three list radii
        self.rp = min(case["rc"] + 0.6, min(box) / 3.0)
        self.at = None

    def wrap(self):
        q, L = self.q, self.L
        q = torch.where(q < 0.0, q + L, q)
        self.q = torch.where(q >= L, q - L, q)

    def forces(self):
        """(F, pe, vir) at the current positions."""
        if self.at is not None:
            d = self.q - self.at
            d -= self.L * torch.round(d / self.L)
            if 2.0 * float((d * d).sum(1).max()) ** 0.5 >= self.rp - self.case["rc"]:
                self.at = None
        if self.at is None:
            self.i, self.j = _pairs(self.q, self.L, self.rp)
            self.at = self.q.clone()
        F = torch.zeros_like(self.q)
        pe = vir = 0.0
        for k in range(0, self.i.numel(), 1 << 24):
            i, j = self.i[k:k + (1 << 24)], self.j[k:k + (1 << 24)]
            d = self.q[j] - self.q[i]
            d -= self.L * torch.round(d / self.L)
            r2 = (d * d).sum(1)
            near = r2 < self.rc2
            inv3 = r2 ** -3
            f = torch.where(near, (24.0 * inv3 - 48.0 * inv3 * inv3) / r2 + 8.0 * self.c2, 0.0)
            e = torch.where(near, 4.0 * (inv3 * inv3 - inv3 + self.c2 * r2 + self.c0), 0.0)
            pe += float(e.sum())
            vir += float((f * r2).sum())
            d *= f[:, None]
            F.index_add_(0, i, d)
            F.index_add_(0, j, -d)
        return F, pe, vir

    def ke(self):
        return 0.5 * float((self.v * self.v).sum())


def _exact_run(case, q, v, box):
    x = _Exact(case, q, v, box)
    h, D, built = 0.5 * DT, 0.0, None
    thermo = case["kind"] == "thermostat"
    g = 3.0 * q.shape[0] - 3.0
    gT, Q, xi = g * case["T"], g * case["T"] * 0.25, 0.0
    x.wrap()
    built = x.q.clone()
    F, _, _ = x.forces()
    kes, pes = [], []

    def bath():
        nonlocal xi
        ke = x.ke()
        xi += 0.5 * h * (2.0 * ke - gT) / Q
        s = math.exp(-xi * h)
        x.v *= s
        xi += 0.5 * h * (2.0 * ke * s * s - gT) / Q

    for _ in range(case["calls"]):
        for k in range(1, case["steps"] + 1):
            if thermo:
                bath()
            x.v += h * F
            x.q += DT * x.v
            D += DT * float((x.v * x.v).sum(1).max()) ** 0.5
            if case["policy"] == B.MD_REBUILD_DUTC:
                again = 2.0 * D > case["skin"]
            else:
                again = 2.0 * float(((x.q - built) ** 2).sum(1).max()) ** 0.5 > case["skin"]
            if again:
                x.wrap()
                D, built = 0.0, x.q.clone()
            F, pe, _ = x.forces()
            x.v += h * F
            if thermo:
                bath()
            if case["energy_every"] and k % case["energy_every"] == 0:
                kes.append(x.ke())
                pes.append(pe)
    return x.q, x.v, np.array(kes).reshape(-1, 1), np.array(pes).reshape(-1, 1), xi


def exact(case, seed):
    kind = case["kind"]
    if kind in ("bubbles", "neighbors"):  # whole numbers
        return None
    if sum(n for n, _ in _boxes_of(case)) > EXACT_MAX:
        return None
    states = _states(case, seed)
    if kind == "static":
        q, v, box = states[0]
        x = _Exact(case, q, v, box)
        x.wrap()
        F, pe, vir = x.forces()
        return {"force": F, "energy": np.array([x.ke(), pe]),
                "pressure": np.array([(2.0 * x.ke() - vir) / (3.0 * box[0] * box[1] * box[2])])}
    got = [_exact_run(case, *s) for s in states]
    out = {"pos": torch.cat([r[0] for r in got]), "vel": torch.cat([r[1] for r in got])}
    if case["energy_every"]:
        out["ke"], out["pe"] = got[0][2], got[0][3]
    if kind == "thermostat":
        out["xi"] = np.array([got[0][4]])
    return out
