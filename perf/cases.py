"""The workloads whose time and results are followed, through the public entry points.

Scenes are lattices with a seeded disorder, as a flow in motion has it: fluid
particles displaced by up to a tenth of the spacing, a smooth vortical
velocity with a little noise, a hydrostatic density with noise of 1e-3.  The
sizes are those of the repository's own scenes (still-water tank, dam breaks,
batched tanks, channel).  A case's `op` is the call it makes:

  forces   Simulation.forces: the time derivatives on built lists
  build    Simulation.build: the neighbour search of a moved state
  steps    Simulation.run: ten steps launched call by call from a given state
  unit     the same ten steps as one HIP-graph replay (capture_unit)
  backward sph_forces_backward: the adjoint of the derivatives
  rollout  AdjointRollout: ten fixed steps and their reverse
"""
from __future__ import annotations

import math
import random
from types import SimpleNamespace

import numpy as np
import torch

from paper_2207_11328_amd import abi
from paper_2207_11328_amd.adjoint import AdjointRollout
from paper_2207_11328_amd.sim import Simulation

DEV = "cuda"
STEPS = 10          # of a unit: lists are rebuilt every ten steps
LAYERS = 3          # of boundary particles
MODEL = {"kernel": 0, "formulation": 0, "visc": 0, "delta": 0.0, "nu": 0.0}


def _case(name, op, scene, dp, box, column, brick=0, **model):
    """box, column: inside of the tank and water in it, in particles along x, y, z."""
    c = {"name": name, "op": op, "scene": scene, "dp": dp, "brick": brick}
    c.update(dict(zip(("bx", "by", "bz"), box)))
    c.update(dict(zip(("cx", "cy", "cz"), column)))
    c.update(MODEL)
    c.update(model)
    return c


TANK_8K = ((20, 20, 20), (20, 20, 20))
DAM_64K = ((149, 62, 56), (37, 62, 28))
DAM_1M = ((372, 155, 139), (93, 155, 69))
CHANNEL_16M = ((800, 200, 100), (800, 200, 100))


def listed():
    return [
        # the smallest calls: the still-water tank, 8,000 fluid and 7,548 wall particles
        _case("forces_tank_8k", "forces", "tank", 0.02, *TANK_8K),
        # the same tank stepped as the quick start does, one call after the other
        _case("steps_tank_8k", "steps", "tank", 0.02, *TANK_8K),
        # a middle size in graph replays, with the brick shape the autotuner takes there
        _case("unit_dam_64k", "unit", "tank", 0.0107, *DAM_64K, brick=2),
        # another model than the default: cubic spline, Landrini-Morris, Morris viscosity, density diffusion
        _case("forces_dam_64k_variant", "forces", "tank", 0.0107, *DAM_64K, kernel=1, formulation=1, visc=1,
              delta=0.1, nu=1e-4),
        # the adjoint at the size of the differentiable dam break, alone and in a rollout
        _case("backward_dam_64k", "backward", "tank", 0.0107, *DAM_64K, visc=1, nu=1e-4),
        _case("rollout_dam_64k", "rollout", "tank", 0.0107, *DAM_64K, brick=2),
        # the benchmark's dam break, 994,635 fluid and 627,096 wall particles: rebuild, derivatives, adjoint, unit
        _case("build_dam_1m", "build", "tank", 0.0043, *DAM_1M),
        _case("forces_dam_1m", "forces", "tank", 0.0043, *DAM_1M),
        _case("backward_dam_1m", "backward", "tank", 0.0043, *DAM_1M),
        _case("unit_dam_1m", "unit", "tank", 0.0043, *DAM_1M),
        # many scenes in one grid, each with its own viscosity, time step and clock
        _case("unit_batch_32", "unit", "batch", 0.01, (0, 0, 0), (0, 0, 0), tanks=32, tank_seed=4, least=2000,
              most=60000),
        # the largest: the channel, periodic in y, 16.0M fluid and 0.6M wall particles
        _case("forces_channel_16m", "forces", "channel", 0.005, *CHANNEL_16M),
    ]


def draw(rng):
    op = rng.choice(["forces", "forces", "build", "unit", "steps", "backward", "backward", "rollout"])
    model = {"kernel": rng.choice([0, 0, 0, 1, 2, 3]), "formulation": rng.choice([0, 0, 1]),
             "visc": rng.choice([0, 0, 1, 2]), "delta": rng.choice([0.0, 0.0, 0.1])}
    model["nu"] = 1e-4 if model["visc"] else 0.0
    dp = round(math.exp(rng.uniform(math.log(0.004), math.log(0.02))), 4)
    brick = rng.choice([0, 0, 1, 2])
    if op in ("unit", "forces") and rng.random() < 0.2:
        c = _case("", op, "batch", dp, (0, 0, 0), (0, 0, 0), brick, tanks=rng.randint(2, 40),
                  tank_seed=rng.randint(0, 10 ** 6), least=500, most=30000, **model)
    else:
        top = {"rollout": 2e5, "steps": 3e5}.get(op, 1.5e6)
        fluid = math.exp(rng.uniform(math.log(3e3), math.log(top)))
        ax, ay = rng.uniform(0.6, 2.0), rng.uniform(0.6, 2.0)
        cz = max(4, int((fluid / (ax * ay)) ** (1 / 3)))
        column = (max(5, int(ax * cz)), max(9, int(ay * cz)), cz)
        if rng.random() < 0.3:
            c = _case("", op, "channel", dp, column, column, brick, **model)
        else:
            box = (int(column[0] * rng.uniform(1, 3)), column[1], int(cz * rng.uniform(1, 1.8)))
            c = _case("", op, "tank", dp, box, column, brick, **model)
    del c["name"]
    return c


# ---------------------------------------------------------------- scenes
def _params(case):
    h = 1.3 * case["dp"]
    return SimpleNamespace(dp=case["dp"], h=h, r_search=2.2 * h, rho0=1000.0, gamma=7.0, c0=20.0, alpha=0.01,
                           eps_visc=0.01, nu=case["nu"], g=(0.0, 0.0, -9.81), cfl=0.3, visc_model=case["visc"],
                           delta=case["delta"], kernel=case["kernel"], formulation=case["formulation"])


def _grid(lo, hi, rs, periodic):
    """Cells of side at least rs, an axis divided evenly."""
    rs = np.float32(rs)
    cs, nc = np.zeros(3, np.float32), np.zeros(3, np.int32)
    for d in range(3):
        L = hi[d] - lo[d]
        n = max(1, int(L / float(rs)))
        while n > 1 and np.float32(L / n) < rs:
            n -= 1
        cs[d], nc[d] = np.float32(L / n), n
    return SimpleNamespace(origin=np.array(lo), cell_size=cs, ncell=nc, periodic=periodic, cell_base=0)


def _lattice(lo, hi):
    ax = [torch.arange(a, b, device=DEV, dtype=torch.float64) for a, b in zip(lo, hi)]
    z, y, x = torch.meshgrid(ax[2], ax[1], ax[0], indexing="ij")
    return torch.stack([x.reshape(-1), y.reshape(-1), z.reshape(-1)], 1)


def _tank(p, box, column, gen, channel=False):
    """(positions, velocities, densities, number of fluid particles) of a tank
    with its lower inside corner at the origin; a channel has no y walls."""
    dp = p.dp
    xf = (_lattice((0, 0, 0), column) + 0.5) * dp
    lo = (-LAYERS, 0 if channel else -LAYERS, -LAYERS)
    hi = (box[0] + LAYERS, box[1] + (0 if channel else LAYERS), box[2])
    k = _lattice(lo, hi)
    inside = ((k >= 0) & (k < torch.tensor([float(b) for b in box], device=DEV, dtype=torch.float64)))
    xb = (k[~inside.all(1)] + 0.5) * dp
    nf = xf.shape[0]
    xf = xf + (torch.rand(xf.shape, generator=gen, device=DEV, dtype=torch.float64) - 0.5) * (0.2 * dp)
    if channel:
        xf[:, 1] %= box[1] * dp
    L = dp * max(column)
    u = 0.5 * torch.stack([torch.sin(3 * xf[:, 2] / L + 1), torch.cos(4 * xf[:, 0] / L),
                           torch.sin(5 * xf[:, 1] / L)], 1)
    u = u + 0.05 * torch.randn(u.shape, generator=gen, device=DEV, dtype=torch.float64)
    x = torch.cat([xf, xb])
    v = torch.zeros_like(x)
    v[:nf] = u
    B = p.rho0 * p.c0 ** 2 / p.gamma
    rho = p.rho0 * (1 + p.rho0 * 9.81 * (column[2] * dp - x[:, 2]).clamp(min=0) / B) ** (1 / p.gamma)
    rho = rho * (1 + 1e-3 * torch.randn(rho.shape, generator=gen, device=DEV, dtype=torch.float64))
    return x, v, rho, nf


def _encode(grid, x):
    """Cell indices and float32 offsets from the cell centres, in [-cs/2, cs/2)."""
    cs = torch.tensor(grid.cell_size, device=DEV)
    nc = torch.tensor(grid.ncell, device=DEV, dtype=torch.int64)
    rel = x - torch.tensor(grid.origin, device=DEV)
    c = torch.floor(rel / cs.double()).long()
    c = torch.minimum(c.clamp(min=0), nc - 1)
    off = (rel - (c + 0.5) * cs.double()).float()
    over = (off >= 0.5 * cs) & (c < nc - 1)
    off = torch.where(over, off - cs, off)
    off = torch.minimum(torch.maximum(off, -0.5 * cs), torch.nextafter(0.5 * cs, torch.zeros_like(cs)))
    c = c + over
    return (c[:, 0] + nc[0] * (c[:, 1] + nc[1] * c[:, 2])).int(), off


def _scene(case, seed):
    """The state a program starts from, on the GPU, in lattice order."""
    gen = torch.Generator(device=DEV)
    gen.manual_seed(seed * 7919 + 13)
    p = _params(case)
    rs = float(np.float32(p.r_search))
    alpha = scene_of = None
    if case["scene"] == "batch":
        # tanks of log-uniform size along z, at least two empty layers apart,
        # each started at a multiple of three cells
        r = random.Random(case["tank_seed"])
        parts, z, spans = [], 0, []
        ext = [0, 0]
        for _ in range(case["tanks"]):
            target, a = math.exp(r.uniform(math.log(case["least"]), math.log(case["most"]))), r.uniform(0.3, 2.0)
            nl = max(3, int(round((target / a) ** (1 / 3))))
            nh = max(3, int(round(a * nl)))
            box = (3 * nl, nl, int(math.ceil(1.5 * max(nh, nl))))
            x, v, rho, nf = _tank(p, box, (nl, nl, nh), gen)
            x = x + LAYERS * p.dp
            e = [math.ceil((b + 2 * LAYERS) * p.dp / rs - 1e-9) for b in box[:2]]
            ez = math.ceil(1.5 * (box[2] + LAYERS) * p.dp / rs)
            x[:, 2] += z * rs
            parts.append((x, v, rho, nf))
            spans.append((z, r.uniform(0.005, 0.05)))
            ext = [max(ext[0], e[0]), max(ext[1], e[1])]
            z = -(-(z + ez + 2) // 3) * 3
        grid = SimpleNamespace(origin=np.zeros(3), cell_size=np.full(3, np.float32(rs), np.float32),
                               ncell=np.array([ext[0], ext[1], z], np.int32), periodic=0, cell_base=0)
        layer = np.zeros(z, np.int32)
        coef = np.zeros(z, np.float32)
        for k, (z0, a) in enumerate(spans):
            layer[z0:], coef[z0:] = k, a
        scene_of = np.repeat(layer, ext[0] * ext[1]).astype(np.int32)
        alpha = np.repeat(coef, ext[0] * ext[1]).astype(np.float32)
        x = torch.cat([q[0] for q in parts])
        v = torch.cat([q[1] for q in parts])
        rho = torch.cat([q[2] for q in parts])
        kind = torch.cat([(torch.arange(q[0].shape[0], device=DEV) >= q[3]).int() for q in parts])
    else:
        box, column = [tuple(case[a + b] for b in "xyz") for a in "bc"]
        channel = case["scene"] == "channel"
        x, v, rho, nf = _tank(p, box, column, gen, channel)
        m = LAYERS * p.dp
        lo = (-m, 0.0 if channel else -m, -m)
        hi = (box[0] * p.dp + m, box[1] * p.dp + (0.0 if channel else m), 1.5 * box[2] * p.dp + m)
        grid = _grid(lo, hi, rs, 2 if channel else 0)
        kind = (torch.arange(x.shape[0], device=DEV) >= nf).int()
    n = x.shape[0]
    cell, off = _encode(grid, x)
    mass = torch.full((n, 1), float(np.float32(p.rho0 * p.dp ** 3)), device=DEV)
    pos = torch.cat([off, mass], 1)
    vel = torch.cat([v, rho[:, None]], 1).float()
    info = (kind << 30) | torch.arange(n, device=DEV, dtype=torch.int32)
    return SimpleNamespace(case=case, p=p, grid=grid, cell=cell, pos=pos, vel=vel, info=info, n=n, alpha=alpha,
                           scene_of=scene_of, gen=gen)


def _host(s):
    return (s.cell.cpu().numpy(), s.pos.cpu().numpy(), s.vel.cpu().numpy(), s.info.cpu().numpy().view(np.uint32))


def _order(s):
    """Places of the particles in (cell, type, id) order."""
    return torch.argsort(s.cell.long() * (1 << 32) + (s.info.long() & 0xFFFFFFFF))


def _cotangents(s, seed):
    """Upstream adjoints of the derivatives, or of a final state, in sorted
    order: growing outwards from the middle of the scene, as a loss on
    positions has them, with noise."""
    gen = torch.Generator(device=DEV)
    gen.manual_seed(seed * 104729 + 7)
    order = _order(s)
    cell, nc = s.cell[order].long(), [int(v) for v in s.grid.ncell]
    c = torch.stack([cell % nc[0], (cell // nc[0]) % nc[1], cell // (nc[0] * nc[1])], 1)
    x = (c + 0.5) * torch.tensor(s.grid.cell_size, device=DEV) + s.pos[order, :3]
    x = x - x.mean(0)
    x = torch.cat([x, x.norm(dim=1, keepdim=True)], 1) / x.abs().max()
    return tuple(x + 0.1 * torch.randn((s.n, 4), generator=gen, device=DEV) for _ in range(2))


DRIFT = 2e-4  # seconds between the last rebuild and the one of a `build` case
DT = 5e-5     # fixed step of a rollout


# ---------------------------------------------------------------- the calls
def prepare(case, seed):
    s = _scene(case, seed)
    op = case["op"]
    brick = abi.sph_brick_shapes()[case["brick"]]
    st = SimpleNamespace(op=op, n=s.n)
    if op == "rollout":
        st.roll = AdjointRollout(s.grid, s.p, *_host(s), steps=STEPS, dt=DT, brick=brick)
        a, b = _cotangents(s, seed)
        a[:, 3] = 0
        st.gpos, st.gvel = a, b
        return st
    sim = st.sim = Simulation(s.grid, s.p, *_host(s), brick=brick, cell_alpha=s.alpha, cell_scene=s.scene_of)
    sim.build()
    if op == "build":
        sim.pos[:, :3] += DRIFT * sim.vel[:, :3]
    if op == "backward":
        cap = sim.capacity
        st.gforce = _cotangents(s, seed)[0]
        st.gpos, st.gvel = torch.zeros((cap, 4), device=DEV), torch.zeros((cap, 4), device=DEV)
        st.gparams = torch.zeros(3, dtype=torch.float64, device=DEV)
        st.ws = torch.zeros(abi.sph_forces_backward_workspace_bytes(cap, sim.n_cells), dtype=torch.uint8, device=DEV)
    if op in ("steps", "unit"):
        st.saved = [(t, t.clone()) for t in (sim.cell, sim.pos, sim.vel, sim.info, sim.d_time)]
        if op == "unit":
            sim.capture_unit()
    sim.check_status()
    return st


def run(st):
    if st.op == "rollout":
        r = st.roll
        r.reset()
        s = r.forward()
        pos, vel = s.pos, s.vel
        gp, gv, gpar = r.backward(st.gpos, st.gvel)
        return {"pos": pos, "vel": vel, "gpos": gp, "gvel": gv, "gparams": gpar.float()}
    s = st.sim
    if st.op == "forces":
        return s.forces()
    if st.op == "build":
        s.build()
        return {"cell": s.cell, "pos": s.pos, "vel": s.vel, "info": s.info, "start": s.cell_start,
                "end": s.cell_end, "count": s.neib_count, "neibs": s.neibs, "status": s.status}
    if st.op == "backward":
        abi.sph_forces_backward(s.g, s.p, s.parts, s.neibs, s.neib_count, s.max_neibs, st.gforce, st.gpos, st.gvel,
                                st.gparams, False, st.ws, None, *s.brick_args())
        return {"gpos": st.gpos, "gvel": st.gvel, "gparams": st.gparams.float()}
    for t, saved in st.saved:  # from the saved state, as a program that repeats a run does
        t.copy_(saved)
    if st.op == "steps":
        s.run(STEPS)
    else:
        s.replay_units(1)
    return {"cell": s.cell, "info": s.info, "pos": s.pos, "vel": s.vel, "time": s.d_time.float(),
            "dt": s.d_dt.float()}


def _counts(case):
    """About how many particles, particles with neighbours, and listed entries."""
    if case["scene"] == "batch":
        fluid = case["tanks"] * (case["most"] - case["least"]) / math.log(case["most"] / case["least"])
        return 3 * fluid, 1.4 * fluid, 85 * fluid
    cx, cy, cz = case["cx"], case["cy"], case["cz"]
    bx, by, bz = case["bx"], case["by"], case["bz"]
    w = 0 if case["scene"] == "channel" else 2 * LAYERS
    fluid = cx * cy * cz
    wall = (bx + 2 * LAYERS) * (by + w) * (bz + LAYERS) - bx * by * bz
    wet = min(wall, (cx + LAYERS) * (cy + w) * (cz + LAYERS) - fluid)
    return fluid + wall, fluid + wet, 92 * fluid


def work(case):
    """Bytes: state and lists read once, results written once.  Flops: 43 of a
    pair term (110 of its adjoint), 9 of a distance test per listed pair."""
    n, _, listed_pairs = _counts(case)
    pairs = 0.87 * listed_pairs
    forces = (52 * n + 2 * listed_pairs, 43 * pairs)
    back = (84 * n + 2 * listed_pairs, 110 * pairs)
    build = (88 * n + 6 * listed_pairs, 9 * listed_pairs)
    step = tuple(2 * f + g for f, g in zip(forces, (200 * n, 40 * n)))
    unit = tuple(b + STEPS * s for b, s in zip(build, step))
    both = tuple(u + STEPS * (2 * b + c) for u, b, c in zip(unit, back, (200 * n, 40 * n)))
    total = {"forces": forces, "backward": back, "build": build, "unit": unit, "steps": unit, "rollout": both}
    b, f = total[case["op"]]
    return {"bytes": b, "flops": f}


# ---------------------------------------------------------------- the same in 64 bits
def _f32(v):
    return float(np.float32(v))


class _Exact:
    """The sums over pairs in float64, on the sorted state of a scene."""

    CHUNK = 4_000_000

    def __init__(self, s):
        self.s, self.p, g = s, s.p, s.grid
        order = _order(s)
        self.order = order
        self.cell = s.cell[order].long()
        self.kind = (s.info[order].long() & 0xFFFFFFFF) >> 30
        self.off = s.pos[order, :3].double()
        self.m = s.pos[order, 3].double()
        self.u, self.rho = s.vel[order, :3].double(), s.vel[order, 3].double()
        self.nc = [int(v) for v in g.ncell]
        self.cs = torch.tensor(g.cell_size.astype(np.float64), device=DEV)
        self.cc = torch.stack([self.cell % self.nc[0], (self.cell // self.nc[0]) % self.nc[1],
                               self.cell // (self.nc[0] * self.nc[1])], 1)
        self.centre = (self.cc + 0.5) * self.cs
        p = self.p
        self.h, self.rs = _f32(p.h), _f32(p.r_search)
        self.alpha = torch.full((s.n,), _f32(p.alpha), device=DEV, dtype=torch.float64)
        if s.alpha is not None:
            self.alpha = torch.tensor(s.alpha, device=DEV)[self.cell].double()
        self.c0 = torch.tensor(_f32(p.c0), device=DEV, dtype=torch.float64)
        self.nu = torch.tensor(_f32(p.nu), device=DEV, dtype=torch.float64)
        self.kept = None

    def separation(self, x, i, j):
        d = (self.centre[i] - self.centre[j]) + (x[i] - x[j])
        for a in range(3):
            if (self.s.grid.periodic >> a) & 1:
                L = self.nc[a] * self.cs[a]
                d[:, a] -= L * torch.round(d[:, a].detach() / L)
        return d

    def pairs(self):
        """The listed pairs (i, j), in chunks; boundary particles list fluid ones only."""
        n, total = self.s.n, self.nc[0] * self.nc[1] * self.nc[2]
        cnt = torch.bincount(self.cell, minlength=total)
        start = torch.cumsum(cnt, 0) - cnt
        occ = int(cnt.max())
        step = max(1, 40_000_000 // (27 * occ))
        shifts = torch.tensor([(a, b, c) for c in (-1, 0, 1) for b in (-1, 0, 1) for a in (-1, 0, 1)], device=DEV)
        nc = torch.tensor(self.nc, device=DEV)
        for i0 in range(0, n, step):
            i = torch.arange(i0, min(n, i0 + step), device=DEV)
            c = self.cc[i][:, None, :] + shifts[None]
            ok = torch.ones(c.shape[:2], dtype=torch.bool, device=DEV)
            for a in range(3):
                if (self.s.grid.periodic >> a) & 1:
                    c[:, :, a] %= self.nc[a]
                else:
                    ok &= (c[:, :, a] >= 0) & (c[:, :, a] < nc[a])
            lin = torch.where(ok, c[:, :, 0] + nc[0] * (c[:, :, 1] + nc[1] * c[:, :, 2]), torch.zeros_like(c[:, :, 0]))
            num = torch.where(ok, cnt[lin], torch.zeros_like(lin))
            k = torch.arange(occ, device=DEV)
            slot = (k[None, None] < num[:, :, None]).reshape(len(i), -1).nonzero()
            row, t = slot[:, 0], slot[:, 1]
            j = start[lin][row, t // occ] + t % occ
            ii = i[row]
            d = self.separation(self.off, ii, j)
            keep = ((d * d).sum(1) < self.rs ** 2) & (ii != j) & ((self.kind[ii] == 0) | (self.kind[j] == 0))
            ii, j = ii[keep], j[keep]
            for a in range(0, len(ii), self.CHUNK):
                yield ii[a:a + self.CHUNK], j[a:a + self.CHUNK]

    def keep(self):
        self.kept = list(self.pairs())

    def chunks(self):
        return self.kept if self.kept is not None else self.pairs()

    def factor(self, r2):
        """F(r) = W'(r)/r."""
        h, k = self.h, self.p.kernel
        r = torch.sqrt(r2)
        q = r / h
        if k == 0:
            return 105 / (128 * math.pi * h ** 5) * (q - 2) ** 3
        if k == 1:
            return torch.where(q < 1, 2.25 * q - 3, -0.75 * (2 - q) ** 2 / q) / (math.pi * h ** 5)
        if k == 2:
            return 15 / (32 * math.pi * h ** 5) * (1 - 2 / q)
        C = 1 / (4 * math.pi * h ** 3 * (math.sqrt(math.pi) / 4 * math.erf(2) - 11 / 3 * math.exp(-4)))
        return -2 * C / h ** 2 * torch.exp(-q * q)

    def terms(self, x, u, rho, alpha, c0, nu, i, j):
        """Per pair: contributions to (a_i, Drho_i/Dt)."""
        p, h = self.p, self.h
        d = self.separation(x, i, j)
        r2 = (d * d).sum(1)
        near = (r2.detach() < _f32(2 * np.float32(h)) ** 2) & (r2.detach() > 0)
        i, j, d, r2 = i[near], j[near], d[near], r2[near]
        uu = u[i] - u[j]
        w = (uu * d).sum(1)
        mF = self.m[j] * self.factor(r2)
        ri, rj = rho[i], rho[j]
        rho0 = _f32(p.rho0)
        B = rho0 * c0 * c0 / 7

        def eos(r):
            b = r / rho0
            return B * (b ** 7 - 1), c0 * b ** 3

        (Pi, ci), (Pj, cj) = eos(ri), eos(rj)
        e2 = r2 + _f32(p.eps_visc) * h * h
        visc = -alpha[i] * h * (ci + cj) / (ri + rj) * w.clamp(max=0) / e2
        if p.formulation:
            s = (Pi + Pj) / (ri * rj)
            dr = ri / rj * mF * w
        else:
            s = Pi / ri ** 2 + Pj / rj ** 2
            dr = mF * w
        a = -(mF * (s + visc))[:, None] * d
        if p.visc_model == 1:
            a = a + (4 * nu * mF / (ri + rj))[:, None] * uu
        elif p.visc_model == 2:
            a = a + (20 * nu * mF / (ri + rj) * w / e2)[:, None] * d
        if p.delta:
            both = ((self.kind[i] == 0) & (self.kind[j] == 0)).double()
            dr = dr - both * 2 * _f32(p.delta) * h * c0 * (rj - ri) * mF * r2 / e2 / rj
        return i, a, dr

    def forces(self, x, u, rho):
        f = torch.zeros((self.s.n, 4), device=DEV, dtype=torch.float64)
        for i, j in self.chunks():
            i, a, dr = self.terms(x, u, rho, self.alpha, self.c0, self.nu, i, j)
            f.index_add_(0, i, torch.cat([a, dr[:, None]], 1))
        return f

    def reverse(self, x, u, rho, g):
        """Adjoints of (x, u, rho) and of (alpha, c0, nu) for the upstream g of the derivatives."""
        leaf = [t.detach().clone().requires_grad_(True) for t in (x, u, rho, self.alpha, self.c0, self.nu)]
        with torch.enable_grad():
            for i, j in self.chunks():
                i, a, dr = self.terms(*leaf, i, j)
                ((a * g[i, :3]).sum() + (dr * g[i, 3]).sum()).backward()
        z = [t.grad if t.grad is not None else torch.zeros_like(t) for t in leaf]
        return z[0], z[1], z[2], torch.stack([z[3].sum(), z[4], z[5]])

    def rate(self, u, f):
        """Time derivatives of (x, u, rho): fixed boundary particles, gravity on the fluid."""
        fl = (self.kind == 0).double()[:, None]
        g = torch.tensor([_f32(v) for v in self.p.g], device=DEV, dtype=torch.float64)
        return fl * u, fl * (f[:, :3] + g), f[:, 3]

    def step_size(self, rho, f, groups, n_groups):
        p, h = self.p, self.h
        fl = self.kind == 0
        c = _f32(p.c0) * (rho / _f32(p.rho0)) ** 3
        g = torch.tensor([_f32(v) for v in p.g], device=DEV, dtype=torch.float64)
        a = (f[:, :3] + g).norm(dim=1)
        z = torch.zeros(n_groups, device=DEV, dtype=torch.float64)
        cm = z.scatter_reduce(0, groups[fl], c[fl], "amax")
        am = z.scatter_reduce(0, groups[fl], a[fl], "amax")
        dt = torch.minimum(h / cm, torch.sqrt(h / am))
        if p.nu > 0:
            dt = dt.clamp(max=0.125 * h * h / _f32(p.nu))
        return _f32(p.cfl) * dt

    def state(self, x, u, rho):
        return torch.cat([x, self.m[:, None]], 1), torch.cat([u, rho[:, None]], 1)


def exact(case, seed):
    op = case["op"]
    if op == "build":  # whole numbers and moved inputs: nothing is computed
        return None
    s = _scene(case, seed)
    e = _Exact(s)
    x, u, rho = e.off, e.u, e.rho
    with torch.no_grad():
        if op == "forces":
            return e.forces(x, u, rho)
        e.keep()
        if op == "backward":
            gx, gu, gr, gp = e.reverse(x, u, rho, _cotangents(s, seed)[0].double())
            return {"gpos": torch.cat([gx, torch.zeros_like(gr)[:, None]], 1),
                    "gvel": torch.cat([gu, gr[:, None]], 1), "gparams": gp}
        groups, many = torch.zeros_like(e.cell), 1
        if s.scene_of is not None:
            groups, many = torch.tensor(s.scene_of, device=DEV)[e.cell].long(), int(s.scene_of.max()) + 1
        time = torch.zeros(many, device=DEV, dtype=torch.float64)
        tape = []
        for _ in range(STEPS):
            f = e.forces(x, u, rho)
            dt = torch.full((1,), DT, device=DEV, dtype=torch.float64) if op == "rollout" else \
                e.step_size(rho, f, groups, many)
            t = dt[groups]
            k = e.rate(u, f)
            y = (x + 0.5 * t[:, None] * k[0], u + 0.5 * t[:, None] * k[1], rho + 0.5 * t * k[2])
            tape.append(((x, u, rho), y))
            k = e.rate(y[1], e.forces(*y))
            x, u, rho = x + t[:, None] * k[0], u + t[:, None] * k[1], rho + t * k[2]
            time = time + dt
        pos, vel = e.state(x, u, rho)
        if op != "rollout":
            return {"cell": None, "info": None, "pos": pos, "vel": vel, "time": time, "dt": dt}
        gp, gv = _cotangents(s, seed)
        gx, gu, gr = gp[:, :3].double(), gv[:, :3].double(), gv[:, 3].double()
        fl = (e.kind == 0).double()[:, None]
        par = torch.zeros(3, device=DEV, dtype=torch.float64)
        for yn, ys in reversed(tape):
            up = torch.cat([DT * fl * gu, DT * gr[:, None]], 1)
            a, b, c, q = e.reverse(*ys, up)
            b = b + DT * fl * gx  # dL/dy*
            par = par + q
            up = torch.cat([0.5 * DT * fl * b, 0.5 * DT * c[:, None]], 1)
            gx, gu, gr = gx + a, gu + b + 0.5 * DT * fl * a, gr + c
            a, b, c, q = e.reverse(*yn, up)
            gx, gu, gr, par = gx + a, gu + b, gr + c, par + q
        back = torch.empty_like(e.order)
        back[e.order] = torch.arange(s.n, device=DEV)
        return {"pos": pos, "vel": vel, "gpos": torch.cat([gx, torch.zeros_like(gr)[:, None]], 1)[back],
                "gvel": torch.cat([gu, gr[:, None]], 1)[back], "gparams": par}
