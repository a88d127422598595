"""The work items of the brick kernels where they can go wrong: bricks that
hold more particles than LDS (cut into runs of rows, or left to the gather
path), grids of few bricks (cut so that every CU has work), lists at the
edges of a lane's runs of eight entries.  Against the FP64 oracle, to the
derivative bar of the parity tests (1e-5 of the magnitude scale)."""
import numpy as np
import pytest

from workloads import scenes as S

from parity import check_forces, compare_build, edge_allowance, log, make_sim, oracle_forces_of, torch_sync

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

SHAPES = [(3, 4, 3), (3, 3, 3), (3, 2, 3)]


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def _brick_totals(sc, brick):
    """Particles of every brick with its one-cell halo (closed axes)."""
    nx, ny, nz = (int(v) for v in sc.grid.ncell)
    cnt = np.bincount(sc.cell, minlength=nx * ny * nz).reshape(nz, ny, nx)
    return np.array([cnt[max(z - 1, 0):z + brick[2] + 1, max(y - 1, 0):y + brick[1] + 1,
                         max(x - 1, 0):x + brick[0] + 1].sum()
                     for z in range(0, nz, brick[2]) for y in range(0, ny, brick[1]) for x in range(0, nx, brick[0])])


@pytest.mark.parametrize("brick", SHAPES, ids=["x".join(map(str, b)) for b in SHAPES])
def test_crowded_bricks(brick):
    """2.2 times the lattice density: with the default shape every brick is
    beyond the LDS capacity (3760 particles), some cut into runs of rows, some
    beyond what is cut (4800); the smaller shapes mix whole and cut bricks."""
    sc = S.random_cloud(n=17500, box=(0.4, 0.4, 0.4), dp=0.02, seed=21, boundary_frac=0.2, u_sigma=0.2)
    t = _brick_totals(sc, brick)
    if brick == (3, 4, 3):
        assert t.min() > 3760 and (t <= 4800).any() and (t > 4800).any(), t
    sim = make_sim(sc, max_neibs=416, brick=brick)
    sim.build()
    a = sim.forces(bricks=True).clone()
    b = sim.forces(bricks=True).clone()
    torch_sync()
    assert torch.equal(a, b)
    ob = compare_build(sc, sim, max_neibs=416)
    _, (acc, drho, sa, sd, _ni) = oracle_forces_of(sc, ob)
    check_forces(a[: sc.n].cpu().numpy(), acc, drho, sa, sd, label="crowded")


@pytest.mark.parametrize("brick", SHAPES, ids=["x".join(map(str, b)) for b in SHAPES])
@pytest.mark.parametrize("n", [1, 2, 9, 65, 700, 2100])
def test_few_bricks(n, brick):
    """One to a few bricks, so that each is cut into its rows; the lists run
    from empty ones over the edges of a run of eight (n = 9) to full ones."""
    box = (0.12, 0.12, 0.12) if n < 100 else (0.2, 0.27, 0.16)
    sc = S.random_cloud(n=n, box=box, dp=0.02, seed=300 + n, boundary_frac=0.2, u_sigma=0.2)
    log("case few bricks n=%d" % n)
    sim = make_sim(sc, max_neibs=256, brick=brick, capacity=n + 3)
    sim.build()
    sim.forces_n.fill_(float("nan"))
    f = sim.forces(bricks=True).clone()
    torch_sync()
    assert torch.isnan(f[n:]).all(), "rows past n written"
    ob = compare_build(sc, sim, max_neibs=256)
    _, (acc, drho, sa, sd, _ni) = oracle_forces_of(sc, ob)
    check_forces(f[:n].cpu().numpy(), acc, drho, sa, sd, label="few bricks %d" % n, allowance=edge_allowance(sc, ob))


@pytest.mark.parametrize("side,brick", [(1.1, (3, 2, 3)), (1.3, (3, 4, 3))], ids=["3x2x3", "3x4x3"])
def test_rounds_of_bricks(side, brick):
    """Somewhat more bricks than workgroups, so that those left over by the
    whole round are cut, and dealt out: every particle's derivatives, and the
    adjoint's parameter sums."""
    from test_gpu_adjoint import _backward_parity
    box = (side, side, 0.8 * side)
    n = int(9000 * side ** 3 * 4)
    sc = S.random_cloud(n=n, box=box, dp=0.02, seed=int(100 * side), boundary_frac=0.1, u_sigma=0.2, alpha=0.2)
    nb = int(np.prod([-(-int(c) // b) for c, b in zip(sc.grid.ncell, brick)]))
    log("case rounds: n=%d, %d bricks of %s" % (n, nb, brick))
    sim = make_sim(sc, max_neibs=96, brick=brick)
    sim.build()
    sim.forces_n.fill_(float("nan"))
    f = sim.forces(bricks=True).clone()
    torch_sync()
    ob = compare_build(sc, sim, max_neibs=96)
    _, (acc, drho, sa, sd, _ni) = oracle_forces_of(sc, ob)
    check_forces(f[:n].cpu().numpy(), acc, drho, sa, sd, label="rounds", allowance=edge_allowance(sc, ob))
    _backward_parity(sc, 96, True, brick, "rounds")


@pytest.mark.parametrize("brick", SHAPES, ids=["x".join(map(str, b)) for b in SHAPES])
def test_crowded_bricks_adjoint(brick):
    """The adjoint on the crowded cloud (its LDS holds fewer particles, so
    more bricks are cut or left to the global lists), parameter sums included;
    its own checks repeat the call bit for bit."""
    from test_gpu_adjoint import _backward_parity
    sc = S.random_cloud(n=17500, box=(0.4, 0.4, 0.4), dp=0.02, seed=21, boundary_frac=0.2, u_sigma=0.2, alpha=0.2)
    _backward_parity(sc, 416, True, brick, "crowded")


@pytest.mark.parametrize("n", [2, 65, 700])
def test_few_bricks_adjoint(n):
    from test_gpu_adjoint import _backward_parity
    box = (0.12, 0.12, 0.12) if n < 100 else (0.2, 0.27, 0.16)
    sc = S.random_cloud(n=n, box=box, dp=0.02, seed=300 + n, boundary_frac=0.2, u_sigma=0.2, alpha=0.2)
    _backward_parity(sc, 256, True, None, "few bricks %d" % n)


def test_adjoint_same_after_every_build():
    """The table of bricks, and with it the order in which the parameter
    partials are summed, is the same after every build of a state."""
    from paper_2207_11328_amd import abi
    sc = S.dam_break_64k()
    got = []
    for _ in range(2):
        sim = make_sim(sc)
        for _ in range(2):
            sim.build()
            gf = torch.sin(torch.arange(4 * sim.capacity, device=sim.device, dtype=torch.float32)).view(-1, 4)
            gp, gv = torch.zeros_like(sim.pos), torch.zeros_like(sim.vel)
            par = torch.zeros(3, dtype=torch.float64, device=sim.device)
            ws = torch.zeros(abi.sph_forces_backward_workspace_bytes(sim.capacity, sim.n_cells), dtype=torch.uint8,
                             device=sim.device)
            abi.sph_forces_backward(sim.g, sim.p, sim.parts, sim.neibs, sim.neib_count, sim.max_neibs, gf, gp, gv,
                                    par, False, ws, None, *sim.brick_args())
            torch_sync()
            got.append((gp, gv, par))
    for g in got[1:]:
        assert all(torch.equal(a, b) for a, b in zip(got[0], g))


@pytest.mark.parametrize("visc", [0, 1], ids=["av", "morris"])
def test_small_scale_adjoint(visc):
    """Spacing 0.1 mm, no walls.  The first staged particle of the corner brick
    is one of its centrals, and the slots past the end of its list point to
    itself (r = 0), where the kernel's second factor, F'/r, is beyond float32
    before its mask: such a slot has to add nothing."""
    import dataclasses
    from oracle import oracle as O
    from test_gpu_adjoint import _backward_parity
    sc = S.random_cloud(n=1100, box=(0.0013, 0.001, 0.001), dp=1e-4, seed=51, boundary_frac=0.0, u_sigma=0.3,
                        rho_sigma=0.01, alpha=0.3)
    sc = dataclasses.replace(sc, params=dataclasses.replace(sc.params, visc_model=visc, nu=1e-6 if visc else 0.0))
    L = O.build_f32(sc.grid, sc.params, sc.cell, sc.pos, sc.vel, sc.info)["lists"]
    assert (L.nf[0] + L.nb[0]) % 8, "no slot past the list"
    _backward_parity(sc, 192, True, None, "small scale")


@pytest.mark.parametrize("brick", SHAPES, ids=["x".join(map(str, b)) for b in SHAPES])
@pytest.mark.parametrize("M", [1, 8, 40])
def test_short_lists(M, brick):
    """Lists of fewer groups of eight than a central's lanes request ahead, where
    an item has no table of centrals: rows without a list, and (the crowd in one
    corner, beyond what is staged) rows on the gather path.  Both forms take
    the same kept entries; particles without one get zeros."""
    sparse = S.random_cloud(n=150, box=(0.6, 0.6, 0.6), dp=0.02, seed=33, boundary_frac=0.0, u_sigma=0.2)
    crowd = S.random_cloud(n=6000, box=(0.6, 0.6, 0.6), dp=0.02, seed=34, boundary_frac=0.0, u_sigma=0.2)
    crowd.cell[:] = crowd.cell % 3 + 10 * (crowd.cell // 10 % 3) + 100 * (crowd.cell // 100 % 3)
    assert tuple(sparse.grid.ncell) == (10, 10, 10)
    for sc in (sparse, crowd):
        log("case short lists M=%d n=%d" % (M, sc.n))
        sim = make_sim(sc, max_neibs=M, brick=brick, capacity=sc.n)
        sim.build()
        sim.forces_n.fill_(float("nan"))
        b = sim.forces(bricks=True).clone()
        g = sim.forces(bricks=False).clone()
        torch_sync()
        cnt = sim.neib_count[: sc.n].cpu().numpy()
        assert torch.isfinite(b).all() and (b[: sc.n].cpu().numpy()[cnt == 0] == 0).all()
        scale = g.abs().amax(dim=0)
        if sc is crowd:
            assert (cnt == M).all() and _brick_totals(sc, brick).max() > 4800
            assert torch.equal(b, g)
        else:
            assert (cnt == 0).any() and (cnt > 0).any()
            assert ((b - g).abs() <= 1e-5 * scale).all(), (b - g).abs().max(dim=0)


def test_lists_around_255():
    """Lists on both sides of the length that no longer fits an entry of the
    table of centrals, in items that are staged."""
    sc = S.random_cloud(n=640, box=(0.12, 0.12, 0.12), dp=0.02, seed=77, boundary_frac=0.1, u_sigma=0.2)
    sim = make_sim(sc, max_neibs=512)
    sim.build()
    f = sim.forces(bricks=True).clone()
    torch_sync()
    cnt = sim.neib_count[: sc.n].cpu().numpy().view(np.uint32)
    cnt = (cnt & 0xFFFF) + (cnt >> 16)
    log("case long lists: n=%d, lists of %d to %d" % (sc.n, cnt.min(), cnt.max()))
    assert np.isin([254, 255, 256], cnt).any() and cnt.min() < 200 and 256 < cnt.max() <= 512
    ob = compare_build(sc, sim, max_neibs=512)
    _, (acc, drho, sa, sd, _ni) = oracle_forces_of(sc, ob)
    check_forces(f[: sc.n].cpu().numpy(), acc, drho, sa, sd, label="long lists")


def test_the_largest_whole_brick():
    """15 x 17 x 15 lattice places in the halo of a brick (the most at 1.3
    spacings per smoothing length, but for one alignment): within three of
    what is staged whole."""
    dp, m = 0.02, (24, 29, 24)
    p = S.sph_params(dp)
    grid = S.make_grid((0.0,) * 3, tuple(k * dp for k in m), p.r_search)
    i = np.stack(np.meshgrid(*[np.arange(k) for k in m], indexing="ij"), -1).reshape(-1, 3)
    cell, off = S.encode_positions(grid, (i + 0.5) * dp)
    n = len(i)
    rng = np.random.default_rng(4)
    pos = np.zeros((n, 4), np.float32)
    pos[:, :3] = off
    pos[:, 3] = 1000.0 * dp ** 3
    vel = rng.normal(0.0, 0.2, (n, 4)).astype(np.float32)
    vel[:, 3] = 1000.0 * (1 + rng.normal(0.0, 3e-3, n))
    sc = S.Scene("lattice", grid, p, cell, pos, vel, np.arange(n, dtype=np.uint32), n, 0)
    assert _brick_totals(sc, (3, 4, 3)).max() == 3825
    log("case largest brick: n=%d" % n)
    sim = make_sim(sc)
    sim.build()
    f = sim.forces(bricks=True).clone()
    torch_sync()
    ob = compare_build(sc, sim)
    _, (acc, drho, sa, sd, _ni) = oracle_forces_of(sc, ob)
    check_forces(f[:n].cpu().numpy(), acc, drho, sa, sd, label="largest brick")


def _layers(sizes, brick, dp=0.02, per_cell=8, seed=1):
    """A row of bricks along x, brick k with every inner cell filled for
    sizes[k] = 1 and only one layer of cells along y for sizes[k] = 0."""
    p = S.sph_params(dp)
    cs = np.float32(p.r_search)
    nx = brick[0] * len(sizes)
    grid = S.Grid(origin=np.zeros(3), cell_size=np.array([cs] * 3), ncell=np.array([nx, brick[1], brick[2]], np.int32))
    x, y, z = np.meshgrid(np.arange(nx), np.arange(brick[1]), np.arange(brick[2]), indexing="ij")
    full = np.asarray(sizes, bool)[x // brick[0]] | (y == 0)
    lin = (x + nx * (y + brick[1] * z))[full]
    cell = np.repeat(lin, per_cell).astype(np.int32)
    n = cell.size
    rng = np.random.default_rng(seed)
    pos = np.zeros((n, 4), np.float32)
    pos[:, :3] = rng.uniform(-0.49, 0.49, (n, 3)) * cs
    pos[:, 3] = 1000.0 * float(cs) ** 3 / per_cell
    vel = rng.normal(0.0, 0.2, (n, 4)).astype(np.float32)
    vel[:, 3] = 1000.0 * (1 + rng.normal(0.0, 3e-3, n))
    info = (np.arange(n) | ((rng.random(n) < 0.1).astype(np.int64) << 30)).astype(np.uint32)
    return S.Scene("layers", grid, p, cell, pos, vel, info, int((info >> 30 == 0).sum()), int((info >> 30 == 1).sum()))


# bricks, every how manyth is light (0: none), particles per filled cell (13: heavy)
ROUNDS = [(300, 0, 13), (300, 0, 8), (400, 3, 13), (430, 4, 13), (520, 0, 13), (560, 5, 13), (700, 0, 13), (800, 2, 13)]


@pytest.mark.parametrize("brick", SHAPES, ids=["x".join(map(str, b)) for b in SHAPES])
@pytest.mark.parametrize("bricks,every,per_cell", ROUNDS)
def test_rounds_of_heavy_and_light_bricks(bricks, every, per_cell, brick):
    """One to three rounds of bricks, heavy and light ones, on each side of the
    lines of the split: every particle's derivatives and adjoint against the
    gather forms, which have no items, and the parameter sums."""
    from paper_2207_11328_amd import abi
    sc = _layers([0 if every and k % every == 0 else 1 for k in range(bricks)], brick, per_cell=per_cell)
    log("case rounds of %d bricks %s: n=%d" % (bricks, brick, sc.n))
    sim = make_sim(sc, max_neibs=192, brick=brick)
    sim.build()
    assert sim.status_host()["overflow"] == 0
    cap, E = sim.capacity, -(-sim.capacity // 64) * 512 * 24
    t = sim.neibs_brick[E:].view(torch.int32)
    assert int(t[0]) + int(t[cap + 1]) == bricks and (per_cell < 12 or int(t[cap + 1]) == (-(-bricks // every) if every else 0))
    gf = torch.sin(torch.arange(4 * cap, device=sim.device, dtype=torch.float32)).view(-1, 4)
    got = []
    for b in (True, False):
        sim.forces_n.fill_(float("nan"))
        f = sim.forces(bricks=b).clone()
        gp, gv = torch.full_like(sim.pos, float("nan")), torch.full_like(sim.pos, float("nan"))
        par = torch.zeros(3, dtype=torch.float64, device=sim.device)
        ws = torch.zeros(abi.sph_forces_backward_workspace_bytes(cap, sim.n_cells), dtype=torch.uint8, device=sim.device)
        abi.sph_forces_backward(sim.g, sim.p, sim.parts, sim.neibs, sim.neib_count, sim.max_neibs, gf, gp, gv, par,
                                False, ws, None, *sim.brick_args(b))
        torch_sync()
        got.append((f[: sc.n], gp[: sc.n, :3], gv[: sc.n], par))
    # a particle without its item, or with a part of its sum twice, is off by
    # the size of its terms; the two forms differ by rounding
    for a, b in zip(*got):
        scale = b.abs().amax(dim=0)
        assert torch.isfinite(a).all() and ((a - b).abs() <= 1e-4 * scale).all(), ((a - b).abs() / scale).amax()
