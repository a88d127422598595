"""The matrix form of the list build where it can go wrong: cells at the edges
of a group of 16 centrals, more candidates than a list page (640), more
neighbours than a window of entries (128), lists cut in the middle of a window
or a group of eight, walls.  Lists against the oracle's float32 build: they
are whole numbers and have to be the same."""
import numpy as np
import pytest

from workloads import scenes as S

from parity import check_forces, compare_build, log, make_sim, oracle_forces_of, torch_sync

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

# n, box side, wall share, max_neibs; the particles of a cell, of its neighbourhood
SCENES = [
    (2000, 0.3, 0.0, 160),    # 6 to 28: one page
    (2000, 0.3, 0.3, 160),    # with walls
    (4100, 0.3, 0.0, 256),    # 19 to 51, to 1000: two pages of a plain list
    (4100, 0.3, 0.4, 256),    # two pages with walls
    (4100, 0.3, 0.2, 37),     # cut within a page
    (4100, 0.3, 0.0, 150),    # cut in the second page
    (600, 0.12, 0.0, 352),    # 68 to 84, 600: one page, windows of a plain list
    (600, 0.12, 0.3, 352),    # windows with walls
    (600, 0.12, 0.0, 133),    # cut within the second window
    (1500, 0.12, 0.3, 900),   # 165 to 202, 1500: three pages, seven windows
]


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def _rows(entries, n, M):
    """The brick-local lists, one row per particle."""
    e = entries.view(torch.int16).reshape(-1, -(-M // 8), 64, 8)
    return e.permute(0, 2, 1, 3).reshape(-1, 8 * -(-M // 8))[:n].cpu().numpy()


@pytest.mark.parametrize("brick", [(3, 4, 3), (3, 2, 3)], ids=["3x4x3", "3x2x3"])
@pytest.mark.parametrize("n,side,walls,M", SCENES)
def test_lists(n, side, walls, M, brick):
    sc = S.random_cloud(n=n, box=(side, side, side), dp=0.02, seed=500 + n, boundary_frac=walls, u_sigma=0.1)
    counts = np.bincount(sc.cell, minlength=int(np.prod(sc.grid.ncell)))
    log("case lists n=%d M=%d walls=%g cells of %d to %d" % (n, M, walls, counts.min(), counts.max()))
    sim = make_sim(sc, max_neibs=M, brick=brick, capacity=n + 5)
    sim.neibs_brick.view(torch.uint8).fill_(0xA5)
    sim.build()
    ob = compare_build(sc, sim, max_neibs=M)
    entries = -(-sim.capacity // 64) * 64 * 8 * -(-M // 8)
    first = sim.neibs_brick[:entries].clone()
    if sim.status_host()["overflow"] == 0 and M <= 416:
        f = sim.forces(bricks=True).clone()
        torch_sync()
        _, (acc, drho, sa, sd, _ni) = oracle_forces_of(sc, ob)
        check_forces(f[: sc.n].cpu().numpy(), acc, drho, sa, sd, label="lists")
    # the entries and the rest of their last group are the same bytes whatever
    # the array held
    other = make_sim(sc, max_neibs=M, brick=brick, capacity=n + 5)
    other.neibs_brick.view(torch.uint8).fill_(0x5A)
    other.build()
    torch_sync()
    a, b = _rows(first, n, M), _rows(other.neibs_brick[:entries], n, M)
    cnt = sim.neib_count[:n].cpu().numpy().view(np.uint32).astype(np.int64)
    kept = ((cnt & 0xFFFF) + (cnt >> 16))[:, None]
    at = np.arange(a.shape[1])[None, :]
    written = at < -(-kept // 8) * 8
    assert (a == b)[written].all()
    assert (a[written & (at >= kept)] == 0).all()


def test_last_particle_of_the_largest_capacity():
    """The particle of index 2^26 - 1, seen from the cell below it along every
    axis: index and image fields of the entry have all bits set."""
    from paper_2207_11328_amd import abi
    dev = torch.device("cuda")
    n, M, per_cell = abi.MAX_CAPACITY, 8, 4
    ncell = (256, 512, 128)
    grid = S.Grid(origin=np.zeros(3), cell_size=np.ones(3, np.float32), ncell=np.array(ncell, np.int32))
    assert grid.n_cells * per_cell == n
    params = S.Params(dp=0.05, h=0.09, r_search=0.2)
    log("case last particle: n=%d, %d cells" % (n, grid.n_cells))
    ids = torch.arange(n, dtype=torch.int32, device=dev)
    cell = ids // per_cell
    pos = torch.zeros((n, 4), device=dev)
    pos[:, 3] = 1.0
    vel = torch.zeros((n, 4), device=dev)
    vel[:, 3] = 1000.0
    # four coincident particles a cell, but one of the last cell at its lower
    # corner and one of the cell diagonally below at its upper corner
    below = (ncell[0] - 2) + ncell[0] * ((ncell[1] - 2) + ncell[1] * (ncell[2] - 2))
    i = below * per_cell
    pos[n - 1, :3] = -0.45
    pos[i, :3] = 0.45
    neibs = torch.zeros(abi.sph_neib_list_entries(n, M), dtype=torch.int32, device=dev)
    brick = torch.zeros(abi.sph_neib_brick_entries(n, M), dtype=torch.int16, device=dev)
    count = torch.zeros(n, dtype=torch.int32, device=dev)
    ranges = torch.zeros((2, grid.n_cells), dtype=torch.int32, device=dev)
    status = torch.zeros(abi.STATUS_WORDS, dtype=torch.int32, device=dev)
    ws = torch.zeros(abi.sph_build_workspace_bytes(n, grid.n_cells), dtype=torch.uint8, device=dev)
    abi.sph_build_neighbors(abi.grid_struct(grid), abi.params_struct(params),
                            abi.particles_struct(n, cell, pos, vel, ids), neibs, count, M, ranges[0], ranges[1],
                            status, ws, None, None, brick)
    torch_sync()
    assert status[:4].tolist() == [n, per_cell - 1, 0, 0]

    def listed(k):
        c = int(count[k])
        assert c >> 16 == 0
        return [int(neibs[(k // 64) * 64 * M + 64 * e + k % 64]) & 0xFFFFFFFF for e in range(c)]

    assert listed(i) == [0xFFFFFFFF]
    assert listed(n - 1) == [i | 0b010101 << 26]
    assert int((count == per_cell - 1).sum()) == n - 2 * per_cell
    assert int((count == per_cell - 2).sum()) == 2 * (per_cell - 1)


def test_slots_beyond_16_bits():
    """A brick whose halo holds more than 65535 particles: the brick-local
    entries saturate, as the layout says."""
    rng = np.random.default_rng(8)
    sc = S.random_cloud(n=66600, box=(0.29, 0.29, 0.29), dp=0.02, seed=8, boundary_frac=0.0, u_sigma=0.1)
    nx, ny, nz = (int(v) for v in sc.grid.ncell)
    assert (nx, ny, nz) == (5, 5, 5)
    # all but 600 into the cells y = 0, x and z up to 3 (staged by brick 0); the others
    # into the cells y = 2, x and z up to 2, of the same brick
    crowd = 66000
    x, z = rng.integers(0, 4, crowd), rng.integers(0, 4, crowd)
    sc.cell[:crowd] = x + nx * (ny * z)
    x, z = rng.integers(0, 3, sc.n - crowd), rng.integers(0, 3, sc.n - crowd)
    sc.cell[crowd:] = x + nx * (2 + ny * z)
    log("case 16-bit slots: n=%d" % sc.n)
    sim = make_sim(sc, max_neibs=96, brick=(3, 3, 3))
    sim.build()
    torch_sync()
    cell = sim.cell[: sc.n].cpu().numpy()
    mine = (cell // nx) % ny == 2
    cnt = sim.neib_count[: sc.n].cpu().numpy().view(np.uint32)[mine]
    assert mine.sum() == 600 and (cnt > 0).all()
    e = _rows(sim.neibs_brick[: -(-sim.capacity // 64) * 64 * 96], sc.n, 96)[mine].view(np.uint16)
    assert (e[np.arange(96)[None, :] < cnt[:, None]] == 65535).all()


@pytest.mark.parametrize("scale", [2.0 ** 56, 2.0 ** -30])
def test_lists_at_any_scale(scale):
    """Lengths times a power of two: the same lists, bit for bit."""
    sc = S.random_cloud(n=2000, box=(0.3, 0.3, 0.3), dp=0.02, seed=5, boundary_frac=0.3, u_sigma=0.1)
    import dataclasses
    log("case scale %g" % scale)
    got = []
    for f in (1.0, scale):
        g, p = sc.grid, sc.params
        s = sc.copy()
        s.grid = dataclasses.replace(g, origin=g.origin * f, cell_size=(g.cell_size * np.float32(f)).astype(np.float32))
        s.params = dataclasses.replace(p, dp=p.dp * f, h=p.h * f, r_search=p.r_search * f)
        s.pos[:, :3] *= np.float32(f)
        sim = make_sim(s, max_neibs=160)
        sim.build()
        torch_sync()
        got.append((sim.neibs, sim.neib_count, sim.neibs_brick))
    for a, b in zip(*got):
        assert torch.equal(a, b)


@pytest.mark.parametrize("brick", [(3, 4, 3), (3, 2, 3)], ids=["3x4x3", "3x2x3"])
def test_table_of_many_bricks(brick):
    """A long thin grid of more bricks than the ordering blocks take one tile
    of each: the table holds the bricks with a pair by size class, large ones
    first, and by id in a class."""
    rng = np.random.default_rng(3)
    nx = 3 * 300000 - 1
    cells = rng.choice(nx, size=3000, replace=False)
    cell = np.repeat(cells, rng.integers(1, 80, size=cells.size)).astype(np.int32)
    n = cell.size
    p = S.sph_params(0.02)
    cs = np.float32(p.r_search)
    grid = S.Grid(origin=np.zeros(3), cell_size=np.array([cs, cs, cs]), ncell=np.array([nx, 1, 1], np.int32))
    pos = np.zeros((n, 4), np.float32)
    pos[:, :3] = rng.uniform(-0.45, 0.45, (n, 3)) * cs
    pos[:, 3] = 8e-3
    vel = np.zeros((n, 4), np.float32)
    vel[:, 3] = 1000.0
    log("case table: n=%d, %d bricks" % (n, nx // 3 + 1))
    sc = S.Scene("thin", grid, p, cell, pos, vel, np.arange(n, dtype=np.uint32), n, 0)
    M = 256
    sim = make_sim(sc, max_neibs=M, brick=brick)
    sim.build()
    torch_sync()
    bid = sim.cell[:n].cpu().numpy() // 3
    listed = np.unique(bid[sim.neib_count[:n].cpu().numpy() > 0])
    size = np.bincount(bid, minlength=listed.max() + 1)[listed]
    width = 12 * brick[0] * brick[1] * brick[2] // 27
    key = np.minimum(size // width, 62)
    order = listed[np.lexsort((listed, -key))]
    heavy = int((key >= 27).sum())
    t = sim.neibs_brick[-(-sim.capacity // 64) * 512 * (M // 8):].view(torch.int32).cpu().numpy()
    cap = sim.capacity
    nh, nl = int(t[0]), int(t[cap + 1])
    got = np.concatenate([t[1:1 + nh], t[cap + 1 - nl:cap + 1][::-1]])
    assert nh == heavy and nh + nl == order.size
    assert np.array_equal(got, order)
