"""CIC deposit by tiles of 8^3 points: ragged and tiny grids, clouds over tile edges and
corners, the workgroup tables' overflow, and counts of more than one pass, against the
oracle (relative to the largest value; sums of at most a few thousand terms: 1e-12)."""
import numpy as np
import pytest

import oracle as O
from paper_1905_08890_amd import grmg, synth

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

PRM = dict(a=0.7, omega_m=synth.OMEGA_M, c_tilde=synth.C_TILDE)


def _check(n, pos, seed):
    rng = np.random.default_rng(seed)
    u = 1e-2 * rng.standard_normal(pos.shape)
    psi = 10.0 * rng.standard_normal((n, n, n))
    mass = 1.0 / max(1, len(pos))
    g = grmg.Grid(n, **PRM)
    g.set_field("Psi", psi)
    ref = O.cic_deposit(n, pos, u, mass, psi=psi, prm=O.params(**PRM))
    for _ in range(2):
        g.deposit_sources(pos, u, mass)
        for name, r in zip(("s0", "sx", "sy", "sz", "sm"), ref):
            d = np.abs(g.get_field(name).cpu().numpy() - r).max()
            assert d <= 1e-12 * np.abs(r).max(), (name, d)


@pytest.mark.parametrize("n,count", [(2, 700), (4, 3), (8, 1), (8, 600), (10, 999), (12, 5000), (20, 4097), (24, 30000),
                                     (16, 150000), (2, 70000)])
def test_counts_and_sides(n, count):
    """Sides that 8 divides and does not; the last two counts need several passes."""
    print(f"[gpu] deposit n={n} count={count}", flush=True)
    _check(n, np.random.default_rng(n + count).uniform(-0.5, 1.5, (count, 3)), n)


@pytest.mark.parametrize("n", [8, 16, 40, 160])
def test_clouds_over_tile_corners(n):
    """Every cloud over eight tiles where the grid has them; at 160^3 (8000 tiles, corners in
    random order) a workgroup reaches more tiles than its table holds."""
    print(f"[gpu] deposit corners n={n}", flush=True)
    rng = np.random.default_rng(n)
    corner = 8 * rng.integers(0, n // 8, (20000, 3))
    _check(n, (corner + rng.uniform(-0.45, 0.45, corner.shape)) / n, n)


def test_one_dense_lump():
    """Most particles in one tile."""
    n = 32
    print("[gpu] deposit lump", flush=True)
    rng = np.random.default_rng(3)
    pos = rng.uniform(0, 1, (8000, 3))
    pos[:6000] = 0.3 + 0.01 * rng.standard_normal((6000, 3))
    _check(n, pos, 3)


@pytest.mark.parametrize("n", [8, 16, 32])
@pytest.mark.parametrize("c_tilde", [49.0, 2997.92458 / 256.0, 1.5])
def test_lattice_at_rest_gives_exactly_one(n, c_tilde):
    """A particle of mass n^-3 at rest at every cell centre: every factor of s0 =
    m W / (c h^3) with W = c is exact, so s0 is 1 and the other sources 0, to the bit."""
    print(f"[gpu] deposit, lattice at rest n={n} c={c_tilde}", flush=True)
    g = grmg.Grid(n, a=1.0, omega_m=0.3, c_tilde=c_tilde)
    x = (np.arange(n) + 0.5) / n
    pos = np.stack([a.ravel() for a in np.meshgrid(x, x, x, indexing="ij")], axis=1)
    g.deposit_sources(pos, np.zeros_like(pos), 1.0 / n ** 3)
    for name, want in zip(("s0", "sx", "sy", "sz", "sm"), (1.0, 0.0, 0.0, 0.0, 0.0)):
        assert np.all(g.get_field(name).cpu().numpy() == want), name


@pytest.mark.parametrize("n,nbytes", [(2, 148224), (8, 392960), (16, 2194176), (20, 4147200), (30, 13474816),
                                      (34, 19560448), (48, 55713280), (62, 117871360)])
def test_workspace_without_room_for_the_extras(n, nbytes):
    """Workspaces of the sizes that grids asked for before helper hierarchies below 64^3
    and long deposit passes on small grids: bound and used to the last byte, deposits in
    several passes, vector components in turn.  Solves are the same bit for bit, a smaller
    buffer is refused, and a larger one bound again brings the helpers back."""
    print(f"[gpu] small workspace n={n}", flush=True)
    h = grmg.create_grid(n, PRM["a"], PRM["omega_m"], PRM["c_tilde"])
    full = grmg.Grid(n, **PRM)
    try:
        assert nbytes <= grmg.workspace_bytes(h)
        guard = 4096
        ws = torch.full((nbytes + guard,), 0x5A, dtype=torch.uint8, device="cuda")
        stream = torch.cuda.current_stream().cuda_stream
        with pytest.raises(grmg.GrError):
            grmg.bind(h, ws[:nbytes * 3 // 4 // 256 * 256], stream)
        rng = np.random.default_rng(n)
        count = 5 * n ** 3 + 100
        pos = torch.tensor(rng.uniform(0, 1, (count, 3)), device="cuda")
        u = torch.tensor(1e-2 * rng.standard_normal((count, 3)), device="cuda")
        ref = O.cic_deposit(n, pos.cpu().numpy(), u.cpu().numpy(), 1.0 / count, prm=O.params(**PRM))
        for buf in (ws[:nbytes], torch.empty(grmg.workspace_bytes(h), dtype=torch.uint8, device="cuda"), ws[:nbytes]):
            grmg.bind(h, buf, stream)
            grmg.deposit_sources(h, pos, u, 1.0 / count)
            x = torch.empty((n, n, n), dtype=torch.float64, device="cuda")
            for k, name in enumerate(("s0", "sx", "sy", "sz", "sm")):
                grmg.get_field(h, grmg.FIELD_IDS[name], x, grmg.F64)
                assert float((x.cpu() - torch.tensor(ref[k])).abs().max()) <= 1e-12 * np.abs(ref[k]).max(), name
                full.set_field(name, x)
            grmg.solve_constraints(h, grmg.default_opts(rtol=0.0, max_cycles=2))
            full.solve_constraints(rtol=0.0, max_cycles=2)
            for f in range(10):
                grmg.get_field(h, f, x, grmg.F64)
                assert torch.equal(x, full.get_field(f)), f
        assert bool((ws[nbytes:] == 0x5A).all())
    finally:
        torch.cuda.synchronize()
        grmg.destroy_grid(h)


@pytest.mark.parametrize("corners", [False, True])
def test_hash_table_of_tiles(corners):
    """Above 32768 tiles (33^3 here) a workgroup counts its tiles in a hash table of 8192
    slots: particles in random order reach about 9800 tiles a workgroup, clouds over
    tile corners 30000, so entries without a slot count in memory in both."""
    n = 264
    print(f"[gpu] deposit hash table corners={corners}", flush=True)
    rng = np.random.default_rng(17)
    if corners:
        pos = (8 * rng.integers(0, n // 8, (20000, 3)) + rng.uniform(-0.45, 0.45, (20000, 3))) / n
    else:
        pos = rng.uniform(0.0, 1.0, (30000, 3))
    _check(n, pos, 17)


@pytest.mark.parametrize("n,count", [(2, 0), (2, 64001), (6, 255), (8, 0), (8, 256), (8, 512), (8, 6144), (8, 130001),
                                     (12, 4096), (12, 64000), (14, 70000), (16, 2047), (16, 64000), (16, 64001), (18, 40000),
                                     (24, 40000), (24, 65537), (32, 32768), (32, 61440), (32, 61441), (64, 65536),
                                     (64, 65537), (66, 5000)])
def test_chains_and_lists(n, count):
    """Chains instead of lists: one and several workgroups a tile, one and several passes,
    the largest counts and grids that take them and the next larger."""
    print(f"[gpu] deposit chains n={n} count={count}", flush=True)
    rng = np.random.default_rng(1000 * n + count)
    pos = rng.uniform(-0.5, 1.5, (count, 3))
    pos[: count // 3] = 0.4 + 0.02 * rng.standard_normal((count // 3, 3))   # a lump: long chains
    _check(n, pos, n)
