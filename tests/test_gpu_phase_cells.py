"""The phase cells' matrix screen at every edge of its tiles: node degrees round the multiples of
the registers and row tiles, lattice sizes round the multiples of the column tiles.  Every owner
is the FP64 scan's (SG_EXACT_CELLS gives the same matrix, source and sun cells bit for bit), and
K agrees with the FP64 oracle."""
import sys

import numpy as np
import pytest

import oracle
from paper_2503_16037_amd import scenes

pytestmark = pytest.mark.gpu

DEGREES = [1, 2, 3, 4, 5, 7, 8, 9, 12, 15, 16, 17, 20, 21, 23, 24, 25, 28, 29, 31, 32, 33, 40, 47, 48, 49, 56, 63, 64]


def say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


@pytest.fixture(scope="module")
def ctx():
    from paper_2503_16037_amd import sgrt
    c = sgrt.Context(0)
    yield c
    c.close()


def hub_scene(n_fib, most, centred=False, surface=True):
    """Volume nodes of every degree of DEGREES up to `most` (and their partners' odd ones); with
    centred, nodes at the voxel centres, where many dot products are equal."""
    rng = np.random.default_rng(n_fib)
    sc = scenes.make_random_small(5, nx=9, ny=8, nz=5, two_phase=True, kscale=0.5, surface=surface)
    if centred:
        sc = sc.with_(vol_pos_fx=scenes.jittered_positions(rng, 9, 8, 5, jitter=0.0))
    a, b = [], []
    hubs = [d for d in DEGREES if d <= most]
    others = np.arange(len(hubs), sc.n_nodes)
    for h, d in enumerate(hubs):
        a += [h] * d
        b += list(rng.choice(others, d, replace=False))
    ap, ai = scenes.adjacency_from_pairs(sc.n_nodes, np.array(a), np.array(b))
    sc = sc.with_(adj_ptr=ap, adj_idx=ai, n_fib=n_fib)
    assert list(np.diff(ap)[:len(hubs)]) == hubs
    return sc


@pytest.mark.parametrize("n_fib", [2, 7, 8, 9, 31, 32, 33, 40, 41, 63, 64, 72, 95, 100, 104, 105, 128])
@pytest.mark.parametrize("most, centred", [(64, False), (28, True)])
def test_screened_cells_are_exact(ctx, n_fib, most, centred):
    from paper_2503_16037_amd import sgrt
    sc = hub_scene(n_fib, most, centred)
    say("phase cells", n_fib, "lattice points, degrees up to", int(sc.degrees().max()))
    with sgrt.Scene(ctx, sc) as g:
        got = []
        for screen in (True, False):
            g.solve(precision="fp64", screen=screen, scatter_order=1)
            got.append((g.export_csr()[2], g.export_vector("source"), g.export_vector("qsun")))
        for x, y in zip(*got):
            assert np.array_equal(x, y)
    ora = oracle.run(sc, scatter_order=1)
    assert np.abs(got[0][0] - ora["val"]).max() <= 1e-12 * np.abs(ora["val"]).max()


def test_weights_of_a_direction_sum_to_one(ctx):
    """Every lattice point is given to exactly one out-edge: the sun's cells sum to 1."""
    from paper_2503_16037_amd import sgrt
    sc = hub_scene(100, 64)
    with sgrt.Scene(ctx, sc) as g:
        g.solve(scatter_order=1)
        q = g.export_vector("qsun")
    tail = np.repeat(np.arange(sc.n_nodes), sc.degrees())
    total = np.bincount(tail, q, minlength=sc.n_nodes)
    assert np.abs(total[sc.degrees() > 0] - 1.0).max() < 1e-6


@pytest.mark.parametrize("most", [8, 64, 300])
def test_zero_length_out_edges(ctx, most):
    """Coupled general nodes at one place: their direction is no number, and the FP64 sequence
    alone decides every cell of such a node."""
    from paper_2503_16037_amd import sgrt
    rng = np.random.default_rng(most)
    sc = scenes.make_random_small(5, nx=9, ny=8, nz=5, vza=30.0, vaa=200.0, kscale=0.5, surface=False)
    pos, lp, ln, lt = oracle.los_nodes(sc.nx, sc.ny, sc.nz, sc.view_dir, sc.voxel_m, "step", step_m=45.0)
    n = len(pos)
    pos[1::20] = pos[0::20][:len(pos[1::20])]
    a, b = [], []
    for h in range(0, n - 1, 20):
        others = np.setdiff1d(np.arange(n), [h, h + 1])
        a += [h] * most
        b += [h + 1, *rng.choice(others, most - 1, replace=False)]
    ap, ai = scenes.adjacency_from_pairs(n, np.array(a), np.array(b))
    say("zero-length out-edges, degree", most)
    with sgrt.Scene(ctx, scenes.with_los_nodes(sc, pos, lp, ln, lt).with_(adj_ptr=ap, adj_idx=ai)) as g:
        got = []
        for screen in (True, False):
            g.solve(screen=screen, scatter_order=1)
            got.append((g.export_csr()[2], g.export_vector("source"), g.export_vector("qsun")))
        for x, y in zip(*got):
            assert np.array_equal(x, y, equal_nan=True)


def dense_scene(hubs, n_fib, centred):
    """Nodes of the given degrees, above 64 and round the multiples of the row tiles (32), the
    wavefronts' sums (512), the FP64 scans (256) and the resident out-edges (1024); the last hub is
    a surface node."""
    rng = np.random.default_rng(n_fib)
    sc = scenes.make_random_small(6, nx=20, ny=18, nz=12, two_phase=True, kscale=0.3, surface=True)
    if centred:
        sc = sc.with_(vol_pos_fx=scenes.jittered_positions(rng, 20, 18, 12, jitter=0.0))
    nvol = sc.n_vol
    at = list(range(len(hubs) - 1)) + [nvol]
    a, b = [], []
    for h, d in zip(at, hubs):
        a += [h] * d
        b += list(rng.choice(np.arange(len(hubs), nvol), d, replace=False))
    ap, ai = scenes.adjacency_from_pairs(sc.n_nodes, np.array(a), np.array(b))
    assert [int(np.diff(ap)[h]) for h in at] == hubs
    return sc.with_(adj_ptr=ap, adj_idx=ai, n_fib=n_fib)


@pytest.mark.parametrize("hubs, n_fib, centred, against", [
    ([65, 66, 95, 96, 97, 127, 128, 129, 255, 256, 257, 70], 100, False, "oracle"),
    ([65, 511, 512, 513, 300], 100, True, "oracle"),
    ([64, 65, 1023, 1024, 1025, 900], 31, False, "oracle"),
    ([1056, 1055, 100], 128, True, "oracle"),
    ([300, 77, 65], 2, False, "oracle"),
    ([2049, 4096, 4095, 3000], 64, False, "scan"),
])
def test_cells_of_dense_nodes(ctx, hubs, n_fib, centred, against):
    from paper_2503_16037_amd import sgrt
    sc = dense_scene(hubs, n_fib, centred)
    say("dense nodes", hubs, n_fib, "lattice points")
    with sgrt.Scene(ctx, sc) as g:
        got = []
        for screen in (True, False):
            g.solve(precision="fp64", screen=screen, scatter_order=1)
            got.append((g.export_csr()[2], g.export_vector("source"), g.export_vector("qsun")))
        for x, y in zip(*got):
            assert np.array_equal(x, y)
    if against == "oracle":
        ora = oracle.run(sc, scatter_order=1)
        assert np.abs(got[0][0] - ora["val"]).max() <= 1e-12 * np.abs(ora["val"]).max()


@pytest.mark.parametrize("most", [5, 24, 40, 64])
def test_wavelength_tiles_at_every_degree(ctx, most):
    """The narrow wavelength tiles stage the cells' columns, the wide one whole blocks: nodes of
    every degree give the same bits in all of them, and the oracle's radiances."""
    from paper_2503_16037_amd import sgrt
    sc = hub_scene(33, most)
    sc = sc.with_(abs_scale=np.linspace(0.2, 3.0, 5).astype(np.float32))
    say("wavelength tiles, degrees up to", int(sc.degrees().max()))
    with sgrt.Scene(ctx, sc) as g:
        ref, info = g.solve(lambda_tile=64)
        phi = g.export_vector("phi")
        for tile in (8, 16, 32):
            rad, again = g.solve(lambda_tile=tile)
            assert np.array_equal(rad, ref) and np.array_equal(g.export_vector("phi"), phi)
            assert again["sweeps"] == info["sweeps"]
    for k in (0, 4):
        ora = oracle.run(sc, abs_scale=float(sc.abs_scale[k]))["radiance"]
        assert np.abs(ref[k] - ora).max() <= 1e-4 * np.abs(ora).max()


@pytest.mark.parametrize("n_fib", [2, 5, 8, 9, 31, 32, 33, 40, 41, 64, 72, 73, 100, 127, 128])
@pytest.mark.parametrize("most, centred", [(64, False), (28, True)])
def test_coloured_cells_are_exact(ctx, n_fib, most, centred):
    """The colouring's seeds through the screen and by the FP64 scan alone, and the oracle's cells."""
    from paper_2503_16037_amd import sgrt
    sc = hub_scene(n_fib, most, centred).with_(sigma_mode=1)
    say("coloured cells", n_fib, "lattice points")
    with sgrt.Scene(ctx, sc) as g:
        got = []
        for screen in (True, False):
            g.solve(precision="fp64", screen=screen, scatter_order=1)
            got.append((g.export_csr()[2], g.export_vector("source"), g.export_vector("qsun")))
        for x, y in zip(*got):
            assert np.array_equal(x, y)
    ora = oracle.run(sc, scatter_order=1)
    assert np.abs(got[0][0] - ora["val"]).max() <= 1e-12 * np.abs(ora["val"]).max()
