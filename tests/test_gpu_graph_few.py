"""Graphs of few general nodes, whose pairs are all listed in order, and of more, which are ranked
against a sampled threshold in spans that depend on the node count: the oracle's graph at the edges of the
workgroups (256 nodes j, 8 nodes i; 512 nodes i), with surface nodes and without, couplings that are
zero, equal or infinite; and the refusal of bad inputs, checked on the host where nodes are few."""
import sys

import numpy as np
import pytest

import oracle
from paper_2503_16037_amd import scenes

pytestmark = pytest.mark.gpu

FX = scenes.FX


def say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


@pytest.fixture(scope="module")
def ctx():
    from paper_2503_16037_amd import sgrt
    c = sgrt.Context(0)
    yield c
    c.close()


def scattered(n, seed=3, surface=False, zero=0.0, twins=0, dims=(9, 7, 5)):
    """n general nodes anywhere in the box; a share of the voxels scatters nothing, and the first `twins`
    nodes come twice."""
    nx, ny, nz = dims
    sc = scenes.make_random_small(seed, nx=nx, ny=ny, nz=nz, surface=surface)
    rng = np.random.default_rng(seed + n)
    pos = np.stack([rng.integers(1, w * FX, n) for w in dims], 1).astype(np.int32)
    pos[n - twins:] = pos[:twins]
    mu = sc.mu_s.copy()
    mu[rng.random(mu.shape) < zero] = 0.0
    return sc.with_(node_pos_fx=pos, mu_s=mu, los_ptr=np.zeros(nx * ny + 1, np.int64), los_node=np.zeros(0, np.int32),
                    los_t=np.zeros(0))


def same(ctx, sc, **kw):
    from paper_2503_16037_amd import sgrt
    ap, ai = sgrt.graph_build(ctx, sc, **kw)
    oap, oai = oracle.coupling_graph(sc, **kw)
    assert np.array_equal(ap, oap) and np.array_equal(ai, oai), kw
    return len(ai)


@pytest.mark.parametrize("surface", [False, True])
@pytest.mark.parametrize("n", [1, 2, 7, 8, 9, 255, 256, 257, 513, 800, 4000])
def test_few_nodes(ctx, n, surface):
    sc = scattered(n, surface=surface)
    say("few nodes", n, surface)
    for n_pairs in (1, n, 7 * n, n * n):
        same(ctx, sc, n_pairs=n_pairs)
    same(ctx, sc, c_min=0.0)
    same(ctx, sc, c_min=0.02)


@pytest.mark.parametrize("zero, twins", [(0.9, 0), (0.0, 60), (1.0, 0)])
def test_zero_and_infinite_couplings(ctx, zero, twins):
    sc = scattered(700, zero=zero, twins=twins)
    if zero == 1.0:
        sc = sc.with_(mu_s=np.zeros_like(sc.mu_s))
    for n_pairs in (10, 60, 5000, 10 ** 6):
        same(ctx, sc, n_pairs=n_pairs)


@pytest.mark.parametrize("n", [4200, 5119, 9001])
def test_more_nodes_than_are_listed(ctx, n):
    sc = scattered(n, surface=True, dims=(24, 20, 12))
    for kw in (dict(n_pairs=1), dict(n_pairs=777), dict(n_pairs=40 * n), dict(c_min=0.3)):
        say("spans", n, kw, same(ctx, sc, **kw) // 2)


def test_equal_couplings_of_a_voxel_grid(ctx):
    sc = scenes.make_random_small(2, nx=9, ny=8, nz=7)
    sc = sc.with_(vol_pos_fx=scenes.jittered_positions(np.random.default_rng(0), 9, 8, 7, jitter=0.0),
                  mu_s=np.full_like(sc.mu_s, 0.01))
    for kw in (dict(n_pairs=1), dict(n_pairs=700), dict(n_pairs=10 ** 6), dict(c_min=0.02)):
        same(ctx, sc, **kw)


@pytest.mark.parametrize("big", [False, True])
@pytest.mark.parametrize("what, message", [("mu", "mu_s"), ("nan", "mu_s"), ("inf", "mu_s"), ("albedo", "surf_albedo"),
                                           ("outside", "outside the box (node 5)"), ("ground", "outside the box (node 5)"),
                                           ("voxel", "inside its voxel (node 5)")])
def test_bad_inputs_are_refused(ctx, what, message, big):
    from paper_2503_16037_amd import sgrt
    dims = (24, 20, 12) if big else (9, 7, 5)
    sc = scattered(5000 if big else 40, surface=True, dims=dims)
    if what in ("mu", "nan", "inf"):
        mu = sc.mu_s.copy()
        mu[2, 3, 4] = {"mu": -0.5, "nan": np.nan, "inf": np.inf}[what]
        sc = sc.with_(mu_s=mu)
    elif what == "albedo":
        alb = sc.surf_albedo.copy()
        alb[1, 1] = 1.5
        sc = sc.with_(surf_albedo=alb)
    elif what == "voxel":
        pos = sc.vol_pos_fx.copy().reshape(-1, 3)
        pos[5, 0] = 0
        sc = sc.with_(node_pos_fx=None, vol_pos_fx=pos)
    else:
        pos = sc.node_pos_fx.copy()
        pos[5] = [FX, FX, 0] if what == "ground" else [dims[0] * FX, 5, 5]
        pos[6, 2] = -1
        sc = sc.with_(node_pos_fx=pos)
    with pytest.raises(sgrt.SgError) as e:
        sgrt.graph_build(ctx, sc, n_pairs=20)
    assert e.value.status == sgrt.SG_E_INVALID and message in str(e.value)
