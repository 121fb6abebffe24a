"""Sweeps over the front against whole sweeps of the same scene, both asked for: every edge of phi,
the radiances and the number of sweeps are equal bit for bit.  Small scenes, where a wavefront's share
of the marks ends early or holds no node at all: one node, counts that are not multiples of 8, isolated
nodes, hubs above 64 couplings, periodic slabs, line-of-sight nodes; both precisions, every wavelength
tile; the same in the bounds-checked build."""
import os
import subprocess
import sys

import numpy as np
import pytest

import oracle
from paper_2503_16037_amd import scenes

pytestmark = pytest.mark.gpu
ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


@pytest.fixture(scope="module")
def ctx():
    from paper_2503_16037_amd import sgrt
    c = sgrt.Context(0)
    yield c
    c.close()


def small(nx, ny, nz, seed=1, surface=False, **kw):
    return scenes.make_random_small(seed, nx=nx, ny=ny, nz=nz, surface=surface, kscale=2.0, **kw)


def hubs(degrees, isolated=0):
    """Nodes of the given degrees among a radius graph's others, and `isolated` nodes without edges."""
    sc = scenes.make_random_small(5, nx=12, ny=11, nz=9, kscale=1.0)
    rng = np.random.default_rng(len(degrees))
    tail = np.repeat(np.arange(sc.n_nodes), sc.degrees())
    up = (tail < sc.adj_idx) & (tail >= isolated) & (sc.adj_idx >= isolated)
    a, b = [tail[up]], [sc.adj_idx[up]]
    for h, d in enumerate(degrees):
        a.append(np.full(d, isolated + h))
        b.append(rng.choice(np.arange(isolated + 50, sc.n_vol), d, replace=False))
    ap, ai = scenes.adjacency_from_pairs(sc.n_nodes, np.concatenate(a), np.concatenate(b))
    return sc.with_(adj_ptr=ap, adj_idx=ai)


def los():
    sc = small(6, 5, 4, vza=30.0, vaa=200.0)
    pos, lp, ln, lt = oracle.los_nodes(sc.nx, sc.ny, sc.nz, sc.view_dir, sc.voxel_m, "step", step_m=45.0)
    return scenes.with_los_nodes(sc, pos, lp, ln, lt, radius_vox=1.8)


SCENES = {
    "1": lambda: small(1, 1, 1, surface=True),
    "7": lambda: small(7, 1, 1),
    "9": lambda: small(3, 3, 1),
    "65": lambda: small(13, 5, 1),
    "surface": lambda: small(9, 8, 7, surface=True),
    "isolated": lambda: hubs([], isolated=37),
    "hubs": lambda: hubs([90, 300, 65, 64], isolated=3),
    "slab": lambda: scenes.make_slab(nx=11, ny=9, nz=5),
    "los": los,
}


def same_bits(sgrt, ctx, sc, variants, **opts):
    """The scene solved by whole sweeps and over the front: first solve, tuned and captured,
    replayed, and launch by launch."""
    with sgrt.Scene(ctx, sc) as g:
        ref, info = g.solve(front=False, **opts)
        phi = g.export_vector("phi")
        assert info["converged"] == 1 and np.all(np.isfinite(phi))
        for more in variants:
            rad, again = g.solve(front=True, **opts, **more)
            assert again["sweeps"] == info["sweeps"], more
            assert np.array_equal(rad, ref) and np.array_equal(g.export_vector("phi"), phi), more
    return info


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("what", list(SCENES))
def test_one_wavelength(ctx, what, precision):
    from paper_2503_16037_amd import sgrt
    sc = SCENES[what]()
    say("front bits", what, precision, sc.n_nodes)
    info = same_bits(sgrt, ctx, sc, ({}, {}, {}, dict(timing=True), dict(graphs=False, autotune=False)), precision=precision)
    if what in ("surface", "hubs", "slab", "los"):
        assert info["sweeps"] > 5, "no sweep over the front"


@pytest.mark.parametrize("n_lambda", [2, 8, 12, 16, 33, 70])
@pytest.mark.parametrize("what", ["7", "65", "surface", "isolated", "slab", "los"])
def test_wavelengths(ctx, what, n_lambda):
    from paper_2503_16037_amd import sgrt
    sc = SCENES[what]()
    sc = sc.with_(abs_scale=np.geomspace(0.2, 4.0, n_lambda).astype(np.float32))
    say("front bits", what, n_lambda, "wavelengths", sc.n_nodes)
    tiles = [dict(lambda_tile=t) for t in (8, 16, 64) if t >= n_lambda or t == 64]
    info = same_bits(sgrt, ctx, sc, [*tiles, *tiles, {}, {}, dict(timing=True)])
    if what in ("surface", "slab", "los"):
        assert info["sweeps"] > 6, "no sweep over the front"


@pytest.mark.parametrize("opts", [dict(precision="fp32"), dict(precision="fp64"), dict(n_lambda=12), dict(n_lambda=31)])
def test_more_nodes_than_resident_wavefronts(ctx, opts):
    """39,960 nodes: several rows of the front's stride, the last one ragged."""
    from paper_2503_16037_amd import sgrt
    opts = dict(opts)
    sc = scenes.make_cloud(seed=9, nx=45, ny=37, nz=23, n_lambda=opts.pop("n_lambda", 0))
    say("front bits", sc.name, opts, sc.n_lambda)
    assert same_bits(sgrt, ctx, sc, ({}, {}), **opts)["sweeps"] > 6


@pytest.mark.timeout(300)
def test_in_the_checked_build():
    child = ("import sys; sys.path[:0] = [%r, %r]\n" % (ROOT, os.path.join(ROOT, "tests")) + r'''
import numpy as np
import test_gpu_front_bits as t
from paper_2503_16037_amd import sgrt
ctx = sgrt.Context(0)
assert sgrt.debug_bounds(ctx) == (True, 0)
for what, make in t.SCENES.items():
    for precision in ("fp32", "fp64"):
        t.say("checked", what, precision)
        t.same_bits(sgrt, ctx, make(), ({}, dict(timing=True)), precision=precision)
    if what == "hubs":
        continue
    for n, tiles in ((3, (8, 16, 64)), (70, (64,))):
        t.say("checked", what, n, "wavelengths")
        sc = make().with_(abs_scale=np.geomspace(0.2, 4.0, n).astype(np.float32))
        t.same_bits(sgrt, ctx, sc, [dict(lambda_tile=w) for w in tiles])
assert sgrt.debug_bounds(ctx) == (True, 0)
print("checked front: clean", flush=True)
''')
    r = subprocess.run([sys.executable, "-u", "-c", child], env=dict(os.environ, SGRT_LIB="debug"), capture_output=True,
                       text=True, timeout=280)
    print(r.stdout[-3000:])
    assert r.returncode == 0, r.stderr[-4000:]
    assert "checked front: clean" in r.stdout
