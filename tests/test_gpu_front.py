"""Sweeps over the front: matrices above the size from which a series' later sweeps visit only
the nodes that can still change.  Such a sweep leaves every edge the bits a whole sweep gives, so
the solutions meet the bars of the whole solve on every edge: against the FP64 oracle (pixels 1e-10
in FP64 and 1e-4 in FP32, as everywhere; phi at the stopping rule's per-edge accuracy), on ragged
node counts, a periodic slab, a graph with a few nodes above 64 couplings, under graph replay and
launch by launch, and with an iterate that overflows."""
import sys

import numpy as np
import pytest

import oracle
from paper_2503_16037_amd import scenes

pytestmark = pytest.mark.gpu

DIMS = (45, 37, 23)  # 39,960 nodes, about 19 M structural nonzeros: above the front's 16 M


def say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


@pytest.fixture(scope="module")
def ctx():
    from paper_2503_16037_amd import sgrt
    c = sgrt.Context(0)
    yield c
    c.close()


def rel_err(a, b):
    return np.abs(np.asarray(a) - np.asarray(b)) / np.maximum(np.abs(np.asarray(b)), 1e-300)


def with_hub(sc, n=90):
    """The scene with one more node of degree above 64: node 7 coupled to n spread nodes."""
    tail = np.repeat(np.arange(sc.n_nodes), np.diff(sc.adj_ptr))
    far = np.linspace(1000, sc.nvox - 1, n).astype(np.int64)
    up = tail < sc.adj_idx
    ap, ai = scenes.adjacency_from_pairs(sc.n_nodes, np.concatenate([tail[up], np.full(n, 7)]),
                                         np.concatenate([sc.adj_idx[up], far]))
    return sc.with_(adj_ptr=ap, adj_idx=ai)


@pytest.mark.parametrize("what, precision", [("cloud", "fp32"), ("cloud", "fp64"), ("slab", "fp32"), ("hub", "fp64")])
def test_front_matches_oracle(ctx, what, precision):
    from paper_2503_16037_amd import sgrt
    sc = (scenes.make_plume(seed=8, nx=DIMS[0], ny=DIMS[1], nz=DIMS[2], periodic=3) if what == "slab" else
          scenes.make_cloud(seed=9, nx=DIMS[0], ny=DIMS[1], nz=DIMS[2]))
    if what == "hub":
        sc = with_hub(sc)
    say("front", what, precision, sc.n_nodes, sc.nnz(), int(sc.degrees().max()))
    assert sc.nnz() >= 16_000_000 and (sc.degrees().max() > 64) == (what == "hub")
    ora = oracle.run(sc)
    bar, phi_bar = (1e-10, 1e-11) if precision == "fp64" else (1e-4, 2e-5)
    with sgrt.Scene(ctx, sc) as g:
        first, info = g.solve(precision=precision)
        assert info["converged"] == 1
        assert rel_err(first, ora["radiance"]).max() < bar
        phi = g.export_vector("phi")
        lit = np.abs(ora["phi"]) > 1e-25
        assert rel_err(phi[lit], ora["phi"][lit]).max() < phi_bar
        # tuned and captured (second solve), replayed (third), launch by launch
        for opts in ({}, {}, dict(timing=True), dict(graphs=False, autotune=False)):
            rad, again = g.solve(precision=precision, **opts)
            assert again["sweeps"] == info["sweeps"]
            assert np.array_equal(rad, first), opts
        assert np.array_equal(g.export_vector("phi"), phi)


def test_front_overflow_is_seen(ctx):
    """Four nodes of the top layer within 14 / 2^16 voxel of each other under the literal node
    weight make the FP32 iterate overflow after the sweeps have gone over to the front; the
    convergence measures have to stay non-finite, and GMRES solves the scene."""
    from paper_2503_16037_amd import sgrt
    nx, ny, nz = DIMS
    sc = scenes.make_plume(seed=8, nx=nx, ny=ny, nz=nz)
    rng = np.random.default_rng(0)
    pos = sc.vol_pos_fx.copy().reshape(nz, ny, nx, 3)
    mu_s = sc.mu_s.copy()
    S = scenes.FX
    for iy in range(2):
        for ix in range(2):
            pos[nz - 1, iy, ix] = [S + (2 * ix - 1) * rng.integers(2, 14), S + (2 * iy - 1) * rng.integers(2, 14),
                                   nz * S - rng.integers(2, 14)]
            mu_s[nz - 1, iy, ix] = 2000.0 / sc.voxel_m
    pos = pos.reshape(-1, 3)
    ap, ai = scenes.radius_graph(pos, nx, ny, nz, 1.8, jitter=0.5)
    sc = sc.with_(vol_pos_fx=pos, mu_s=mu_s, adj_ptr=ap, adj_idx=ai, node_weight_mode=1)
    say("front overflow", sc.n_nodes, sc.nnz())
    assert sc.nnz() >= 16_000_000
    with sgrt.Scene(ctx, sc) as g:
        rad, info = g.solve(allow_noconv=True)
        assert info["gmres_used"] == 1, info
        if info["converged"]:
            ref, ref_info = g.solve(solver="gmres")
            assert ref_info["converged"] == 1
            assert np.all(np.isfinite(rad))
            assert np.abs(rad - ref).max() <= 1e-4 * np.abs(ref).max()
        else:
            assert not info["rel_residual"] <= 1e-6, info


@pytest.mark.parametrize("n_lambda", [7, 12, 31])
def test_batched_front_has_whole_sweeps_bits(ctx, n_lambda):
    """A 32-lane tile takes whole sweeps, the others go over to the front: every tile gives the
    same bits, for every wavelength."""
    from paper_2503_16037_amd import sgrt
    sc = scenes.make_cloud(seed=9, nx=DIMS[0], ny=DIMS[1], nz=DIMS[2], n_lambda=n_lambda)
    say("batched front", n_lambda, 4 * sc.nnz() + 8 * sc.n_edges * n_lambda)
    assert 4 * sc.nnz() + 8 * sc.n_edges * n_lambda >= 128_000_000
    with sgrt.Scene(ctx, sc) as g:
        ref, info = g.solve(lambda_tile=32)
        phi = g.export_vector("phi")
        assert info["converged"] == 1
        err = rel_err(ref[n_lambda // 2], oracle.run(sc, abs_scale=float(sc.abs_scale[n_lambda // 2]))["radiance"])
        assert err.max() < 1e-4
        tiles = [t for t in (8, 16, 64) if t >= n_lambda]
        for opts in [dict(lambda_tile=t) for t in tiles] + [{}, dict(timing=True), {}]:
            rad, again = g.solve(**opts)
            assert again["sweeps"] == info["sweeps"], opts
            assert np.array_equal(rad, ref), opts
            assert np.array_equal(g.export_vector("phi"), phi), opts


def test_batched_front_two_columns(ctx):
    """More than 64 wavelengths: two columns of wavefronts mark and visit the same nodes."""
    from paper_2503_16037_amd import sgrt
    sc = scenes.make_plume(seed=8, nx=41, ny=29, nz=17, n_lambda=70)
    say("batched front, two columns", 4 * sc.nnz() + 8 * sc.n_edges * 70)
    assert 4 * sc.nnz() + 8 * sc.n_edges * 70 >= 128_000_000
    with sgrt.Scene(ctx, sc) as g:
        rad, info = g.solve()
        assert info["converged"] == 1
        for k in (0, 63, 64, 69):
            assert rel_err(rad[k], oracle.run(sc, abs_scale=float(sc.abs_scale[k]))["radiance"]).max() < 1e-4
        again, _ = g.solve()
        assert np.array_equal(again, rad)
