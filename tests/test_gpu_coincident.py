"""Coupled general nodes at one place: the edge between them has no direction.  Such an out-edge
owns and seeds no lattice point (unless no out-edge of the node has a direction: the first then takes
all), and such an incoming direction counts as straight down.  Both rules for the cells, below and above
degree 64, screened and by the FP64 scan alone, against the FP64 oracle's owners and colours of the
remaining out-edges."""
import sys

import numpy as np
import pytest

import oracle
from paper_2503_16037_amd import scenes

pytestmark = pytest.mark.gpu


def say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


@pytest.fixture(scope="module")
def ctx():
    from paper_2503_16037_amd import sgrt
    c = sgrt.Context(0)
    yield c
    c.close()


def coincident_scene(most, first, sigma_mode):
    """Hubs of degree `most` whose twin (a node at the same place) is their first out-edge or the
    one after it, and a group of three nodes at one place coupled to each other alone."""
    rng = np.random.default_rng(most)
    sc = scenes.make_random_small(5, nx=9, ny=8, nz=5, vza=30.0, vaa=200.0, kscale=0.5, surface=False)
    pos, lp, ln, lt = oracle.los_nodes(sc.nx, sc.ny, sc.nz, sc.view_dir, sc.voxel_m, "step", step_m=45.0)
    n = len(pos)
    pos[1:200:20] = pos[0:200:20]
    pos[n - 2:] = pos[n - 3]
    a, b = [n - 3, n - 3, n - 2], [n - 2, n - 1, n - 1]
    others = np.arange(200, n - 3)
    for h in range(20, 200, 20):
        a += [h] * most
        lower = [] if first else [h - 20]  # a partner with a lower id than the twin's
        b += [h + 1, *lower, *rng.choice(others, most - 1 - len(lower), replace=False)]
    ap, ai = scenes.adjacency_from_pairs(n, np.array(a), np.array(b))
    return scenes.with_los_nodes(sc, pos, lp, ln, lt).with_(adj_ptr=ap, adj_idx=ai, sigma_mode=sigma_mode)


def cells(u, s, NF, sigma_mode):
    """Owner of every lattice point, out-edges without a direction (all zero) left out."""
    has = np.flatnonzero(np.any(s != 0.0, axis=1))
    if len(has) == 0:
        return np.zeros(NF, np.int64)
    u = u if np.any(u != 0.0) else np.array([0.0, 0.0, -1.0])
    own = oracle.colours(u, s[has], NF) if sigma_mode else oracle.ownership(u, s[has], NF)
    return has[own]


@pytest.mark.parametrize("sigma_mode", [0, 1])
@pytest.mark.parametrize("most, first", [(4, True), (8, False), (31, False), (33, True), (64, False), (65, True), (300, False)])
def test_coincident_nodes(ctx, most, first, sigma_mode):
    from paper_2503_16037_amd import sgrt
    sc = coincident_scene(most, first, sigma_mode)
    say("coincident nodes, degree", int(sc.degrees().max()), "cells", sigma_mode)
    NF, w = sc.n_fib, oracle.hg_table(float(sc.hg_g[0]), sc.n_fib)
    sun = -np.asarray(sc.sun_dir, np.float64) / np.linalg.norm(np.asarray(sc.sun_dir, np.float64))
    with sgrt.Scene(ctx, sc) as g:
        got = []
        for screen in (True, False):
            g.solve(precision="fp64", screen=screen, scatter_order=1)
            rp, _, val = g.export_csr(cols=False)
            got.append((rp, val, g.export_vector("qsun")))
        for x, y in zip(*got):
            assert np.array_equal(x, y)
    rp, val, qsun = got[0]
    pos = np.asarray(sc.node_pos_fx, np.float64)
    n = len(pos)
    for l in list(range(20, 200, 20)) + [21, n - 3, n - 1]:
        off, end = int(sc.adj_ptr[l]), int(sc.adj_ptr[l + 1])
        d = end - off
        D = pos[sc.adj_idx[off:end]] - pos[l]
        length = np.sqrt((D * D).sum(1))
        s = D / np.where(length > 0, length, 1.0)[:, None]
        assert (length == 0).any()
        block = val[rp[off]:rp[end]].reshape(d, d)  # row: out-edge, column: in-edge
        for m in list(range(min(d, 12))) + [d - 1, -1]:
            ref = np.bincount(cells(sun if m < 0 else -s[m], s, NF, sigma_mode), w, minlength=d)
            if m < 0:
                assert np.abs(qsun[off:end] - ref).max() < 1e-6, (l, "sun")
            elif block[:, m].sum() > 0:
                assert np.abs(block[:, m] / block[:, m].sum() - ref).max() < 1e-11, (l, m)
