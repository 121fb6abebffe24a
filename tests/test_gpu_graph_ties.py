"""The strongest couplings among far more equal ones than are asked for: the candidates at the
threshold do not fit a list, and the pairs come in the order of their node ids all the same."""
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


def heap(n, together, seed=4):
    """n general nodes, the ones with odd ids and then others up to `together` of them at one
    place (their couplings are infinite), the rest anywhere in a plume's box."""
    sc = scenes.make_plume(seed=3, nx=24, ny=20, nz=12)
    rng = np.random.default_rng(seed)
    pos = np.stack([rng.integers(1, w * FX, n) for w in (24, 20, 12)], 1).astype(np.int32)
    order = np.concatenate([np.arange(1, n, 2), np.arange(0, n, 2)])[:together]
    pos[order] = [11 * FX + 77, 9 * FX + 5, 4 * FX + 123]
    mu = sc.mu_s.copy()
    mu[4, 9, 11] = mu.max()
    return sc.with_(node_pos_fx=pos, mu_s=mu, los_ptr=np.zeros(24 * 20 + 1, np.int64), los_node=np.zeros(0, np.int32),
                    los_t=np.zeros(0), surface_nodes=0), np.sort(order)


def forward(ap, ai):
    tail = np.repeat(np.arange(len(ap) - 1), np.diff(ap))
    up = tail < ai
    return np.stack([tail[up], ai[up]], 1)


@pytest.mark.parametrize("n, together, n_pairs", [(70_000, 66_000, 1000), (70_000, 66_000, 200_000), (9000, 9000, 50_000)])
def test_more_equal_couplings_than_a_list_holds(ctx, n, together, n_pairs):
    """Above 2^31 (and 2^25) infinite couplings: the first pairs in order of (i, j)."""
    from paper_2503_16037_amd import sgrt
    sc, at = heap(n, together)
    say("equal couplings", n, together * (together - 1) // 2, n_pairs)
    ap, ai = sgrt.graph_build(ctx, sc, n_pairs=n_pairs)
    want, i = [], 0
    while sum(map(len, want)) < n_pairs:
        want.append(np.stack([np.full(together - 1 - i, at[i]), at[i + 1:]], 1))
        i += 1
    assert np.array_equal(forward(ap, ai), np.concatenate(want)[:n_pairs])


@pytest.mark.parametrize("together", [5900, 1500])
def test_strongest_couplings_with_ties_match_oracle(ctx, together):
    """All the infinite couplings and some finite ones, or a part of them: the oracle's graph."""
    from paper_2503_16037_amd import sgrt
    sc, at = heap(6000, together)
    for n_pairs in (30_000, together * (together - 1) // 2 + 30_000):
        say("ties against the oracle", together, n_pairs)
        ap, ai = sgrt.graph_build(ctx, sc, n_pairs=n_pairs)
        oap, oai = oracle.coupling_graph(sc, n_pairs=n_pairs)
        assert np.array_equal(ap, oap) and np.array_equal(ai, oai)
