"""Radix sorts of 25 to 28-bit keys in three passes of 9 and 10 bits: sides of
more than 2^24 and 2^27 vertices and just enough edges for wide digits, by both
walks and on both sides, against the oracle (whole numbers: equality)."""
import numpy as np
import pytest

import oracle
from paper_2601_17707_amd import bbc, synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import __graft_entry__

    __graft_entry__._ensure_built()
    c = bbc.Context(0)
    yield c
    c.close()


def graph(n_u, n_v, m):
    """A dense corner at both ends of the ids and edges all over."""
    rng = np.random.default_rng(m)
    u = np.concatenate([rng.integers(0, 3000, m // 4), n_u - 1 - rng.integers(0, 3000, m // 4),
                        rng.integers(0, n_u, m - m // 2)])
    v = np.concatenate([rng.integers(0, 3000, m // 4), n_v - 1 - rng.integers(0, 3000, m // 4),
                        rng.integers(0, n_v, m - m // 2)])
    key = np.unique(u * n_v + v)
    return synth.from_edges(n_u, n_v, key // n_v, key % n_v, np.where(rng.random(key.size) < 0.3, -1, 1))


# from both sides (4 to 1, either way) and one-sided (beyond 8 to 1)
@pytest.mark.parametrize("n_u,n_v", [((1 << 24) + 5, 1 << 22), (1 << 22, (1 << 24) + 5), ((1 << 27) + 3, 1 << 25),
                                     ((1 << 24) + 5, 1 << 20)])
def test_wide_keys(ctx, n_u, n_v):
    g = graph(n_u, n_v, 290_000)
    assert g.m >= 278_528
    t = bbc.graph_tensors(g, "cuda:0")
    want = oracle.count(g)
    assert want > 0
    for side in ("u", "v"):
        assert ctx.count(*t, g.n_v, opts=bbc.options(side=side)) == want, side
