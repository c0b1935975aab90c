"""Counts from both sides on sides whose ranks leave the hashed slots narrower
counters: anchors on either side of each bound (2^20, 2^22, 2^24 ranks), pairs
with one common neighbour less than a counter holds, as many, and more (which
are left to the bands), in the wave, the table and the band regimes, against
the oracle (whole numbers: equality)."""
import numpy as np
import pytest
import torch

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


def cluster(n_u, n_v, rows, mids, loose, seed):
    """`rows` U vertices over `mids` common V vertices (every tenth edge left
    out), the vertices of highest degree and so of the highest ranks, and
    `loose` edges between other vertices, none of them meeting another's
    often."""
    rng = np.random.default_rng(seed)
    u, v = (x.ravel() for x in np.meshgrid(np.arange(rows), np.arange(mids), indexing="ij"))
    keep = (u * 3 + v) % 10 != 0 if rows > 8 else np.ones(u.size, bool)
    lu, lv = rng.integers(rows, n_u, loose), rng.integers(mids, n_v, loose)
    key = np.unique(np.concatenate([u[keep] * n_v + v[keep], lu * n_v + lv]))
    return synth.from_edges(n_u, n_v, key // n_v, key % n_v, np.where(rng.random(key.size) < 0.3, -1, 1))


@pytest.mark.parametrize("ranks,bits", [(1 << 20, 5), (1 << 22, 4), (1 << 24, 3)])
@pytest.mark.parametrize("rows", [2, 40, 700])
def test_counter_bounds(ctx, ranks, bits, rows):
    most = (1 << bits) - 1
    for mids in (most - 1, most, most + 1, 2 * most + 2, 2 * most + 3):
        # the highest ranks straddle the bound
        g = cluster(ranks + rows // 2, ranks // 4, rows, mids, 1000, mids)
        t = bbc.graph_tensors(g, "cuda:0")
        want = oracle.count(g)
        for kw in ({}, {"wave_max_work": -1}):
            assert ctx.count(*t, g.n_v, opts=bbc.options(queue_chunk=1, **kw)) == want, (mids, kw)


@pytest.mark.parametrize("n_u,n_v", [((1 << 20) + 9, 140_000), (300_000, (1 << 20) + 20), ((1 << 22) + 9, 600_000)])
@pytest.mark.parametrize("rows,mids", [(20, 30), (20, 33), (300, 66)])
def test_per_vertex(ctx, n_u, n_v, rows, mids):
    g = cluster(n_u, n_v, rows, mids, 70_000, rows + mids)
    t = bbc.graph_tensors(g, "cuda:0")
    pv = torch.empty(n_u + n_v, dtype=torch.int64, device="cuda:0")
    want = oracle.count(g)
    assert ctx.count(*t, g.n_v, per_vertex=pv) == want
    assert np.array_equal(pv.cpu().numpy(), np.asarray(oracle.per_vertex(g)).astype(np.int64))


@pytest.mark.parametrize("gen", ["uniform", "power law"])
def test_wide_sides(ctx, gen):
    n_u, n_v, m = 2_600_003, 1_300_001, 6_000_000
    g = (synth.uniform_graph(n_u, n_v, m, 0.3, 3) if gen == "uniform" else
         synth.chung_lu_graph(n_u, n_v, m, 2.1, 2.1, 20_000, 20_000, 3, p_neg=0.3))
    t = bbc.graph_tensors(g, "cuda:0")
    assert ctx.count(*t, g.n_v) == oracle.count(g)
