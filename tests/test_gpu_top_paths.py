"""Counts from both sides reach the regimes that their tests name: the bands of
the statistics are those of the band kernel alone, so hashed anchors leave it at
zero and anchors that overflow, or have many wedges, do not.  All against the
oracle (whole numbers: equality)."""
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


def block(rows, mids, n_u, n_v, seed):
    """A complete block among vertices without an edge."""
    rng = np.random.default_rng(seed)
    u, v = (x.ravel() for x in np.meshgrid(np.arange(rows), np.arange(mids), indexing="ij"))
    return synth.from_edges(n_u, n_v, u, v, np.where(rng.random(u.size) < 0.3, -1, 1))


def bands(ctx, g, **kw):
    t = bbc.graph_tensors(g, "cuda:0")
    assert ctx.count(*t, g.n_v, opts=bbc.options(queue_chunk=1, **kw)) == oracle.count(g)
    st = ctx.stats()
    assert st["band_words"] in (16384, 32768)  # the default shapes of the count from both sides
    return st["bands"]


# neither side has more than 63 vertices, so no pair more common middles: the
# wave regime (up to 1,024 wedges) and the two tables (4,096 and 16,384)
@pytest.mark.parametrize("rows,mids", [(10, 20), (17, 63), (60, 63), (63, 63)])
@pytest.mark.parametrize("light", [0, -1])
def test_hashed(ctx, rows, mids, light):
    assert bands(ctx, block(rows, mids, 4000, 4000, rows), wave_max_work=light) == 0


# more than 63 common middles of one kind overflow a hashed counter (of rows or,
# where these are the longer lists, of columns); 300 x 63 wedges are more than
# the tables take
@pytest.mark.parametrize("rows,mids", [(12, 300), (60, 130), (200, 63), (300, 63)])
def test_bands(ctx, rows, mids):
    assert bands(ctx, block(rows, mids, 4000, 4000, rows)) > 0


def test_many_band_anchors(ctx):
    """A queue per XCD from 512 anchors."""
    g = synth.chung_lu_graph(70_000, 50_000, 1_200_000, 2.0, 2.0, 9000, 9000, 17, p_neg=0.3)
    assert bands(ctx, g) >= 512


@pytest.mark.parametrize("gen", ["uniform", "power law"])
def test_wide_sides(ctx, gen):
    """Beyond 2^20 ranks light anchors stay hashed."""
    n_u, n_v, m = 2_600_003, 1_300_001, 3_000_000
    if gen == "uniform":
        assert bands(ctx, synth.uniform_graph(n_u, n_v, m, 0.3, 3)) == 0
    else:
        assert bands(ctx, synth.chung_lu_graph(n_u, n_v, m, 2.1, 2.1, 20_000, 20_000, 3, p_neg=0.3)) < 20_000


# counters of 16 and of 32 bits, per vertex
@pytest.mark.parametrize("rows,mids", [(3, 300), (3, 65_535), (3, 65_536), (5, 70_000)])
def test_per_vertex_widths(ctx, rows, mids):
    g = block(rows, mids, 20_000, mids + 20_000, mids)
    h = synth.uniform_graph(20_000, g.n_v, 70_000, 0.3, 3)
    u, v, s = (np.concatenate(x) for x in zip(g.edges(), h.edges()))
    key, first = np.unique(u.astype(np.int64) * g.n_v + v, return_index=True)
    g = synth.from_edges(20_000, g.n_v, key // g.n_v, key % g.n_v, s[first])
    t = bbc.graph_tensors(g, "cuda:0")
    pv = torch.empty(g.n_u + g.n_v, dtype=torch.int64, device="cuda:0")
    assert ctx.count(*t, g.n_v, per_vertex=pv) == oracle.count(g)
    st = ctx.stats()
    assert st["band_words"] == 16384 and st["bands"] > 0
    assert np.array_equal(pv.cpu().numpy().astype(np.uint64), np.asarray(oracle.per_vertex(g)).astype(np.uint64))
