"""Totals of single graphs by the one-sided walk: its kernel shapes, schedules,
grids and regimes, on graphs that the count from both sides leaves to it (sides
beyond 8 to 1, by isolated vertices, or a mean degree above 64), with a knob of
the walk set so that no matrix product is taken.  test_route.py checks that
these graphs take this route; all against the oracle (whole numbers: equality)."""
import functools

import numpy as np
import pytest

import oracle
from paper_2601_17707_amd import bbc, synth

pytestmark = pytest.mark.gpu


def widened(g, n_u, n_v):
    """The same edges among more vertices."""
    u, v, s = g.edges()
    return synth.from_edges(n_u, n_v, u, v, s)


@functools.lru_cache(None)
def power_law():
    """Hubs, middling anchors and light ones over several bands of every shape."""
    return widened(synth.chung_lu_graph(60_000, 40_000, 500_000, 2.1, 2.0, 3_000, 900, 77, p_neg=0.35), 400_000, 40_000)


@functools.lru_cache(None)
def widths():
    """Degrees of every counter width (4, 8, 16 and 32 bits)."""
    rng = np.random.default_rng(22)
    n_u, n_v = 9 * 70_000, 70_000
    us, vs = [], []
    for i, d in enumerate([3, 15, 16, 200, 255, 256, 900, 66_000]):
        for k in range(2):  # two of a kind, so that they share centres
            us.append(100 + np.arange(d) + k)
            vs.append(np.full(d, n_v - 1 - 2 * i - k))
            if d <= 900:
                us.append(np.full(d, 2 * i + k))
                vs.append(np.arange(d) + k)
    key = np.unique(np.concatenate(us).astype(np.int64) * n_v + np.concatenate(vs) % n_v)
    return synth.from_edges(n_u, n_v, key // n_v, key % n_v, np.where(rng.random(key.size) < 0.3, -1, 1))


@functools.lru_cache(None)
def light_limit():
    """An anchor of 100 centres and only 70 wedges: beyond the wave regime's 63
    centres, among light ones (anchors on V)."""
    rng = np.random.default_rng(3)
    us, vs = list(range(100)) + list(range(30, 180)), [0] * 100 + [1] * 150
    for v in range(2, 41):
        for c in rng.choice(180, size=int(rng.integers(2, 9)), replace=False):
            us.append(int(c))
            vs.append(v)
    return synth.from_edges(8 * 41 + 1, 41, us, vs, np.where(rng.random(len(us)) < 0.4, -1, 1))


@functools.lru_cache(None)
def wide_anchors():
    """More than 2^20 anchors: the lowest have more ranks above them than a
    wave's key holds."""
    return synth.chung_lu_graph(9_000_000, 1_100_000, 3_500_000, 2.1, 2.1, 2_000, 2_000, 9, p_neg=0.4)


@functools.lru_cache(None)
def dense():
    return synth.uniform_graph(12_000, 12_000, 800_000, 0.3, 4)


GRAPHS = {"power law": power_law, "widths": widths, "light limit": light_limit, "wide anchors": wide_anchors,
          "dense": dense}
BY_DEFAULT = ("power law", "widths", "wide anchors", "dense")  # also without a knob


@functools.lru_cache(None)
def want(name):
    return oracle.count(GRAPHS[name]())


@pytest.fixture(scope="module")
def ctx():
    import __graft_entry__

    __graft_entry__._ensure_built()
    c = bbc.Context(0)
    yield c
    c.close()


@pytest.mark.parametrize("bw,wg", bbc.WEDGE_SHAPES)
@pytest.mark.parametrize("name", ["power law", "widths", "dense"])
def test_every_shape(ctx, name, bw, wg):
    t = bbc.graph_tensors(GRAPHS[name](), "cuda:0")
    n_v = GRAPHS[name]().n_v
    for side in ("u", "v"):
        for kw in ({}, {"schedule": "static"}, {"schedule": "static", "wg_per_cu": 1}, {"wg_per_cu": 2, "wave_max_work": -1},
                   {"queue_chunk": 5, "wave_max_work": 100}):
            assert ctx.count(*t, n_v, opts=bbc.options(side=side, band_words=bw, wg_size=wg, **kw)) == want(name), (side, kw)
            assert ctx.stats()["band_words"] == bw and ctx.stats()["block"] == wg


SETTINGS = [dict(wave_max_work=-1), dict(queue_chunk=1), dict(wave_max_work=1), dict(wave_max_work=16),
            dict(wave_max_work=200), dict(queue_chunk=3), dict(queue_chunk=64, wave_max_work=300),
            dict(schedule="static", queue_chunk=5), dict(wave_max_work=100000)]


@pytest.mark.parametrize("kw", SETTINGS, ids=[str(k) for k in SETTINGS])
@pytest.mark.parametrize("name", ["power law", "widths", "light limit"])
def test_every_setting(ctx, name, kw):
    t = bbc.graph_tensors(GRAPHS[name](), "cuda:0")
    for side in ("u", "v"):
        assert ctx.count(*t, GRAPHS[name]().n_v, opts=bbc.options(side=side, **kw)) == want(name), side
        assert ctx.stats()["band_words"] == 8192  # the one-sided walk's default shape


@pytest.mark.parametrize("kw", [dict(), dict(wave_max_work=-1), dict(queue_chunk=16)], ids=str)
def test_wide_anchor_side(ctx, kw):
    t = bbc.graph_tensors(wide_anchors(), "cuda:0")
    assert ctx.count(*t, wide_anchors().n_v, opts=bbc.options(side="v", **kw)) == want("wide anchors")
    assert ctx.stats()["band_words"] == 8192


@pytest.mark.parametrize("name", ["power law", "widths", "dense"])
def test_defaults(ctx, name):
    t = bbc.graph_tensors(GRAPHS[name](), "cuda:0")
    assert ctx.count(*t, GRAPHS[name]().n_v) == want(name)
    assert ctx.stats()["band_words"] == 8192
    if name != "widths":
        assert ctx.count_noalloc(*t, GRAPHS[name]().n_v) == want(name)
