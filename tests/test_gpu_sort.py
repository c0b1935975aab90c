"""Sizes where the radix sort changes its passes: one tile, few tiles (every
workgroup sums the histogram), many tiles, digits of 9 and 10 bits (from
278,528 items with 17 to 20-bit or 25 to 30-bit keys), and the edges of their
tiles.  The total and the per-vertex counts sort by both sides' ids; all
against the oracle (whole numbers: equality)."""
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


def check(ctx, g):
    import torch

    t = bbc.graph_tensors(g, "cuda:0")
    pv = torch.empty(g.n_u + g.n_v, dtype=torch.int64, device="cuda:0")
    want = oracle.count(g)
    assert ctx.count(*t, g.n_v, opts=bbc.options(queue_chunk=1)) == want
    assert ctx.count(*t, g.n_v, per_vertex=pv) == want
    assert int(pv.sum()) == 4 * want
    ref = oracle.per_vertex(g) if hasattr(oracle, "per_vertex") else None
    if ref is not None:
        assert np.array_equal(pv.cpu().numpy(), np.asarray(ref))


@pytest.mark.parametrize("m", [4095, 4096, 4097, 8192, 128 * 4096, 128 * 4096 + 1])
def test_tiles(ctx, m):
    check(ctx, synth.uniform_graph(3000, 2000, m, 0.3, m))


@pytest.mark.parametrize("n_u,n_v", [(70_000, 65_537), (131_073, 262_145), (600_000, 1000)])
@pytest.mark.parametrize("m", [278_527, 278_528, 8704 * 33 + 1, 17408 * 17 - 1])
def test_wide_digits(ctx, n_u, n_v, m):
    check(ctx, synth.chung_lu_graph(n_u, n_v, m, 2.1, 2.1, 300, 300, m, p_neg=0.3))
