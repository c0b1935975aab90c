"""Calls without the duplicate check on graphs that repeat pairs: the count is
the one-sided walk's over the multigraph, and no call writes outside its
output.  The counts from both sides rely on a simple graph (hashed 6-bit
counters, counter widths by degree), so such graphs never reach them: neither
the small ones worked out by hand here nor per-vertex calls of the size that
the count from both sides otherwise takes."""
import numpy as np
import pytest
import torch

from paper_2601_17707_amd import bbc, synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import __graft_entry__

    __graft_entry__._ensure_built()
    c = bbc.Context(0)
    yield c
    c.close()


def multigraph(n_u, n_v, edges):
    """CSR of (u, v, sign) rows with repeats kept, in the given order per row."""
    e = sorted(edges, key=lambda x: x[0])
    off = np.zeros(n_u + 1, np.int32)
    for u, _, _ in e:
        off[u + 1] += 1
    arrays = (np.cumsum(off, dtype=np.int32), np.array([x[1] for x in e], np.int32), np.array([x[2] for x in e], np.int8))
    return [torch.from_numpy(a).to("cuda:0") for a in arrays]


# v0 over two vertices, each pair c times: the lower vertex meets the upper one
# in c * c wedges and its own copies in C(c, 2), the upper one its own copies
# in C(c, 2), and every number of agreeing wedges n adds C(n, 2)
@pytest.mark.parametrize("copies,want", [(2, 6), (3, 42)])
@pytest.mark.parametrize("call", ["count", "count_noalloc"])
def test_value(ctx, call, copies, want):
    t = multigraph(2, 2, [(u, 0, 1) for u in (0, 1) for _ in range(copies)])
    o = bbc.options(side="u", checks=bbc.CHECK_SIGNS)
    assert getattr(ctx, call)(*t, 2, opts=o) == want
    with pytest.raises(bbc.BbcError) as e:
        getattr(ctx, call)(*t, 2, opts=bbc.options(side="u"))
    assert e.value.status == bbc.EDUP


def repeated(n, m, pairs, seed):
    """A uniform graph of n x n and m edges, and stars of a few vertices whose
    pairs come `pairs` times, with opposite signs at their two ends."""
    g = synth.uniform_graph(n, n, m, 0.3, seed)
    off, adj, sg = np.array(g.offsets, np.int64), np.array(g.adj), np.array(g.signs)
    u = np.repeat(np.arange(n), np.diff(off))
    eu, ev, es = [u], [adj], [sg]
    for i in range(8):
        for x, s in ((10 + i, 1), (n - 20 + i, -1)):
            eu.append(np.full(pairs, x))
            ev.append(np.full(pairs, 100 + i))
            es.append(np.full(pairs, s))
    eu, ev, es = np.concatenate(eu), np.concatenate(ev), np.concatenate(es)
    k = np.argsort(eu, kind="stable")
    off = np.concatenate([[0], np.cumsum(np.bincount(eu, minlength=n))]).astype(np.int32)
    return [torch.from_numpy(a).to("cuda:0") for a in (off, ev[k].astype(np.int32), es[k].astype(np.int8))]


# 8 copies: 64 disagreeing wedges of one pair, past a 6-bit counter; 300: past
# every narrow counter of vertices of 300 edges
@pytest.mark.parametrize("pairs", [2, 8, 9, 300])
@pytest.mark.parametrize("n,m", [(6000, 70_000), (40_000, 90_000)])
def test_per_vertex_stays_in_its_output(ctx, n, m, pairs):
    t = repeated(n, m, pairs, pairs)
    o = bbc.options(checks=bbc.CHECK_SIGNS)
    guard = 4096
    buf = torch.full((2 * n + 2 * guard,), -7, dtype=torch.int64, device="cuda:0")
    out = buf[guard:guard + 2 * n]
    first = None
    for _ in range(2):
        total = ctx.count(*t, n, per_vertex=out, opts=o)
        got = (total, out.cpu().numpy().tobytes())
        assert first in (None, got)
        first = got
    assert bool((buf[:guard] == -7).all()) and bool((buf[guard + 2 * n:] == -7).all())
    with pytest.raises(bbc.BbcError) as e:
        ctx.count(*t, n, per_vertex=out)
    assert e.value.status == bbc.EDUP
    # a simple graph right after is counted as ever, checked or not
    g = synth.uniform_graph(n, n, m, 0.3, 5)
    s = bbc.graph_tensors(g, "cuda:0")
    want = ctx.count(*s, n, per_vertex=out)
    pv = out.clone()
    assert ctx.count(*s, n, per_vertex=out, opts=o) == want and bool((out == pv).all())
