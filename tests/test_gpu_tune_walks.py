"""The tuning table serves several kernels: a choice timed on the one-sided walk
(batches) is not applied to a count from both sides of the same size class, and
the other way round; a loaded line serves both; calls counted by matrix products
report no tuned shape."""
import pytest

import oracle
from paper_2601_17707_amd import bbc, synth

pytestmark = pytest.mark.gpu


@pytest.fixture()
def ctx():
    import __graft_entry__

    __graft_entry__._ensure_built()
    c = bbc.Context(0)
    yield c
    c.close()


@pytest.fixture(scope="module")
def single():
    # anchors 10,000 (14 bits), mean list 20 (5 bits): counted from both sides
    return synth.chung_lu_graph(20_000, 10_000, 200_000, 2.1, 2.1, 800, 800, 3, p_neg=0.3)


@pytest.fixture(scope="module")
def members():
    # the same class, as a batch
    return [synth.chung_lu_graph(5_000, 2_500, 50_000, 2.1, 2.1, 300, 300, 10 + i, p_neg=0.3) for i in range(4)]


def count(ctx, g, **kw):
    n = ctx.count(*bbc.graph_tensors(g, "cuda:0"), g.n_v, opts=bbc.options(**kw))
    return n, ctx.stats()


def test_batch_choice_stays_with_batches(ctx, single, members):
    _, plain = count(ctx, single)
    batch = bbc.Batch(members, "cuda:0")
    chosen = ctx.autotune_batched(batch, reps=1)
    n, st = count(ctx, single)
    assert n == oracle.count(single)
    assert st["tuned"] == 0 and (st["band_words"], st["block"]) == (plain["band_words"], plain["block"])
    assert ctx.count_batched(batch).cpu().tolist()[:4] == [oracle.count(g) for g in members]
    assert ctx.stats()["tuned"] == 1 and ctx.stats()["band_words"] == chosen["band_words"]


def test_each_walk_uses_its_own_choice(ctx, single, members):
    batch = bbc.Batch(members, "cuda:0")
    off, adj, sg = bbc.graph_tensors(single, "cuda:0")
    both = ctx.autotune(off, adj, sg, single.n_v, reps=1)
    n, st = count(ctx, single)
    assert n == oracle.count(single) and st["tuned"] == 1
    assert (st["band_words"], st["block"]) == (both["band_words"], both["wg_size"])
    # the same graph was timed on the one-sided walk too, for batches of its class
    ctx.count_batched(batch)
    assert ctx.stats()["tuned"] == 1
    # a later batch choice does not change the single call's
    one = ctx.autotune_batched(batch, reps=1)
    n, st = count(ctx, single)
    assert (st["band_words"], st["block"], st["tuned"]) == (both["band_words"], both["wg_size"], 1)
    ctx.count_batched(batch)
    assert ctx.stats()["band_words"] == one["band_words"]


def test_loaded_line_serves_both(ctx, single, members, tmp_path):
    p = str(tmp_path / "tune.txt")
    with open(p, "w") as f:
        f.write("bbc-tune 3 gfx950\n14 5 4096 128 2 0 4 -1 0 0 0.5\n")
    ctx.tune_load(p)
    n, st = count(ctx, single)
    assert n == oracle.count(single)
    assert (st["band_words"], st["block"], st["tuned"]) == (4096, 128, 1)
    ctx.count_batched(bbc.Batch(members, "cuda:0"))
    assert (ctx.stats()["band_words"], ctx.stats()["tuned"]) == (4096, 1)
    out = str(tmp_path / "out.txt")
    ctx.tune_save(out)
    assert open(out).read() == "bbc-tune 3 gfx950\n14 5 4096 128 2 0 4 -1 0 0 0.5000\n"


def test_matrix_products_report_their_own_launch(ctx, tmp_path):
    g = synth.workload("uniform-2k-1k-20k", 1)
    p = str(tmp_path / "tune.txt")
    with open(p, "w") as f:
        f.write("bbc-tune 3 gfx950\n10 5 4096 128 2 0 4 -1 0 0 0.5\n")  # 1,000 anchors, mean list 20
    ctx.tune_load(p)
    n, st = count(ctx, g)
    assert n == oracle.count(g)
    # 1,000 rows: 16 x 16 tiles of 64 rows, workgroups of 256 threads
    assert (st["tuned"], st["grid"], st["block"], st["band_words"]) == (0, 256, 256, 0)
    n, st = count(ctx, g, queue_chunk=4)
    assert (st["tuned"], st["band_words"], st["block"]) == (1, 4096, 128)
