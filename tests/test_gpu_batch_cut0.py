"""Batches whose searches are all cut before their first level: a hub's x is
below every other vertex's bound, and degree bounds skip nothing, so that such
batches make up most of the order and end the launch.  They must leave nothing
behind: answers equal the oracle's, and so do complete searches (sums) of the
next call on the same workspace."""
import numpy as np
import pytest

import graphgen
import oracle
from conftest import hip_available

pytestmark = pytest.mark.gpu

if hip_available():
    from paper_1704_01077_amd import tkc
else:
    tkc = None


@pytest.fixture(scope="module")
def ctx():
    if not hip_available():
        pytest.skip("no GPU")
    import torch
    torch.cuda.init()
    c = tkc.Context(0)
    yield c
    c.close()


def hub_graph(directed, n=12000, seed=11):
    """A hub that reaches its whole part of 8,000 in one step, a second part of
    3,000, pairs and lone vertices."""
    r = np.random.default_rng(seed)
    a, b = 8000, 11000
    e = [np.stack([np.zeros(a - 1, np.int64), np.arange(1, a)], 1), r.integers(0, a, (3 * a, 2)),
         r.integers(a, b, (9000, 2)), np.stack([np.arange(b, b + 400, 2), np.arange(b + 1, b + 401, 2)], 1)]
    if directed:
        e.append(np.stack([np.arange(1, a), np.zeros(a - 1, np.int64)], 1))
    e = np.concatenate(e)
    e = e[e[:, 0] != e[:, 1]]
    if not directed:
        e = np.sort(e, axis=1)
    return graphgen.make("hub", n, np.unique(e, axis=0).astype(np.int32), directed)


@pytest.mark.parametrize("width", [64, 256])
@pytest.mark.parametrize("directed", [False, True])
def test_batches_cut_at_level_zero(ctx, directed, width):
    g = hub_graph(directed)
    want = oracle.closeness_topk(g.n, g.edges, directed, 1)
    src = np.random.default_rng(3).choice(g.n, 256, replace=False).astype(np.int32)
    S, r = oracle.sums(g.n, g.edges, directed, sources=src)
    keep = ctx.tuning()
    ctx.tune(batch_width=width)
    try:
        dg = tkc.Graph.from_graphgen(ctx, g)
        pk = tkc.Pack(ctx, [dg])
        for rep in range(8):
            print("cut at level 0", directed, width, rep, flush=True)
            got = tkc.topk_closeness(dg, 1, "degcut", "batched")
            for x, y in zip(got[:4], want):
                assert np.array_equal(x, y)
            assert got[4]["bfs_cut"] > g.n // 2   # nearly every vertex with an arc
            S2, r2 = dg.sums(src)
            assert np.array_equal(S2, S) and np.array_equal(r2, r)
            res, _ = pk.topk([0], [1], "degcut")
            for x, y in zip(res[0], want):
                assert np.array_equal(x, y)
            S2, r2 = dg.sums(src)
            assert np.array_equal(S2, S) and np.array_equal(r2, r)
        pk.close()
        dg.free()
    finally:
        ctx.tune(**keep)
