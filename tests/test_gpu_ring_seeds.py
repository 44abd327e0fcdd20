"""The ring engine's start: workgroups that wait until the first searches have
filled the top k, on large graphs a batch that searches first, and that batch
giving up where the graph turns out to be deep."""
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


@pytest.fixture()
def ctx():
    if not hip_available():
        pytest.skip("no GPU")
    import torch
    torch.cuda.init()
    c = tkc.Context(0)
    yield c
    c.close()


def tree(n, seed=4):
    r = np.random.default_rng(seed)
    v = np.arange(1, n)
    u = (r.random(n - 1) * v).astype(np.int64)
    g = graphgen.make("tree", n, np.stack([u, v], 1).astype(np.int32), False)
    return g


def same(a, b, k=None):
    for x, y in zip(a[:4], b[:4]):
        assert np.array_equal(x, y[:k])


@pytest.mark.parametrize("variant", ["nbcut", "nbbound", "degcut"])
def test_ring_gate(ctx, variant):
    """k below, around and above the number of workgroups."""
    g = tree(2500)
    want = oracle.closeness_topk(g.n, g.edges, False, g.n)
    dg = tkc.Graph.from_graphgen(ctx, g)
    for k in (1, 100, 255, 256, 257, 700, g.n):
        print("gate", variant, k, flush=True)
        same(tkc.topk_closeness(dg, k, variant, "hybrid"), want, k)
    dg.free()


@pytest.mark.parametrize("variant", ["nbcut", "nbbound", "nbcutlb"])
def test_ring_seeds(ctx, variant):
    """A shallow graph of more than 2^18 vertices: a batch ends the query."""
    g = tree((1 << 18) + 1000)
    dg = tkc.Graph.from_graphgen(ctx, g)
    want = tkc.topk_closeness(dg, 10, "nbcut", "plain")
    for turn in range(2):
        got = tkc.topk_closeness(dg, 10, variant, "batched")
        same(got, want)
        if turn:   # (main_kernel goes by time, and a first launch loads its code)
            assert got[4]["main_kernel"] == 1, got[4]
    S, r = oracle.sums(g.n, g.edges, False, sources=got[0])
    assert np.array_equal(S, got[1]) and np.array_equal(r, got[2])
    dg.free()


@pytest.mark.parametrize("variant", ["nbbound", "nbcutlb"])
def test_ring_seeds_give_up(ctx, variant):
    """Streets of more than 2^18 vertices, whose depth only the second query
    knows."""
    g = graphgen.grid_graph(530, 0.05, 60, seed=9)
    assert g.n > 1 << 18
    dg = tkc.Graph.from_graphgen(ctx, g)
    got = [tkc.topk_closeness(dg, 10, variant, "batched") for _ in range(2)]
    same(got[0], got[1])
    for a in got:
        assert a[4]["main_kernel"] == 2 and a[4]["max_level"] > 48, a[4]
    S, r = oracle.sums(g.n, g.edges, False, sources=got[0][0])
    assert np.array_equal(S, got[0][1]) and np.array_equal(r, got[0][2])
    src = np.random.default_rng(1).choice(g.n, 1000, replace=False).astype(np.int32)
    S2, r2 = dg.sums(src)
    assert (r2 == r[0]).all() and S2[~np.isin(src, got[0][0])].min() >= S.max()
    dg.free()


@pytest.mark.parametrize("ties", [False, True])
@pytest.mark.parametrize("variant", ["nbcut", "nbbound", "degcut"])
def test_ring_seeds_give_up_with_lone_vertices(ctx, variant, ties):
    """A path of 100 among lone vertices: the batch places lone vertices in the
    top k before it gives up, so the top k has to start over."""
    n, c, k = (1 << 18) + 500, 100, 150
    at = 7 + 2 * np.arange(c)
    g = graphgen.make("path", n, np.stack([at[:-1], at[1:]], 1).astype(np.int32), False)
    ctx.tune(batch_width=256)
    S, r = oracle.sums(n, g.edges, False, sources=at.astype(np.int32))
    order = np.lexsort((at, S))
    lone = np.setdiff1d(np.arange(n), at)
    dg = tkc.Graph.from_graphgen(ctx, g)
    for turn in range(2):
        if ties:
            got = tkc.topk_closeness_ties(dg, c - 20, variant, "batched")
            m = len(got[0])
            assert m in (c - 20, c - 19)
        else:
            got = tkc.topk_closeness(dg, k, variant, "batched")
            m = c
            assert np.array_equal(got[0][c:], lone[:k - c]) and (got[2][c:] == 1).all() and (got[1][c:] == 0).all()
        assert np.array_equal(got[0][:m], at[order][:m]) and np.array_equal(got[1][:m], S[order][:m])
    dg.free()
