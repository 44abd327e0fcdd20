"""Ring engine (searches one per workgroup, cut or complete, visited set in LDS)
against the oracle's exact answer: widths around its words, degrees around
its four-arc records, levels wider than their LDS copy, disconnected graphs,
searches deeper than its level tables, ties and renumbered graphs."""
import functools

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


def _g(name, n, edges):
    return graphgen.make(name, n, np.asarray(edges, dtype=np.int32).reshape(-1, 2), False)


@functools.lru_cache(maxsize=None)
def graph(name):
    kind, n = name.split(":")
    n = int(n)
    if kind == "path":
        return _g(name, n, [(i, i + 1) for i in range(n - 1)])
    if kind == "cycle":
        return _g(name, n, [(i, (i + 1) % n) for i in range(n)])
    if kind == "grid":
        return graphgen.grid_graph(n, 0.05, None, seed=n)
    if kind == "parts":   # unequal grids, a cycle and lone vertices
        a, b = graphgen.grid_graph(n, 0.05, 2, seed=1), graphgen.grid_graph(n // 2, 0.1, 1, seed=2)
        e = [a.edges, b.edges + a.n, np.array([(a.n + b.n + i, a.n + b.n + (i + 1) % 9) for i in range(9)])]
        return _g(name, a.n + b.n + 14, np.concatenate(e))
    if kind == "fan":     # degree 64, the most a light vertex has, hanging off a grid
        a = graphgen.grid_graph(n, 0.05, 2, seed=3)
        e = [a.edges, np.array([(0, a.n + i) for i in range(64 - int(a.row_ptr[1] - a.row_ptr[0]))])]
        return _g(name, a.n + len(e[1]), np.concatenate(e))
    raise KeyError(name)


@functools.lru_cache(maxsize=None)
def answer(name):
    g = graph(name)
    return oracle.closeness_topk(g.n, g.edges, False, g.n)


@pytest.mark.parametrize("variant", ["nbbound", "degbound", "nbcutlb", "degcutlb", "nbcut", "degcut"])
@pytest.mark.parametrize("name", ["path:2", "path:31", "path:33", "cycle:32", "cycle:257", "grid:9", "grid:60",
                                  "parts:40", "fan:30", "path:3000"])
def test_ring_topk(ctx, name, variant):
    g = graph(name)
    ids, S, r, f = answer(name)
    for relabel in (False, True):
        dg = tkc.Graph.from_graphgen(ctx, g, relabel=relabel)
        for k in (1, 10, g.n if g.n <= 300 else 100):
            print("ring", name, variant, k, relabel, flush=True)
            got = tkc.topk_closeness(dg, k, variant, "hybrid" if variant == "degcut" else "batched")
            kk = min(k, g.n)
            assert got[4]["main_kernel"] == 2
            for a, b in zip(got[:4], (ids, S, r, f)):
                assert np.array_equal(a, b[:kk])
        dg.free()


def test_ring_deeper_than_tables(ctx):
    """A path of 8,500 vertices has searches of more levels than the level
    tables hold: the batched engine takes over, with the same answer."""
    n = 8500
    dg = tkc.Graph.from_graphgen(ctx, _g("deep", n, [(i, i + 1) for i in range(n - 1)]))
    got = tkc.topk_closeness(dg, 3, "nbbound", "batched")
    v = np.arange(n, dtype=np.int64)
    S = v * (v + 1) // 2 + (n - 1 - v) * (n - v) // 2
    order = np.lexsort((v, S))[:3]
    assert np.array_equal(got[0], order) and np.array_equal(got[1], S[order]) and (got[2] == n).all()
    dg.free()


@pytest.mark.parametrize("variant", ["nbbound", "nbcut"])
def test_ring_ties(ctx, variant):
    g = graph("cycle:257")   # every vertex ties
    dg = tkc.Graph.from_graphgen(ctx, g)
    got = tkc.topk_closeness_ties(dg, 5, variant, "batched")
    assert np.array_equal(got[0], np.arange(257)) and len(set(got[1].tolist())) == 1
    dg.free()


def test_ring_wide_levels(ctx):
    """Levels of more than 1,024 vertices (read from the queue): the sums of
    the top 10 equal the oracle's, and no sampled vertex is better."""
    g = graphgen.grid_graph(372, 0.05, 40, seed=9)
    assert g.n > 1 << 17
    dg = tkc.Graph.from_graphgen(ctx, g)
    got = tkc.topk_closeness(dg, 10, "nbbound", "batched")
    assert got[4]["main_kernel"] == 2
    S, r = oracle.sums(g.n, g.edges, False, sources=got[0])
    assert np.array_equal(S, got[1]) and np.array_equal(r, got[2])
    src = np.random.default_rng(1).choice(g.n, 2000, replace=False).astype(np.int32)
    S2, r2 = dg.sums(src)
    assert (r2 == r[0]).all() and S2[~np.isin(src, got[0])].min() >= S.max()
    dg.free()
