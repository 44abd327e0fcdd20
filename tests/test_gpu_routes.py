"""Which engine the hybrid and plain modes run, on both sides of each line, with
the batched engine's answer: the per-workgroup engine follows the seeds at once
on small graphs, on larger ones where a cut search takes few arcs or many
levels, and where its queue may overflow only on deep ones."""
import functools

import numpy as np
import pytest

import graphgen
import oracle
from conftest import hip_available
from test_gpu_swarm import graph as skewed

pytestmark = pytest.mark.gpu

if hip_available():
    from paper_1704_01077_amd import tkc
else:
    tkc = None

BATCHED, SWARM = 1, 2


@pytest.fixture()
def ctx():
    if not hip_available():
        pytest.skip("no GPU")
    import torch
    torch.cuda.init()
    c = tkc.Context(0)
    yield c
    c.close()


def same(a, b):
    for x, y in zip(a[:4], b[:4]):
        assert np.array_equal(x, y)


@functools.lru_cache(maxsize=None)
def graph(kind):
    r = np.random.default_rng(7)
    if kind == "random":   # many cut searches of few arcs
        n = 20000
        e = r.integers(0, n, (300000, 2))
    elif kind == "social":   # cut searches that take a large part of the graph
        return graphgen.ba_graph(20000, 20, 5)
    elif kind == "lattice":   # a ring lattice with few shortcuts: deep
        n = 30000
        v = np.repeat(np.arange(n), 8)
        w = (v + np.tile([1, -1, 2, -2, 3, -3, 4, -4], n)) % n
        w = np.where(r.random(len(v)) < 0.003, r.integers(0, n, len(v)), w)
        e = np.stack([v, w], 1)
    e = e[e[:, 0] != e[:, 1]]
    directed = kind == "lattice"
    if not directed:
        e = np.sort(e, axis=1)
    return graphgen.make(kind, n, np.unique(e, axis=0).astype(np.int32), directed)


@pytest.mark.parametrize("kind,k,engine", [("random", 10, SWARM), ("social", 100, BATCHED), ("lattice", 3, SWARM)])
def test_hybrid_by_arcs_and_levels(ctx, kind, k, engine):
    g = graph(kind)
    assert g.n + len(g.edges) > 1 << 18
    dg = tkc.Graph.from_graphgen(ctx, g)
    for turn in range(2):   # the depth of the graph is known in the second
        a = tkc.topk_closeness(dg, k, "nbcut", "hybrid")
        if turn:   # (main_kernel goes by time, and a first launch loads its code)
            assert a[4]["main_kernel"] == engine, a[4]
        same(a, tkc.topk_closeness(dg, k, "nbcut", "batched"))
        h = tkc.topk_harmonic(dg, k, "nbcut", "hybrid")
        hb = tkc.topk_harmonic(dg, k, "nbcut", "batched")
        assert np.array_equal(h[0], hb[0]) and np.array_equal(h[1], hb[1])
    S, reach = oracle.sums(g.n, g.edges, g.directed, sources=a[0])
    assert np.array_equal(S, a[1]) and np.array_equal(reach, a[2])
    dg.free()


@pytest.mark.parametrize("kind", ["random", "lattice"])
def test_hybrid_short_queue(ctx, kind):
    """A queue shorter than the graph: tried where the graph is deep (searches
    overflow, the batched engine takes them), left out elsewhere."""
    g = graph(kind)
    ctx.tune(swarm_qcap=256)   # before the workspace is laid out
    dg = tkc.Graph.from_graphgen(ctx, g)
    want = tkc.topk_closeness(dg, 3, "nbcut", "batched")
    for turn in range(2):
        a = tkc.topk_closeness(dg, 3, "nbcut", "hybrid")
        assert (a[4]["deferred"] > 0) == (kind == "lattice"), a[4]
        same(a, want)
    dg.free()


def test_hybrid_wide_bitmap(ctx):
    """Deep parts in a graph of so many vertices that the visited set takes
    over 64 KB of LDS."""
    r = np.random.default_rng(3)
    e, at = [], 0
    for c in (2000, 1500, 999):
        v = np.arange(c)
        e += [np.stack([at + v, at + (v + 1) % c], 1), at + r.integers(0, c, (c // 50, 2))]
        at += c
    p = np.arange(at, 545000, 2)
    e = np.concatenate(e + [np.stack([p, p + 1], 1)])
    e = np.unique(e[e[:, 0] != e[:, 1]], axis=0)
    g = graphgen.make("wide", 545001, e.astype(np.int32), True)
    assert (g.n + 31) // 32 * 4 > 64 << 10
    dg = tkc.Graph.from_graphgen(ctx, g)
    for variant in ("nbcut", "degcut", "degcut"):
        a = tkc.topk_closeness(dg, 20, variant, "hybrid")
        same(a, tkc.topk_closeness(dg, 20, variant, "batched"))
        S, reach = oracle.sums(g.n, g.edges, True, sources=a[0])
        assert np.array_equal(S, a[1]) and np.array_equal(reach, a[2])
    assert a[4]["main_kernel"] == SWARM, a[4]
    dg.free()


def test_hybrid_size_line(ctx):
    """Up to 2^18 vertices and edges the per-workgroup engine follows at once:
    its short queue defers searches; beyond, this shallow graph stays batched."""
    ctx.tune(swarm_qcap=64)
    for arcs in (250000, 275000):
        g = skewed(9000, arcs, True)
        dg = tkc.Graph.from_graphgen(ctx, g)
        a = tkc.topk_closeness(dg, 50, "degcut", "hybrid")
        assert (a[4]["deferred"] > 0) == (arcs == 250000), a[4]
        same(a, tkc.topk_closeness(dg, 50, "degcut", "batched"))
        dg.free()


def test_plain_size_lines(ctx):
    """Plain mode: one workgroup up to 2^16 vertices and arcs, up to 2^17 after
    the k searches of the plain engine that fill the top k, the plain engine
    beyond; the same searches everywhere."""
    for arcs, engines in ((50000, {SWARM}), (110000, {0, SWARM}), (140000, {0})):
        g = skewed(9000, arcs, True)
        assert (g.n + len(g.edges) > 1 << 16) == (arcs > 50000)
        dg = tkc.Graph.from_graphgen(ctx, g)
        for k in (1, 5, 60):
            for variant in ("nbcut", "degcut"):
                tkc.topk_closeness(dg, k, variant, "plain")
                a = tkc.topk_closeness(dg, k, variant, "plain")
                assert a[4]["main_kernel"] in engines, a[4]
                same(a, tkc.topk_closeness(dg, k, variant, "batched"))
                done, b, st = tkc.topk_closeness_budget(dg, k, variant, 10**6)
                assert done
                same(a, b)
                for key in ("bfs_started", "bfs_exact", "bfs_cut", "skipped", "m_vis", "max_level", "mode_used"):
                    assert a[4][key] == st[key], key
            h = tkc.topk_harmonic(dg, k, "nbcut", "plain")
            hb = tkc.topk_harmonic(dg, k, "nbcut", "batched")
            assert np.array_equal(h[0], hb[0]) and np.array_equal(h[1], hb[1])
            t = tkc.topk_closeness_ties(dg, k, "nbcut", "plain")
            tb = tkc.topk_closeness_ties(dg, k, "nbcut", "batched")
            same(t, tb)
        dg.free()
