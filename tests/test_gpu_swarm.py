"""Per-workgroup engine (visited set in LDS) against the oracle: widths around
its bitmap's words, searches that overflow their queue, and graphs on both
sides of the size up to which it is used, alone (plain mode) and many at once."""
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


@functools.lru_cache(maxsize=None)
def graph(n, arcs, directed):
    r = np.random.default_rng(n + arcs)
    # a few popular heads, the rest at random
    a, b = r.integers(0, n, arcs), (n * r.random(arcs) ** 2).astype(np.int64)
    e = np.unique(np.stack([a, b], 1)[a != b], axis=0).astype(np.int32)
    if not directed:
        e = np.unique(np.sort(e, axis=1), axis=0)
    return graphgen.make("swarm", n, e, directed)


@pytest.mark.parametrize("qcap", [64, 1 << 18])
@pytest.mark.parametrize("n", [31, 32, 33, 64, 65, 1000, 4097])
def test_swarm_words(ctx, n, qcap):
    g = graph(n, 6 * n, True)
    want = oracle.closeness_topk(g.n, g.edges, True, g.n)
    h = oracle.harmonic(g.n, g.edges, True)
    keep = ctx.tuning()
    ctx.tune(swarm_qcap=qcap, seed_lanes=4)
    try:
        dg = tkc.Graph.from_graphgen(ctx, g)
        for k in (1, 7, min(n, 300)):
            for variant in ("nbcut", "degcut"):
                for mode in ("hybrid", "plain"):
                    print("swarm", n, qcap, k, variant, mode, flush=True)
                    got = tkc.topk_closeness(dg, k, variant, mode)
                    for a, b in zip(got[:4], want):
                        assert np.array_equal(a, b[:k])
            ids = oracle.harmonic_topk(h, k)
            for mode in ("hybrid", "plain"):
                hv, hh = tkc.topk_harmonic(dg, k, "nbcut", mode)[:2]
                assert np.array_equal(hv, ids) and np.array_equal(hh, h[ids])
        dg.free()
    finally:
        ctx.tune(**keep)


@pytest.mark.parametrize("directed", [True, False])
def test_swarm_size_line(ctx, directed):
    """Both sides of 2^18 vertices and edges: the hybrid's answer is the
    batched engine's, and only the small side runs one search a workgroup."""
    for arcs in (250000, 275000):
        g = graph(9000, arcs, directed)
        assert (g.n + len(g.edges) <= 1 << 18) == (arcs == 250000)
        dg = tkc.Graph.from_graphgen(ctx, g)
        a = tkc.topk_closeness(dg, 50, "degcut", "batched")
        b = tkc.topk_closeness(dg, 50, "degcut", "hybrid")
        for x, y in zip(a[:4], b[:4]):
            assert np.array_equal(x, y)
        assert b[4]["mode_used"] == 2
        dg.free()


def test_swarm_plain_line(ctx):
    """Plain mode on both sides of 2^17 vertices and arcs: the same searches
    (their counters too) and the same answer as with a search cap, which only
    the plain engine has."""
    for arcs in (110000, 140000):
        g = graph(9000, arcs, True)
        assert (g.n + len(g.edges) <= 1 << 17) == (arcs == 110000)
        dg = tkc.Graph.from_graphgen(ctx, g)
        a = tkc.topk_closeness(dg, 5, "nbcut", "plain")
        done, b, st = tkc.topk_closeness_budget(dg, 5, "nbcut", 10**6)
        assert done
        for x, y in zip(a[:4], b):
            assert np.array_equal(x, y)
        for key in ("bfs_started", "bfs_exact", "bfs_cut", "skipped", "m_vis", "max_level", "mode_used"):
            assert a[4][key] == st[key], key
        dg.free()
