"""Batched engine's pull items and shared push rows against the oracle's
sums: in-degrees around an item's arcs (256) and a wave's lanes, runs of more
than 64 vertices without arcs, every batch width, with the direction forced
to pull and to push by the context's thresholds."""
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

DEGREES = [0, 1, 3, 4, 5, 63, 64, 65, 127, 128, 255, 256, 257, 260, 511, 512, 513, 700]


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
def graph(name):
    """Vertices of every degree above, each followed by a run of vertices of
    degree 0 to 3 (runs of 70: longer than an item), over a common pool."""
    rng = np.random.default_rng(7)
    directed = name == "directed"
    n_pool = 800
    e, v = [], n_pool
    for d in DEGREES:
        for w in rng.choice(n_pool, d, replace=False):
            e.append((int(w), v))
        v += 1
        for i in range(70):
            for w in rng.choice(n_pool, i % 4, replace=False):
                e.append((int(w), v))
            v += 1
    n = v
    for w in range(1, n_pool):   # the pool: a tree with some chords
        e.append((int(rng.integers(0, w)), w))
    for _ in range(600):
        e.append((int(rng.integers(0, n)), int(rng.integers(0, n))))
    return graphgen.make(name, n, np.array(e, dtype=np.int32), directed)


@functools.lru_cache(maxsize=None)
def want(name):
    g = graph(name)
    return oracle.sums(g.n, g.edges, g.directed)


@pytest.mark.parametrize("name", ["directed", "undirected"])
@pytest.mark.parametrize("width", [32, 64, 128, 256])
@pytest.mark.parametrize("force", ["pull", "push", "default"])
def test_items(ctx, name, width, force):
    g = graph(name)
    S, r = want(name)
    keep = ctx.tuning()
    dg = tkc.Graph.from_graphgen(ctx, g, validate=True)
    try:
        ctx.tune(batch_width=width)
        if force == "pull":
            ctx.tune(batch_alpha=1 << 30, bu_td_beta=1 << 30)
        elif force == "push":
            ctx.tune(bu_td_beta=1, batch_alpha=1)
        print("items", name, width, force, flush=True)
        src = np.concatenate([np.arange(0, g.n, 3), [5, 5, 800, 800]]).astype(np.int32)
        S2, r2 = dg.sums(src)
        assert np.array_equal(S2, S[src]) and np.array_equal(r2, r[src])
        ids, S3, r3, _, _ = tkc.topk_closeness(dg, 25, "nbcut", "batched")
        wi, wS, wr, _ = oracle.closeness_topk(g.n, g.edges, g.directed, 25)
        assert np.array_equal(ids, wi) and np.array_equal(S3, wS) and np.array_equal(r3, wr)
    finally:
        ctx.tune(**keep)
        dg.free()


@pytest.mark.parametrize("groups", [8, 23, 24, 25, 31, 64, 255, 256, 257])
def test_grid_barrier_widths(ctx, groups):
    """512 vertices of a tree to a workgroup: launches around the width from
    which a grid barrier goes by XCD, narrow and wide ones in turn."""
    gs = []
    for k in (groups, 8, 40):
        n = 512 * k
        g = graphgen.make("tree", n, graphgen.tree(n, k), False)
        src = np.arange(0, n, n // 150 + 1, dtype=np.int32)
        gs.append((tkc.Graph.from_graphgen(ctx, g), src, oracle.sums(n, g.edges, False, sources=src)))
    for turn in range(3):
        for dg, src, (S, r) in gs:
            print("barrier", groups, turn, dg.n, flush=True)
            S2, r2 = dg.sums(src)
            assert np.array_equal(S2, S) and np.array_equal(r2, r)
    for dg, _, _ in gs:
        dg.free()
