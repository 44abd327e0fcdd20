"""Results placed in the top k by a whole wave, list lengths around its 64
lanes: every engine's top k, and all ties, equal the oracle's."""
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
def graph(kind):
    if kind == "grid":   # the ring engine's
        g = graphgen.grid_graph(34, 0.08, 3, seed=6)
    elif kind == "king":   # many ties, the batched and per-workgroup engines'
        g = graphgen.grid_graph(33, 0.0, 0, seed=1, king=True)
        e = np.concatenate([g.edges, np.stack([np.zeros(70, np.int64), np.arange(g.n, g.n + 70)], 1)])
        g = graphgen.make(kind, g.n + 70, e.astype(np.int32), False)
    else:
        g = graphgen.rmat_graph(10, 6, 4)
    return g, oracle.closeness_topk(g.n, g.edges, g.directed, g.n)


@pytest.mark.parametrize("mode", ["batched", "hybrid", "plain"])
@pytest.mark.parametrize("kind", ["grid", "king", "web"])
def test_insert(ctx, kind, mode):
    g, want = graph(kind)
    dg = tkc.Graph.from_graphgen(ctx, g)
    for k in (1, 2, 63, 64, 65, 127, 128, 129, 257, 300, 1000, g.n):
        for variant in ("nbcut", "degcut"):
            print("insert", kind, mode, k, variant, flush=True)
            got = tkc.topk_closeness(dg, k, variant, mode)
            for x, y in zip(got[:4], want):
                assert np.array_equal(x, y[:k])
    for k in (1, 64, 65, 300):
        got = tkc.topk_closeness_ties(dg, k, "nbcut", mode)
        n_ties = len(got[0])
        assert n_ties >= k and (n_ties == g.n or want[3][n_ties] > want[3][k - 1])
        for x, y in zip(got[:4], want):
            assert np.array_equal(x, y[:n_ties])
    dg.free()
