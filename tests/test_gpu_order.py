"""The processing order around the size up to which one workgroup sorts it:
keys in ascending order, equal keys by ascending id, keys that agree on whole
digits included."""
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


@pytest.mark.parametrize("kind", ["cycle", "star", "random"])
@pytest.mark.parametrize("n", [2, 3, 63, 64, 65, 255, 257, 1023, 2049, 4095, 4096, 4097, 6145])
def test_degree_order(ctx, n, kind):
    r = np.random.default_rng(n)
    if kind == "cycle":
        e = np.stack([np.arange(n), (np.arange(n) + 1) % n], 1)
    elif kind == "star":
        e = np.stack([np.full(n - 1, n // 2), np.delete(np.arange(n), n // 2)], 1)
    else:
        e = np.stack([r.integers(0, n, 4 * n), (n * r.random(4 * n) ** 3).astype(np.int64)], 1)
    e = np.unique(np.sort(e[e[:, 0] != e[:, 1]], axis=1), axis=0).astype(np.int32)
    g = graphgen.make(kind, n, e, False)
    deg = np.diff(g.row_ptr)
    dg = tkc.Graph.from_graphgen(ctx, g)
    print("order", n, kind, flush=True)
    order = np.asarray(dg.bounds("degcut")[2])
    # a lone vertex (its bound is infinite) comes last
    assert np.array_equal(order, np.lexsort((np.arange(n), np.where(deg == 0, 1, -deg.astype(np.int64)))))
    for variant in ("nbcut", "degcut"):
        got = tkc.topk_closeness(dg, min(n, 9), variant, "batched")
        if n <= 2049:
            want = oracle.closeness_topk(n, g.edges, False, min(n, 9))
            assert all(np.array_equal(a, b) for a, b in zip(got[:4], want))
    dg.free()
