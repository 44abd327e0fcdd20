"""Graphs uploaded unchecked with loops (arcs from a vertex to itself) and
repeated arcs: no search may count its source twice, so sums and top k equal
the oracle's on the graph without them."""
import numpy as np
import pytest

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


def csr(n, src, dst):
    order = np.argsort(src, kind="stable")
    rp = np.concatenate([[0], np.cumsum(np.bincount(src, minlength=n))])
    return rp.astype(np.int32), dst[order].astype(np.int32)


@pytest.mark.parametrize("width", [64, 256])
@pytest.mark.parametrize("directed", [False, True])
def test_loops(ctx, directed, width):
    n, r = 700, np.random.default_rng(21)
    e = r.integers(0, n, (3 * n, 2))
    e = np.concatenate([e, np.stack([np.zeros(100, np.int64), np.arange(1, 101)], 1)])   # a heavy vertex
    e = e[e[:, 0] != e[:, 1]]
    if not directed:
        e = np.sort(e, axis=1)
    e = np.unique(e, axis=0)
    arcs = e if directed else np.concatenate([e, e[:, ::-1]])
    loops = np.repeat(np.arange(0, n, 2), 2).reshape(-1, 2)
    arcs = np.concatenate([arcs, loops, arcs[:0 if not directed else 50]])
    rp, ci = csr(n, arcs[:, 0], arcs[:, 1])
    rev = csr(n, arcs[:, 1], arcs[:, 0]) if directed else (None, None)
    S, reach = oracle.sums(n, e.astype(np.int32), directed)
    want = oracle.closeness_topk(n, e.astype(np.int32), directed, 10)
    keep = ctx.tuning()
    ctx.tune(batch_width=width)
    try:
        dg = tkc.Graph.from_csr(ctx, rp, ci, *rev)
        S2, r2 = dg.sums(np.arange(n, dtype=np.int32))
        assert np.array_equal(S2, S) and np.array_equal(r2, reach)
        for mode in ("batched", "hybrid", "plain"):
            got = tkc.topk_closeness(dg, 10, "degcut", mode)
            for x, y in zip(got[:4], want):
                assert np.array_equal(x, y)
        dg.free()
    finally:
        ctx.tune(**keep)
