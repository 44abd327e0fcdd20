"""Upload on both sides of the line between tables laid out on the host and by
kernels (4 n + arcs against 2^18): graphs just below, at and above it, with long
rows and empty ones, from host arrays, device tensors and renumbered; the same
refusals with the same words on both sides."""
import numpy as np
import pytest

import graphgen
import oracle
from conftest import hip_available

pytestmark = pytest.mark.gpu
LINE = 1 << 18

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


def graph(n, over, directed):
    """Rows of 1,500 and more arcs, empty rows, and 4 n + arcs = LINE + over
    (both CSRs of a directed graph counted; each edge is two arcs either way)."""
    r = np.random.default_rng(n)
    want = (LINE + over - 4 * n) // 2
    e = [np.stack([np.full(1500, u), n // 4 + np.arange(1500)], 1) for u in (0, n // 2, n - 1)]
    e.append(r.integers(0, n, (3 * want, 2)))
    e = np.concatenate(e)
    e = e[(e[:, 0] != e[:, 1]) & ((e[:, 0] % 5 != 3) & (e[:, 1] % 5 != 3) | (np.arange(len(e)) < 4500))]
    if not directed:
        e = np.sort(e, axis=1)
    keys = e[:, 0] * n + e[:, 1]
    _, first = np.unique(keys, return_index=True)
    e = e[np.sort(first)[:want]]
    assert len(e) == want
    return graphgen.make("line", n, e.astype(np.int32), directed)


def arrays(g):
    return [np.ascontiguousarray(a) for a in (g.row_ptr, g.col_idx, g.rrow_ptr, g.rcol_idx) if a is not None]


@pytest.mark.parametrize("directed", [True, False])
@pytest.mark.parametrize("n,over", [(6000, -2), (6000, 0), (6000, 2), (30001, 0), (30001, 4), (7001, 60000)])
def test_both_sides_of_the_line(ctx, n, over, directed):
    import torch
    g = graph(n, over, directed)
    src = np.concatenate([[0, n // 2, n - 1], np.random.default_rng(1).choice(n, 90, replace=False)]).astype(np.int32)
    S, r = oracle.sums(g.n, g.edges, directed, sources=src)
    want = oracle.closeness_topk(g.n, g.edges, directed, 8)
    keep = ctx.tuning()
    try:
        for kw in ({}, {"validate": True}, {"relabel": True}):
            for dev in (False, True):
                print("line", n, over, directed, dev, kw, flush=True)
                a = [torch.as_tensor(x, device="cuda") for x in arrays(g)] if dev else arrays(g)
                dg = tkc.Graph.from_csr(ctx, *a, **kw)
                del a
                for width in (32, 256):
                    ctx.tune(batch_width=width)
                    if "relabel" not in kw:   # (sums are not offered for those)
                        S2, r2 = dg.sums(src)
                        assert np.array_equal(S2, S) and np.array_equal(r2, r)
                    got = tkc.topk_closeness(dg, 8, "nbcut", "batched")
                    for x, y in zip(got[:4], want):
                        assert np.array_equal(x, y)
                dg.free()
    finally:
        ctx.tune(**keep)


@pytest.mark.parametrize("over", [0, 2])
@pytest.mark.parametrize("dev", [False, True])
def test_refusals_on_both_sides(ctx, over, dev):
    import torch
    g = graph(6000, over, True)

    def refused(side, which, at, value, words):
        a = [x.copy() for x in arrays(g)]
        a[2 * side + which][at] = value
        if dev:
            a = [torch.as_tensor(x, device="cuda") for x in a]
        with pytest.raises(tkc.TkcError, match=words):
            tkc.Graph.from_csr(ctx, *a)

    for side, name in ((0, "out-arcs"), (1, "in-arcs")):
        m = len(g.col_idx)
        refused(side, 0, 0, 1, name + r": row_ptr\[0\] must be 0")
        refused(side, 0, 6000, m - 1, name + r": row_ptr\[n\] != m_arcs")
        refused(side, 0, 4000, m + 5, name + ": row_ptr not monotone at 4000")
        refused(side, 1, m - 1, 6000, name + ": vertex id out of range")
        refused(side, 1, 0, -1, name + ": vertex id out of range")
