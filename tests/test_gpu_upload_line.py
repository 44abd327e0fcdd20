"""Upload on both sides of the lines between tables laid out on the host and by
kernels (4 n + arcs against 2^18 for host arrays, 5 2^15 for device tensors): graphs just below, at and above it, with long
rows and empty ones, from host arrays, device tensors and renumbered; the same
refusals with the same words on both sides."""
import numpy as np
import pytest

import graphgen
import oracle
from conftest import hip_available

pytestmark = pytest.mark.gpu
LINE = 1 << 18
DEV = (5 << 15) - LINE

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
@pytest.mark.parametrize("n,over", [(6000, DEV), (6000, DEV + 2), (6000, -2), (6000, 0), (6000, 2), (30001, 0), (30001, 4),
                                    (7001, 60000)])
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


@pytest.mark.parametrize("over", [DEV, DEV + 2, 0, 2])
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


def crowd(n, directed):
    """Most of the first 700 vertices have 60 to 400 arcs, some 2,048 (4 chunks),
    2,049 (5) and 33,000 (65 chunks, and pieces beyond a wave's lanes); then rows
    just below, at and above a pull item's 256 arcs; large enough for the kernels."""
    r = np.random.default_rng(n)
    deg = np.full(n, 1, np.int64)
    deg[:700] = r.integers(60, 400, 700)
    deg[[3, 63, 64, 511, 512, 640]] = [33000, 2048, 2049, 20000, 0, 513]
    deg[n - 700:n - 500] = r.integers(255, 258, 200)
    deg[-1] = 65
    deg[5000:5300] = 0
    src = np.repeat(np.arange(n), deg)
    first = np.concatenate([[0], np.cumsum(deg)])[:-1]
    dst = (r.integers(0, n, n)[src] + (np.arange(len(src)) - first[src])) % n   # consecutive, no repeats
    e = np.stack([src, dst], 1)[src != dst]
    if not directed:
        e = np.unique(np.sort(e, axis=1), axis=0)
    return graphgen.make("crowd", n, e.astype(np.int32), directed)


@pytest.mark.parametrize("directed", [True, False])
@pytest.mark.parametrize("n", [65537, 66000])
def test_crowded_rows_by_kernels(ctx, n, directed):
    import torch
    g = crowd(n, directed)
    assert 4 * n + len(g.col_idx) > LINE
    src = np.concatenate([[0, 3, 63, 64, 511, 512, n - 1], np.random.default_rng(2).choice(n, 57)]).astype(np.int32)
    S, r = oracle.sums(g.n, g.edges, directed, sources=src)
    keep = ctx.tuning()
    try:
        for dev in (False, True):
            a = [torch.as_tensor(x, device="cuda") for x in arrays(g)] if dev else arrays(g)
            dg = tkc.Graph.from_csr(ctx, *a)
            del a
            for width, alpha, beta in ((64, 1, 1), (64, 1 << 30, 1 << 30), (256, 14, 24)):   # push, pull, default
                print("crowd", n, directed, dev, width, alpha, flush=True)
                ctx.tune(batch_width=width, batch_alpha=alpha, bu_td_beta=beta)
                S2, r2 = dg.sums(src)
                assert np.array_equal(S2, S) and np.array_equal(r2, r)
            dg.free()
    finally:
        ctx.tune(**keep)
