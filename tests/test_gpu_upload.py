"""Upload: the device's checks and tables for host arrays and device tensors,
at widths around the tables' spans and runs, with rows around the pieces they
are split into, against the oracle; what is refused is refused either way."""
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


def _graph(n, hub, directed):
    """Random arcs, empty rows, and rows of `hub` arcs at the ends and the middle."""
    r = np.random.default_rng(n + hub)
    e = [r.integers(0, n, (2 * n, 2))]
    for u in {0, n // 2, n - 1}:
        w = r.permutation(n)[:hub]
        e.append(np.stack([np.full(len(w), u), w], 1))
        if directed:
            e.append(np.stack([w, np.full(len(w), u)], 1))
    e = np.concatenate(e)
    e = e[(e[:, 0] != e[:, 1]) & (e[:, 0] % 5 != 3)]
    if not directed:
        e = np.sort(e, axis=1)
    return graphgen.make("upload", n, np.unique(e, axis=0).astype(np.int32).reshape(-1, 2), directed)


@pytest.mark.parametrize("directed", [True, False])
@pytest.mark.parametrize("n,hub", [(1, 0), (2, 1), (63, 20), (64, 64), (65, 65), (511, 255), (512, 257), (513, 300),
                                   (1025, 513), (2100, 1030)])
def test_upload_tables(ctx, n, hub, directed):
    import torch
    g = _graph(n, hub, directed)
    S, r = oracle.sums(g.n, g.edges, directed)
    want = oracle.closeness_topk(g.n, g.edges, directed, min(n, 20))
    arrays = [a for a in (g.row_ptr, g.col_idx, g.rrow_ptr, g.rcol_idx) if a is not None]
    for dev in (False, True):
        print("upload", n, hub, directed, dev, flush=True)
        a = [torch.as_tensor(np.ascontiguousarray(x), device="cuda" if dev else "cpu") for x in arrays]
        dg = tkc.Graph.from_csr(ctx, *a)
        del a
        gs, gr = dg.sums(np.arange(n, dtype=np.int32))
        assert np.array_equal(gs, S) and np.array_equal(gr, r)
        got = tkc.topk_closeness(dg, min(n, 20), "nbcut", "batched")
        for x, y in zip(got[:4], want):
            assert np.array_equal(x, y)
        dg.free()


@pytest.mark.parametrize("dev", [False, True])
@pytest.mark.parametrize("side", [0, 1])
def test_upload_refuses(ctx, dev, side):
    import torch
    g = _graph(600, 70, True)
    good = [np.array(x) for x in (g.row_ptr, g.col_idx, g.rrow_ptr, g.rcol_idx)]

    def bad(change, text):
        a = [x.copy() for x in good]
        change(a[2 * side], a[2 * side + 1])
        a = [torch.as_tensor(x, device="cuda" if dev else "cpu") for x in a]
        with pytest.raises(tkc.TkcError) as e:
            tkc.Graph.from_csr(ctx, *a)
        assert e.value.code == tkc.TKC_EINVAL
        assert ("in-arcs" if side else "out-arcs") + ": " + text in str(e.value)

    def at(i, v, ids=False):
        def f(rp, ci):
            (ci if ids else rp)[i] = v
        return f

    bad(at(0, 1), "row_ptr[0] must be 0")
    bad(at(600, len(g.col_idx) + 1), "row_ptr[n] != m_arcs")
    k = int(np.argmax(np.diff(good[2 * side]) > 0))   # a row that is not empty
    bad(at(k + 1, -1), "row_ptr not monotone at %d" % k)
    bad(at(5, 600, True), "vertex id out of range")
    bad(at(-1, -1, True), "vertex id out of range")
