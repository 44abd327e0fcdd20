"""A server's slot holds what its requests need: the search that measures a
packed street network's depth does not carry an earlier request's level tables
(128 bytes a vertex) over to the larger graph.  And a sliced ring launch that
ends in a search deeper than its level tables."""
import numpy as np
import pytest

import graphgen
import oracle
from conftest import hip_available

pytestmark = pytest.mark.gpu

if hip_available():
    import torch

    from paper_1704_01077_amd import tkc
else:
    tkc = None


@pytest.fixture(scope="module")
def ctx():
    if not hip_available():
        pytest.skip("no GPU")
    torch.cuda.init()
    c = tkc.Context(0)
    yield c
    c.close()


def free_bytes():
    torch.cuda.synchronize()
    return torch.cuda.mem_get_info()[0]


def test_probe_takes_the_request_s_room(ctx):
    small = graphgen.grid_graph(20, 0.05, 3, seed=2)
    large = graphgen.grid_graph(560, 0.05, 30, seed=4)
    used, got = [], []
    for first in (False, True):
        dgs = [tkc.Graph.from_graphgen(ctx, g) for g in (small, large)]
        s = tkc.Server(ctx, 8 << 30, 1)
        ids = [s.add(d) for d in dgs]
        s.enable_packing(1 << 20)
        before = free_bytes()
        if first:
            print("small, level bounds", flush=True)
            r = s.result(s.submit(ids[0], 3, "nbbound"), 3)
            for x, y in zip(r[:4], oracle.closeness_topk(small.n, small.edges, False, 3)):
                assert np.array_equal(x, y)
        print("large", first, flush=True)
        got.append(s.result(s.submit(ids[1], 3, "nbcut"), 3))
        used.append(before - free_bytes())
        s.close()
        for d in dgs:
            d.free()
    for x, y in zip(got[0][:4], got[1][:4]):
        assert np.array_equal(x, y)
    # (128 bytes a vertex would be 40 MB)
    assert used[1] <= used[0] + (16 << 20), used


def test_slices_end_in_a_deep_search(ctx):
    """A path of 12,001 vertices: every search is deeper than 8,192 levels from
    its first thousands of vertices on.  The middle is closest, S = 2 (1 + ... +
    6,000)."""
    h = 6000
    n = 2 * h + 1
    e = np.stack([np.arange(n - 1), np.arange(1, n)], 1).astype(np.int32)
    dg = tkc.Graph.from_graphgen(ctx, graphgen.make("path", n, e, False))
    s = tkc.Server(ctx, 1 << 30, 2)
    gid = s.add(dg)
    d = np.array([0, 1, 1, 2, 2])
    want = h * (h + 1) + d * d
    for t in [s.submit(gid, 5, variant) for variant in ("nbbound", "nbcut")]:
        print("deep slices", flush=True)
        ids, S, r, F = s.result(t, 5)[:4]
        assert np.array_equal(S, want) and np.all(r == n)
        assert np.array_equal(np.sort(ids), np.arange(h - 2, h + 3)) and ids[0] == h
    s.close()
    dg.free()
