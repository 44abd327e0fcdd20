"""Graphs of different kinds asked in turn on one context: after each was asked
once, the workspace holds what all of them need and no call allocates.  And
servers whose budget leaves no room for the ring engine's buffers answer alike
and stay within it."""
import re

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


def test_streets_and_social_in_turn(ctx):
    """A street network (the ring engine's) between a smaller one and a larger
    social network: the second round allocates and frees nothing."""
    gs = [graphgen.grid_graph(70, 0.05, 3, seed=1), graphgen.ba_graph(100000, 4, 2),
          graphgen.grid_graph(40, 0.05, 1, seed=3)]
    dgs = [tkc.Graph.from_graphgen(ctx, g) for g in gs]
    want, seen = {}, []
    for rnd in range(3):
        for i in (0, 1, 2, 1):
            print("in turn", rnd, i, flush=True)
            got = tkc.topk_closeness(dgs[i], 5, "nbcut", "batched")
            assert got[4]["main_kernel"] == (1 if i == 1 else 2)
            for x, y in zip(got[:4], want.setdefault(i, got[:4])):
                assert np.array_equal(x, y)
            if rnd:
                seen.append(free_bytes())
    assert len(set(seen)) == 1, seen
    for i in (0, 2):
        for x, y in zip(want[i], oracle.closeness_topk(gs[i].n, gs[i].edges, False, 5)):
            assert np.array_equal(x, y)
    for d in dgs:
        d.free()


@pytest.mark.parametrize("variant", ["nbcut", "nbbound"])
def test_server_without_ring_buffers(ctx, variant):
    """A budget of the request's workspace alone: the ring engine's buffers
    (over 50 MB for this graph) are left out, the batched engine answers."""
    g = graphgen.grid_graph(180, 0.05, 10, seed=5)
    dg = tkc.Graph.from_graphgen(ctx, g)
    want = tkc.topk_closeness(dg, 5, variant, "batched")
    assert want[4]["main_kernel"] == 2
    s = tkc.Server(ctx, 1, 1)
    gid = s.add(dg)
    with pytest.raises(tkc.TkcError) as e:
        s.submit(gid, 5, variant)
    need = int(re.search(r"needs (\d+) bytes", str(e.value)).group(1))
    s.close()
    s = tkc.Server(ctx, need, 1)
    gid = s.add(dg)
    before = free_bytes()
    for _ in range(2):
        got = s.result(s.submit(gid, 5, variant), 5)
        for x, y in zip(got[:4], want[:4]):
            assert np.array_equal(x, y)
    # (the graph's cached preprocessing, 44 bytes a vertex, is not the slots')
    assert before - free_bytes() <= need + 44 * g.n + (16 << 20)
    s.close()
    # with room for them it runs in slices of the ring engine
    s = tkc.Server(ctx, 1 << 30, 1)
    gid = s.add(dg)
    got = s.result(s.submit(gid, 5, variant), 5)
    for x, y in zip(got[:4], want[:4]):
        assert np.array_equal(x, y)
    s.close()
    dg.free()
