"""The pivot's two searches (pieces of rows, push and pull levels, both
directions at once) against the oracle's components and bounds: hubs around
the size of a piece, searches of around the levels launched at a time, both."""
import numpy as np
import pytest

import graphgen
from conftest import hip_available
from test_gpu_reach import check

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


@pytest.mark.parametrize("extra", [0, 4000])
@pytest.mark.parametrize("depth", [1, 7, 8, 9, 70])
@pytest.mark.parametrize("hub", [1, 255, 256, 257, 513])
def test_hub_and_ring(ctx, hub, depth, extra):
    """Vertex 0 with `hub` leaves both ways, on a cycle of depth + 1 vertices
    (one component), with arcs from and to it, and `extra` vertices around
    that make its frontiers a small part of the graph."""
    n0 = 1 + hub + depth
    e = [(0, i) for i in range(1, hub + 1)] + [(i, 0) for i in range(1, hub + 1)]
    ring = [0] + list(range(hub + 1, n0))
    e += [(ring[i], ring[(i + 1) % len(ring)]) for i in range(len(ring))]
    for i in range(extra):    # in-side vertices reach the component, out-side ones it reaches
        e.append((n0 + i, i % n0) if i % 2 else (i % n0, n0 + i))
    e = np.unique(np.array([x for x in e if x[0] != x[1]], dtype=np.int32), axis=0)
    g = graphgen.make("hub", n0 + extra, e, True)
    dg = tkc.Graph.from_graphgen(ctx, g)
    print("hub", hub, depth, extra, flush=True)
    a, o, sc = dg.reach()
    check(g, a, o, sc)
    assert dg.reach_info()[0] == 1
    dg.free()
