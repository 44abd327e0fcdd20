"""NB bounds of hubs whose chunks' sums are added by a whole wave: chunk counts
around multiples of 64, and walk counts that reach the cap of 2^62 (a clique
and a path behind the hub keep the rounds going): equal to the oracle's, twice
on one workspace."""
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

CHUNK = 512


@pytest.fixture(scope="module")
def ctx():
    if not hip_available():
        pytest.skip("no GPU")
    import torch
    torch.cuda.init()
    c = tkc.Context(0)
    yield c
    c.close()


def hub_graph(deg, directed, deep):
    r = np.random.default_rng(deg)
    n = deg + 1
    e = [np.stack([np.zeros(deg, np.int64), np.arange(1, deg + 1)], 1), r.integers(1, n, (3000, 2))]
    if deep:   # the first 40 vertices a clique, a path of 40 from vertex 1
        i, j = np.triu_indices(40, 1)
        e.append(np.stack([i, j], 1))
        p = np.concatenate([[1], np.arange(n, n + 40)])
        e.append(np.stack([p[:-1], p[1:]], 1))
        n += 40
    e = np.concatenate(e)
    if directed:
        e = np.concatenate([e, e[r.random(len(e)) < 0.5][:, ::-1]])
    e = e[e[:, 0] != e[:, 1]]
    if not directed:
        e = np.sort(e, axis=1)
    return graphgen.make("hub", n, np.unique(e, axis=0).astype(np.int32), directed)


@pytest.mark.parametrize("directed", [True, False])
@pytest.mark.parametrize("deg,deep", [(63 * CHUNK, False), (64 * CHUNK, True), (64 * CHUNK + 1, False),
                                      (128 * CHUNK + 1, True), (200 * CHUNK - 1, False)])
def test_nb_hub(ctx, deg, deep, directed):
    g = hub_graph(deg, directed, deep)
    assert int(g.row_ptr[1] - g.row_ptr[0]) == deg
    dg = tkc.Graph.from_graphgen(ctx, g)
    a, o, _ = oracle.reach_bounds(g.n, g.edges, g.directed)
    wn, wd = oracle.nb(g.n, g.edges, g.directed, a, o)
    for turn in range(2):
        print("nb hub", deg, deep, directed, turn, flush=True)
        num, den, _ = dg.bounds("nbcut")
        assert np.array_equal(den == 0, np.asarray(wd) == 0)
        for v in np.flatnonzero(den):
            assert int(num[v]) * int(wd[v]) == int(wn[v]) * int(den[v])
    dg.free()
