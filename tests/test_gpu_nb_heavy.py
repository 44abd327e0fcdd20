"""NB bounds with vertices of one, two and several 512-arc chunks, whose last
chunk finishes them: equal to the oracle's, twice on one workspace."""
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


@pytest.mark.parametrize("directed", [True, False])
@pytest.mark.parametrize("hub", [64, 65, 511, 512, 513, 1024, 1025, 2600])
def test_nb_chunks(ctx, hub, directed):
    n = 3000
    r = np.random.default_rng(hub)
    e = [r.integers(0, n, (n, 2))]
    for u in (0, 1700, n - 1):
        w = r.permutation(n)[:hub]
        e.append(np.stack([np.full(hub, u), w], 1))
    e = np.concatenate(e)
    e = e[e[:, 0] != e[:, 1]]
    if not directed:
        e = np.sort(e, axis=1)
    g = graphgen.make("nb", n, np.unique(e, axis=0).astype(np.int32), directed)
    dg = tkc.Graph.from_graphgen(ctx, g)
    a, o, _ = oracle.reach_bounds(g.n, g.edges, g.directed)
    wn, wd = oracle.nb(g.n, g.edges, g.directed, a, o)
    for turn in range(2):
        print("nb", hub, directed, turn, flush=True)
        num, den, _ = dg.bounds("nbcut")
        assert np.array_equal(den == 0, np.asarray(wd) == 0)
        for v in np.flatnonzero(den):
            assert int(num[v]) * int(wd[v]) == int(wn[v]) * int(den[v])
    dg.free()
