"""Level-based bounds after batches whose searches were all cut, at once or in
part: such a batch raises no bound and may have set nothing, and what follows
(batches that do raise, complete searches, packs) finds a clean workspace.
Answers equal the oracle's."""
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


def streets_and_hub(directed, n=6000, seed=17):
    """A hub over 3,000 vertices, a long street, a random part, lone vertices."""
    r = np.random.default_rng(seed)
    st = np.arange(3000, 3200)
    e = [np.stack([np.zeros(2999, np.int64), np.arange(1, 3000)], 1), r.integers(0, 3000, (5000, 2)),
         np.stack([st[:-1], st[1:]], 1), r.integers(3200, 5800, (9000, 2)), np.array([[7, 3000]])]
    if directed:
        e.append(np.stack([np.arange(1, 2990), np.zeros(2989, np.int64)], 1))
    e = np.concatenate(e)
    e = e[e[:, 0] != e[:, 1]]
    if not directed:
        e = np.sort(e, axis=1)
    return graphgen.make("cutlb", n, np.unique(e, axis=0).astype(np.int32), directed)


@pytest.mark.parametrize("width", [32, 64, 256])
@pytest.mark.parametrize("directed", [False, True])
def test_level_bounds_after_cut_batches(ctx, directed, width):
    g = streets_and_hub(directed)
    src = np.random.default_rng(5).choice(g.n, 200, replace=False).astype(np.int32)
    S, r = oracle.sums(g.n, g.edges, directed, sources=src)
    keep = ctx.tuning()
    ctx.tune(batch_width=width)
    try:
        dg = tkc.Graph.from_graphgen(ctx, g)
        for k in (1, 25):
            want = oracle.closeness_topk(g.n, g.edges, directed, k)
            for variant in ("degcutlb", "degcut", "nbcutlb", "nbbound", "degcutlb"):
                print("cut, then bounds", directed, width, k, variant, flush=True)
                got = tkc.topk_closeness(dg, k, variant, "batched")
                for x, y in zip(got[:4], want):
                    assert np.array_equal(x, y)
                S2, r2 = dg.sums(src)
                assert np.array_equal(S2, S) and np.array_equal(r2, r)
        dg.free()
    finally:
        ctx.tune(**keep)
