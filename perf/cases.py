"""The work whose speed is watched: whole calls of the public entry points on
graphs of the kinds the library is for.

A case names a kind of graph (``ba``: undirected preferential attachment, a
social network; ``rmat``: directed R-MAT, a web graph; ``road``: an undirected
perturbed grid, a street network), its size and one call on it.  Graphs are
drawn on the GPU from the seed alone.
"""
from __future__ import annotations

import math
from fractions import Fraction

import numpy as np
import torch

from paper_1704_01077_amd import tkc


def listed():
    return [
        # the smallest call: a graph of a few thousand vertices, where
        # launches, host waits and grid barriers are all there is
        dict(name="ba_2k", call="topk", kind="ba", n=2000, deg=5, k=10, variant="auto", mode="hybrid"),
        # the benchmark's social network with the package's default arguments
        dict(name="ba_1m", call="topk", kind="ba", n=1 << 20, deg=5, k=10, variant="auto", mode="hybrid"),
        # a long result list with every tie, on an odd number of vertices
        dict(name="ba_300k_ties", call="ties", kind="ba", n=300007, deg=8, k=100, variant="nbcut", mode="batched"),
        # the benchmark's web graph: directed, renumbered by degree, the
        # widest batches
        dict(name="rmat_1m", call="topk", kind="rmat", n=1 << 20, deg=16, k=10, variant="nbcut", mode="batched",
             width=256, per_cu=4, relabel=True),
        # in-closeness of a smaller web graph, default arguments, own ids
        dict(name="rmat_150k_in", call="topk", kind="rmat", n=150001, deg=8, k=10, variant="auto", mode="hybrid",
             reverse=True),
        # a street network of a country: hundreds of levels per search,
        # level-based bounds
        dict(name="road_1m", call="topk", kind="road", n=1000000, k=10, variant="nbbound", mode="batched",
             width=128),
        # a street network of a town, default arguments: many tiny levels
        dict(name="road_20k", call="topk", kind="road", n=19881, k=10, variant="auto", mode="hybrid"),
        # the other centrality the library ranks by
        dict(name="harmonic_200k", call="harmonic", kind="ba", n=200003, deg=6, k=10, variant="auto",
             mode="batched"),
        # exact sums of chosen vertices: complete searches, nothing cut
        dict(name="sums_260k", call="sums", kind="rmat", n=1 << 18, deg=16, count=500),
        # a graph that is asked once: upload, reachability, bounds, search
        dict(name="once_130k", call="once", kind="rmat", n=1 << 17, deg=16, k=10, variant="nbcut", mode="batched"),
        # small graphs whose requests share one launch
        dict(name="pack_16", call="pack", kind="ba", n=2500, deg=6, k=10, count=16, variant="nbcut"),
        # a resident server: requests of uneven size arriving together
        dict(name="serve_32", call="serve", kind="mixed", n=30000, deg=6, graphs=6, requests=32),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    call = rng.choice(["topk", "topk", "topk", "topk", "ties", "harmonic", "sums", "once", "pack", "serve"])
    if call == "pack":
        return dict(call=call, kind=rng.choice(["ba", "rmat"]), n=_log(rng, 500, 8000), deg=rng.randint(4, 8),
                    k=rng.choice([1, 10, 100]), count=rng.randint(4, 32), variant=rng.choice(["nbcut", "degcut"]))
    if call == "serve":
        return dict(call=call, kind="mixed", n=_log(rng, 3000, 30000), deg=rng.randint(4, 8),
                    graphs=rng.randint(3, 7), requests=rng.randint(8, 32))
    if call == "sums":
        return dict(call=call, kind=rng.choice(["ba", "rmat"]), n=_log(rng, 1000, 500000), deg=rng.randint(4, 16),
                    count=_log(rng, 10, 900))
    if call == "once":
        return dict(call=call, kind=rng.choice(["ba", "rmat"]), n=_log(rng, 1000, 300000), deg=rng.randint(4, 12),
                    k=rng.choice([1, 10, 100]), variant="nbcut", mode=rng.choice(["batched", "hybrid"]))
    if call == "harmonic":
        return dict(call=call, kind=rng.choice(["ba", "rmat"]), n=_log(rng, 1000, 300000), deg=rng.randint(4, 10),
                    k=rng.choice([1, 10, 100]), variant="nbcut", mode=rng.choice(["batched", "hybrid"]))
    kind = rng.choice(["ba", "ba", "rmat", "road"]) if call == "topk" else "ba"
    if kind == "road":
        return dict(call=call, kind=kind, n=_log(rng, 1500, 250000), k=rng.choice([1, 10]),
                    variant=rng.choice(["auto", "nbbound", "nbcutlb"]), mode=rng.choice(["batched", "hybrid"]),
                    width=rng.choice([64, 128]))
    c = dict(call=call, kind=kind, n=_log(rng, 1000, 1000000), deg=rng.randint(3, 10), k=rng.choice([1, 10, 100]),
             variant=rng.choice(["auto", "nbcut"]), mode=rng.choice(["batched", "hybrid"]))
    if c["n"] < 4000 and rng.random() < 0.5:
        c["mode"] = "plain"
    if kind == "rmat":
        c.update(width=rng.choice([64, 128, 256]), relabel=rng.random() < 0.5, reverse=rng.random() < 0.3)
    return c


# ------------------------------------------------------------------ graphs
def _rng(seed, salt=0):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed) * 1000003 + salt * 7919 + 17)
    return g


def _csr(n, src, dst):
    """CSR of the distinct arcs src -> dst without loops, rows sorted."""
    keep = src != dst
    key = torch.unique(src[keep] * n + dst[keep])
    rp = torch.zeros(n + 1, dtype=torch.int64, device="cuda")
    rp[1:] = torch.cumsum(torch.bincount(key // n, minlength=n), 0)
    return rp.to(torch.int32), (key % n).to(torch.int32)


def _ba(n, m, g):
    """Preferential attachment: every new vertex draws m earlier edge ends."""
    e = torch.arange((n - m - 1) * m, device="cuda")
    ci, cj = torch.triu_indices(m + 1, m + 1, 1, device="cuda")
    ne = ci.numel() + e.numel()
    own = torch.cat([ci, m + 1 + e // m])
    ends = torch.empty(2 * ne, dtype=torch.int64, device="cuda")
    ends[0::2] = own
    # slot 2q holds edge q's new vertex, slot 2q + 1 a copy of an earlier slot
    ptr = torch.arange(2 * ne, device="cuda")
    u = torch.rand(e.numel(), generator=g, device="cuda", dtype=torch.float64)
    first = 2 * ci.numel()
    ptr[first + 1::2] = (u * (first + 2 * e).to(torch.float64)).to(torch.int64)
    fixed = torch.zeros(2 * ne, dtype=torch.bool, device="cuda")
    fixed[0::2] = True
    fixed[:first] = True
    while True:
        nxt = torch.where(fixed[ptr], ptr, ptr[ptr])
        if torch.equal(nxt, ptr):
            break
        ptr = nxt
    ends[1:first:2] = cj
    ends = ends[ptr]
    a, b = ends[0::2], ends[1::2]
    return torch.cat([a, b]), torch.cat([b, a])


def _rmat(n, ef, g):
    """R-MAT arcs with (a, b, c, d) = (.57, .19, .19, .05), ids permuted."""
    scale = max(1, (n - 1).bit_length())
    m = n * ef
    src = torch.zeros(m, dtype=torch.int64, device="cuda")
    dst = torch.zeros(m, dtype=torch.int64, device="cuda")
    for _ in range(scale):
        u = torch.rand(m, generator=g, device="cuda")
        src = 2 * src + (u >= 0.76).to(torch.int64)
        dst = 2 * dst + (((u >= 0.57) & (u < 0.76)) | (u >= 0.95)).to(torch.int64)
    ok = (src < n) & (dst < n)
    perm = torch.randperm(n, generator=g, device="cuda")
    return perm[src[ok]], perm[dst[ok]]


def _road(n, g):
    """Grid of about n crossings, 5 % of its streets deleted, one shortcut for
    4,000 crossings, restricted to its largest connected part."""
    rows = max(4, int(math.isqrt(n)))
    cols = max(4, n // rows)
    n = rows * cols
    v = torch.arange(n, device="cuda")
    right, down = v[v % cols < cols - 1], v[v < n - cols]
    a = torch.cat([right, down])
    b = torch.cat([right + 1, down + cols])
    keep = torch.rand(a.numel(), generator=g, device="cuda") >= 0.05
    extra = torch.randint(0, n, (2, max(1, -(-n // 4000))), generator=g, device="cuda")
    a, b = torch.cat([a[keep], extra[0]]), torch.cat([b[keep], extra[1]])
    lab = v.clone()
    while True:   # smallest id of each part: hook onto neighbours' labels, then jump
        nl = lab.clone()
        low = torch.minimum(lab[a], lab[b])
        nl.scatter_reduce_(0, lab[a], low, "amin")
        nl.scatter_reduce_(0, lab[b], low, "amin")
        nl = nl[nl]
        nl = nl[nl]
        if torch.equal(nl, lab):
            break
        lab = nl
    inside = lab == torch.mode(lab[torch.linspace(0, n - 1, 257, device="cuda").to(torch.int64)]).values
    new = torch.cumsum(inside.to(torch.int64), 0) - 1
    both = inside[a] & inside[b]
    a, b = new[a[both]], new[b[both]]
    return int(inside.sum()), torch.cat([a, b]), torch.cat([b, a])


def _arrays(kind, n, deg, g):
    """(n, row_ptr, col_idx, reverse row_ptr, reverse col_idx) on the GPU."""
    if kind == "road":
        n, a, b = _road(n, g)
    else:
        a, b = _ba(n, deg, g) if kind == "ba" else _rmat(n, deg, g)
    rp, ci = _csr(n, a, b)
    if kind == "rmat":
        rrp, rci = _csr(n, b, a)
        return n, rp, ci, rrp, rci
    return n, rp, ci, None, None


def _members(case, seed):
    """The graphs of a case, as arrays (several for packs and servers)."""
    kind, n, deg = case["kind"], case["n"], case.get("deg", 0)
    if case["call"] == "pack":
        # sizes within a factor of four around n, none alike
        return [_arrays(kind, max(64, int(n * 2.0 ** (2.0 * i / case["count"] - 1))) + i, deg, _rng(seed, i))
                for i in range(case["count"])]
    if case["call"] == "serve":
        # every kind in turn, sizes falling from 2 n by factors of two
        return [_arrays(("ba", "rmat", "road")[i % 3], max(1000, int(2 * n / 2.0 ** i)) + i, deg, _rng(seed, i))
                for i in range(case["graphs"])]
    return [_arrays(kind, n, deg, _rng(seed))]


class _Held:
    """What a program keeps between calls; freed in the order the library asks for."""

    def __init__(self):
        self.ctx = tkc.Context(0)
        self.graphs = []
        self.user = None   # pack or server

    def __del__(self):
        if self.user is not None:
            self.user.close()
        for g in self.graphs:
            g.free()
        self.ctx.close()


def _asked(case):
    """(graph, k) of every request of a server case."""
    return [(i * 5 % case["graphs"], (1, 10, 100)[i // 2 % 3]) for i in range(case["requests"])]


def prepare(case, seed):
    st = _Held()
    if case.get("width"):
        st.ctx.tune(batch_width=case["width"])
    if case.get("per_cu"):
        st.ctx.tune(blocks_per_cu=case["per_cu"])
    st.case = case
    st.arrays = None
    members = _members(case, seed)
    if case["call"] == "once":
        st.arrays = members[0]
        return st
    for n, rp, ci, rrp, rci in members:
        st.graphs.append(tkc.Graph.from_csr(st.ctx, rp, ci, rrp, rci, reverse=bool(case.get("reverse")),
                                            relabel=bool(case.get("relabel"))))
    for g in st.graphs:
        g._keep = None   # the library has its copy
    if case["call"] == "sums":
        st.sources = _sources(case, seed)
    elif case["call"] == "pack":
        st.user = tkc.Pack(st.ctx, st.graphs)
    elif case["call"] == "serve":
        st.user = tkc.Server(st.ctx, 16 << 30, 4)
        st.ids = [st.user.add(g) for g in st.graphs]
        st.user.enable_packing(20000)
        st.asked = _asked(case)
    return st


def _sources(case, seed):
    r = np.random.default_rng(seed)
    return r.choice(case["n"], size=min(case["count"], case["n"]), replace=False).astype(np.int32)


def run(st):
    c = st.case
    call = c["call"]
    if call == "topk":
        return tkc.topk_closeness(st.graphs[0], c["k"], c["variant"], c["mode"])[:4]
    if call == "ties":
        return tkc.topk_closeness_ties(st.graphs[0], c["k"], c["variant"], c["mode"])[:4]
    if call == "harmonic":
        return tkc.topk_harmonic(st.graphs[0], c["k"], c["variant"], c["mode"])[:2]
    if call == "sums":
        return st.graphs[0].sums(st.sources)
    if call == "once":
        g = tkc.Graph.from_csr(st.ctx, *st.arrays[1:])
        out = tkc.topk_closeness(g, c["k"], c["variant"], c["mode"])[:4]
        g.free()
        return out
    if call == "pack":
        members = list(range(c["count"]))
        got = st.user.topk(members, [c["k"]] * len(members), c["variant"])[0]
        return _joined(got)
    tickets = [(st.user.submit(st.ids[i], k), k) for i, k in st.asked]
    return _joined([st.user.result(t, k)[:4] for t, k in tickets])


def _joined(parts):
    return tuple(np.concatenate([p[j] for p in parts]) for j in range(4))


def work(case):
    """The graph read once, the results written once; one addition per arc."""
    def graph(kind, n, deg):
        arcs = {"ba": 2 * n * deg, "rmat": n * deg, "road": 3.8 * n}[kind]
        return (4 * (n + 1) + 4 * arcs) * (2 if kind == "rmat" else 1), arcs

    call, n, deg = case["call"], case["n"], case.get("deg", 0)
    if call == "pack":
        got = [graph(case["kind"], int(n * 2.0 ** (2.0 * i / case["count"] - 1)), deg) for i in range(case["count"])]
        rows = case["count"] * case["k"]
    elif call == "serve":
        sizes = [max(1000, int(2 * n / 2.0 ** i)) for i in range(case["graphs"])]
        got = [graph(("ba", "rmat", "road")[i % 3], sizes[i], deg) for i, _ in _asked(case)]
        rows = sum(k for _, k in _asked(case))
    else:
        got = [graph(case["kind"], n, deg)]
        rows = case["count"] if call == "sums" else case["k"]
    return {"bytes": sum(b for b, _ in got) + 28 * rows, "flops": sum(a for _, a in got)}


# ------------------------------------------------------------------- exact
def _levels(n, rp, ci, sources):
    """counts[d][i]: vertices at distance d from sources[i] (float64), by
    products of the adjacency matrix with the 0/1 frontier."""
    src = torch.repeat_interleave(torch.arange(n, device="cuda"), (rp[1:] - rp[:-1]).to(torch.int64))
    # row w of the transpose: the vertices with an arc to w
    A = torch.sparse_coo_tensor(torch.stack([ci.to(torch.int64), src]),
                                torch.ones(ci.numel(), device="cuda"), (n, n)).to_sparse_csr()
    out = []
    for at in range(0, len(sources), 64):
        s = torch.as_tensor(np.asarray(sources[at:at + 64]), device="cuda", dtype=torch.int64)
        f = torch.zeros(n, s.numel(), device="cuda")
        f[s, torch.arange(s.numel(), device="cuda")] = 1.0
        seen = f > 0
        counts = [torch.ones(s.numel(), dtype=torch.float64, device="cuda")]
        while True:
            f = ((A @ f) > 0) & ~seen
            c = f.sum(0, dtype=torch.float64)
            if not bool((c > 0).any()):
                break
            seen |= f
            f = f.to(torch.float32)
            counts.append(c)
        out.append(torch.stack(counts).cpu().numpy())
    deep = max(c.shape[0] for c in out)
    return np.concatenate([np.pad(c, ((0, deep - c.shape[0]), (0, 0))) for c in out], axis=1)


def _exact_topk(arrays, k, ties=False, harmonic=False):
    n, rp, ci = arrays[:3]
    cnt = _levels(n, rp, ci, np.arange(n))
    d = np.arange(cnt.shape[0], dtype=np.float64)
    if harmonic:
        h = np.zeros(n)
        for q in range(1, cnt.shape[0]):
            h += cnt[q] / d[q]
        ids = np.lexsort((np.arange(n), -h))[: min(k, n)]
        return ids.astype(np.int32), h[ids]
    r = cnt.sum(0).astype(np.int64)
    S = (cnt * d[:, None]).sum(0).astype(np.int64)
    far = [Fraction(int(S[v]), int(r[v] - 1) ** 2) if r[v] > 1 else None for v in range(n)]
    order = sorted(range(n), key=lambda v: (far[v] is None, far[v] or 0, v))
    last = min(k, n)
    while ties and last < n and far[order[last]] == far[order[last - 1]]:
        last += 1
    ids = np.array(order[:last], dtype=np.int32)
    with np.errstate(divide="ignore", invalid="ignore"):
        f = np.where(r[ids] > 1, (float(n - 1) * S[ids].astype(np.float64)) / (r[ids] - 1).astype(np.float64) ** 2,
                     np.inf)
    return ids, S[ids], r[ids], f


def exact(case, seed):
    call = case["call"]
    members = _members(case, seed)
    if call == "sums":
        n, rp, ci = members[0][:3]
        cnt = _levels(n, rp, ci, _sources(case, seed))
        d = np.arange(cnt.shape[0], dtype=np.float64)
        return (cnt * d[:, None]).sum(0).astype(np.int64), cnt.sum(0).astype(np.int64)
    if call == "serve" or case["kind"] == "road" or sum(m[0] ** 2 for m in members) > 1 << 28:
        return None   # all-pairs searches of large graphs take too long here
    if case.get("reverse"):
        members = [(n, rrp, rci, rp, ci) for n, rp, ci, rrp, rci in members]
    if call == "pack":
        return _joined([_exact_topk(m, case["k"]) for m in members])
    return _exact_topk(members[0], case["k"], call == "ties", call == "harmonic")
