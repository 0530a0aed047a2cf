"""Calls at the edges of what the kernels are made for: long runs of empty
rows, ids far apart, work or memory too small for a kernel's preparation."""
import time

import numpy as np
import pytest

import torch

import oracle
import synth
from tests import queries as Q

pytestmark = pytest.mark.gpu


def device_array(ptr, n):
    class A:
        __cuda_array_interface__ = {"shape": (n,), "typestr": "<i4", "data": (ptr, False), "version": 2}
    return torch.as_tensor(A(), device="cuda")


@pytest.mark.parametrize("edges", ["none", "low", "high"])
def test_empty_rows(edges):
    """Row pointers of 2^26 vertices nearly all of which have no edges: 1 GiB
    written and read (0.2 ms at the copy rate), where a single wave would take
    2^20 steps (30 ms or more) a direction."""
    import paper_1802_03760_amd as gj
    n = 1 << 26
    rng = np.random.default_rng(3)
    k = 0 if edges == "none" else 5000
    s, d = (rng.integers(0, 1000, k).astype(np.uint32) for _ in range(2))
    if edges == "high":
        s, d = n - 1 - s, n - 1 - d
    ctx = gj.Context(0, allocator="torch")
    best = 1e9
    for _ in range(5):
        t = time.perf_counter()
        G = gj.Graph(ctx, s, d, n)
        best = min(best, time.perf_counter() - t)
        info = G.info()
        rp = device_array(G.csr_ptrs()[0], n + 1).cpu().numpy()
        G.close()
    pairs = np.unique(s[s != d].astype(np.int64) * n + d[s != d])
    assert info["edges"] == len(pairs)
    v = np.concatenate([np.arange(0, 3000), np.arange(n - 3000, n + 1), rng.integers(0, n, 3000)])
    assert np.array_equal(rp[v], np.searchsorted(pairs // n, v))
    assert best < 12e-3, best


class Bounded:
    """hipMalloc / hipFree as a context's allocator: counts the bytes held, and
    refuses a single allocation above `most` once that is set, or the one
    numbered `fail_at`."""

    def __new__(cls, gj):
        import ctypes
        hip = ctypes.CDLL("libamdhip64.so")

        class A(gj.DeviceAllocator):
            live, most, refused, n, fail_at = {}, None, 0, 0, None

            def alloc(self, nbytes, stream):
                self.n += 1
                if (self.most is not None and nbytes > self.most) or self.n == self.fail_at:
                    self.refused += 1
                    return 0
                p = ctypes.c_void_p()
                if hip.hipMalloc(ctypes.byref(p), ctypes.c_size_t(nbytes)) != 0:
                    return 0
                self.live[p.value] = nbytes
                return p.value

            def free(self, ptr, stream):
                del self.live[ptr]
                hip.hipFree(ctypes.c_void_p(ptr))

            @property
            def held(self):
                return sum(self.live.values())

        a = A()
        a.live = {}
        return a


def same(got, want, tag=""):
    for k in ("matches", "prefixes", "extensions"):
        assert got[k] == want[k], (tag, k, got[k], want[k])


@pytest.mark.parametrize("query", [Q.TRIANGLE, Q.CYCLIC_TRIANGLE, Q.HOUSE])
def test_slice_workspace(query):
    """A slice's count takes no workspace in the size of the whole graph, only
    its frontiers (and what a membership index takes, which is off here)."""
    import paper_1802_03760_amd as gj
    s, d = synth.rmat_draws(16, 12, seed=1)
    A = Bounded(gj)
    ctx = gj.Context(0, allocator=A)
    for k, v in (("run_stage_min", 0), ("hash_index", 0), ("frontier_cap", 1 << 14), ("seed_chunk", 1 << 12)):
        ctx.set_option(k, v)
    G = gj.Graph(ctx, s, d, 1 << 16)
    E = G.info()["edges"]
    before = A.held
    hi = 4000 if query[0] == 3 else 3
    got = gj.count(ctx, G, gj.Query(ctx, *query), 0, hi)
    same(got, oracle.run(oracle.Graph(1 << 16, s, d), query, seed_lo=0, seed_hi=hi, threads=8))
    assert A.held - before < 4 * E, (A.held - before, E)


def test_edge_counts_without_room():
    """The house's last stage counted per edge: an allocation that fails there
    leaves the stage to the kernels it replaces."""
    import paper_1802_03760_amd as gj
    s, d = synth.rmat_draws(9, 12, seed=1)
    want = oracle.run(oracle.Graph(512, s, d), Q.HOUSE, threads=8)

    def run(fail_at):
        A = Bounded(gj)
        ctx = gj.Context(0, allocator=A)
        ctx.set_option("run_stage_min", 0)
        G = gj.Graph(ctx, s, d, 512)
        q = gj.Query(ctx, *Q.HOUSE)
        built = A.n
        A.fail_at = built + fail_at if fail_at else None
        try:
            got = gj.count(ctx, G, q)
        except gj.GJError as e:
            assert e.status == gj.GJ_ENOMEM
            got = None
        last = A.n - built
        if got:
            same(got, want, fail_at)
        same(gj.count(ctx, G, q), want, fail_at)
        q.close(), G.close(), ctx.close()
        assert not A.live
        return got is not None, last

    _, last = run(0)
    through = [run(i)[0] for i in range(1, last + 1)]
    # its workspace: counts, row offsets, word offsets, mask, transposed seeds
    assert sum(through) >= 5, through


def test_listing_workspace():
    """A listing without candidates takes no workspace beyond its frontier's: a
    million edges one way between two sets of vertices, and a star."""
    import paper_1802_03760_amd as gj
    rng = np.random.default_rng(2)
    one_way = rng.integers(0, 1 << 16, 1 << 20), rng.integers(1 << 16, 1 << 17, 1 << 20)
    star = np.zeros(200000, np.int64), np.arange(1, 200001)
    for s, d in (one_way, star):
        A = Bounded(gj)
        ctx = gj.Context(0, allocator=A)
        ctx.set_option("seed_chunk", 1 << 12)
        ctx.set_option("frontier_cap", 1 << 14)
        G = gj.Graph(ctx, s.astype(np.uint32), d.astype(np.uint32), 1 << 18)
        E = G.info()["edges"]
        before = A.held
        for q in (Q.TRIANGLE, Q.CYCLIC_TRIANGLE):
            st, rows = gj.enumerate_rows(ctx, G, gj.Query(ctx, *q), out=np.empty((8, 3), np.uint32))
            assert st["matches"] == 0 and st["prefixes"][2] == E and st["extensions"][2] == 0
        assert A.held - before < 4 * E, (A.held - before, E)


def test_listing_without_room():
    """Whole listings where device memory does not hold the mask pass's
    workspace: the rows all the same."""
    import paper_1802_03760_amd as gj
    s, d = synth.rmat_draws(13, 12, seed=2)
    want = oracle.run(oracle.Graph(1 << 13, s, d), Q.TRIANGLE, collect=True, threads=4)
    A = Bounded(gj)
    ctx = gj.Context(0, allocator=A)
    for k, v in (("seed_chunk", 1 << 12), ("frontier_cap", 1 << 14), ("hash_index", 0)):
        ctx.set_option(k, v)
    G = gj.Graph(ctx, s, d, 1 << 13)
    q = gj.Query(ctx, *Q.TRIANGLE)
    out = torch.zeros((want["matches"], 3), dtype=torch.int32, device="cuda")
    A.most = 4 * G.info()["edges"] - 1  # less than a word per edge
    st, _ = gj.enumerate_rows(ctx, G, q, out=out)
    same(st, want)
    assert np.array_equal(out.cpu().numpy().view(np.uint32), want["rows"])


def held_by_counts(n, s, d, queries, **build):
    """The workspace whole counts leave with their context, results checked."""
    import paper_1802_03760_amd as gj
    A = Bounded(gj)
    ctx = gj.Context(0, allocator=A)
    for k, v in (("hash_index", 0), ("frontier_cap", 1 << 14), ("seed_chunk", 1 << 12)):
        ctx.set_option(k, v)
    s, d = s.astype(np.uint32), d.astype(np.uint32)
    G = gj.Graph(ctx, s, d, n, **build)
    if build:
        s, d, _ = oracle.relabel_by_degree(n, s, d)
    O = oracle.Graph(n, s, d)
    before = A.held
    for q in queries:
        same(gj.count(ctx, G, gj.Query(ctx, *q)), oracle.run(O, q, threads=8), q)
    return A.held - before, G.info()["edges"]


@pytest.mark.parametrize("build", [{}, {"degree_order": True}])
@pytest.mark.parametrize("graph", ["uniform", "rmat"])
def test_cliques_ids_apart(graph, build):
    """20,000 edges among 2^24 ids: no workspace per id."""
    rng = np.random.default_rng(4)
    n = 1 << 24
    if graph == "uniform":
        s, d = rng.integers(0, n, (2, 20000))
    else:
        s, d = (x.astype(np.int64) << 10 for x in synth.rmat_draws(14, 1, seed=3))
    held, E = held_by_counts(n, s, d, [Q.CLIQUE4, Q.CLIQUE5], **build)
    assert held < 4 * n, (held, E)


def test_cliques_uniform_above():
    """20,000 vertices without hubs keep their order: the prefixes and the
    lists, and no renamed copy (32 bytes an edge and 36 a vertex more)."""
    rng = np.random.default_rng(5)
    n = 20000
    held, E = held_by_counts(n, *rng.integers(0, n, (2, 80000)), [Q.CLIQUE4, Q.CLIQUE5])
    assert held < 40 * E, (held, E)


@pytest.mark.parametrize("build", [{}, {"degree_order": True}])
def test_cliques_star(build):
    """Nothing lies two edges deep: no preparation, which takes 32 bytes an edge
    and more."""
    k = 10000 if build else 100000
    for s, d in ((np.zeros(k, int), 1 + np.arange(k)), (1 + np.arange(k), np.zeros(k, int))):
        held, E = held_by_counts(k + 1, s, d, [Q.CLIQUE4, Q.CLIQUE5], **build)
        assert held < 16 * E, (held, E)


@pytest.mark.parametrize("draws", [1, 2, 4])
@pytest.mark.parametrize("scale", [8, 10, 12, 14, 16])
def test_cliques_light(scale, draws):
    """R-MAT graphs on both sides of the lines between the ways to count."""
    s, d = synth.rmat_draws(scale, draws, seed=scale)
    held_by_counts(1 << scale, s, d, [Q.CLIQUE4, Q.CLIQUE5])


def test_cliques_without_room():
    """Whole cliques where device memory does not hold the renamed graph."""
    import paper_1802_03760_amd as gj
    s, d = synth.rmat_draws(12, 16, seed=2)
    O = oracle.Graph(1 << 12, s, d)
    want = [(q, oracle.run(O, q, threads=8)) for q in (Q.CLIQUE4, Q.CLIQUE5)]
    A = Bounded(gj)
    ctx = gj.Context(0, allocator=A)
    ctx.set_option("hash_index", 0)
    G = gj.Graph(ctx, s, d, 1 << 12)
    E = G.info()["edges"]
    A.most = 7 * E  # no 64-bit key per edge; a seed's number per edge fits
    for q, w in want:
        same(gj.count(ctx, G, gj.Query(ctx, *q)), w, q)
    assert A.refused
    before = A.held
    A.most = None
    for q, w in want:
        same(gj.count(ctx, G, gj.Query(ctx, *q)), w, q)
    assert A.held > before + 8 * E  # the refused workspace was not kept


@pytest.mark.parametrize("kind,query", [("diamond", Q.DIAMOND), ("cycle4", Q.CYCLE4)])
def test_twopath_without_room(kind, query):
    """Whole diamonds and 4-cycles where device memory does not hold the renamed
    graph: dense counters (8 bytes an id and worker) count."""
    import paper_1802_03760_amd as gj
    n, m = 4096, 2000000
    rng = np.random.default_rng(6)
    s, d = rng.integers(0, n, (2, m)).astype(np.uint32)
    s[:4000], d[:4000] = 7, 50 + np.arange(4000)  # degrees beyond the small graphs' kernel
    s[4000:8000], d[4000:8000] = 60 + np.arange(4000), 7
    want = oracle.twopath(oracle.Graph(n, s, d), kind, threads=8)
    A = Bounded(gj)
    ctx = gj.Context(0, allocator=A)
    G = gj.Graph(ctx, s, d, n)
    q = gj.Query(ctx, *query)
    A.most = 7 * G.info()["edges"]  # no 64-bit key per edge; 512 workers' counters fit
    same(gj.count(ctx, G, q), want)
    assert A.refused
    A.most = None
    same(gj.count(ctx, G, q), want)


@pytest.mark.parametrize("both", [False, True])
def test_cliques_beyond(both):
    """1,100 vertices each joined to 1,100 of as many edges: left to the
    edge-grouped kernels before the edges are sorted (a renamed copy and its
    prefixes take 60 bytes an edge, the keys to be sorted 16).  Both ways, with
    550 neighbours each, they are few enough to stay."""
    import paper_1802_03760_amd as gj
    k = 550 if both else 1100
    s = np.repeat(np.arange(k), k)
    d = k + np.tile(np.arange(k), k)
    if both:
        s, d = np.concatenate([s, d]), np.concatenate([d, s])
    extra = np.random.default_rng(7).integers(0, 2 * k, (2, 3000))  # some cliques
    s, d = np.concatenate([s, extra[0]]), np.concatenate([d, extra[1]])
    held, E = held_by_counts(2 * k, s, d, [Q.CLIQUE4] if both else [Q.CLIQUE4, Q.CLIQUE5])
    if not both:
        assert held < 32 * E, (held, E)


def test_cliques_not_light():
    """6e5 edges of 30 to a vertex are past any light graph: renamed (32 bytes an
    edge and more of workspace), and as right as the edge-grouped kernels."""
    rng = np.random.default_rng(8)
    n = 20000
    s, d = rng.integers(0, n, (2, 30 * n))
    s[:200], d[:200] = 5, 100 + np.arange(200)  # a hub, so that the order matters
    held, E = held_by_counts(n, s, d, [Q.CLIQUE4, Q.CLIQUE5])
    assert E > 1 << 19 and held > 32 * E, (held, E)
