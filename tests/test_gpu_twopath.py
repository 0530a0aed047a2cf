"""Whole diamond and 4-cycle counts (counts and every counter) against the
oracle's 2-path counts, on graphs whose vertices fall into each class of the
kernels that count 2-paths per pair of vertices."""
import numpy as np
import pytest

import oracle
import synth
from tests import queries as Q

pytestmark = pytest.mark.gpu

QUERY = {"diamond": Q.DIAMOND, "cycle4": Q.CYCLE4}


def rmat(scale, draws_per_vertex):
    s, d = synth.rmat_draws(scale, draws_per_vertex, seed=scale)
    return 1 << scale, s, d


def both_ways():
    """Every edge reciprocal: matches with a0 = a3 or a1 = a2 throughout."""
    n, s, d = rmat(11, 12)
    return n, np.concatenate([s, d]), np.concatenate([d, s])


def two_hubs():
    """66,000 vertices between two hubs, in all four directions somewhere: more
    than a 16-bit count holds for one pair."""
    k = 66000
    u = np.arange(2, 2 + k, dtype=np.uint32)
    rng = np.random.default_rng(5)
    s = [np.zeros(k, np.uint32), u, np.ones(k, np.uint32)]
    d = [u, np.ones(k, np.uint32), u]
    more = rng.random(k) < 0.4
    s.append(u[more])
    d.append(np.zeros(int(more.sum()), np.uint32))
    return k + 2, np.concatenate(s), np.concatenate(d)


def many_hubs():
    """33,500 vertices of degree 64 and 42,000 of 51: pairs whose lower vertex
    lies beyond the first 32,768 ids by degree."""
    rng = np.random.default_rng(6)
    hubs, mids = 33500, 42000
    h = np.repeat(np.arange(hubs), 64)
    m = hubs + rng.integers(0, mids, len(h))
    out = rng.random(len(h)) < 0.5
    return hubs + mids, np.where(out, h, m).astype(np.uint32), np.where(out, m, h).astype(np.uint32)


def heavy_rows():
    """A vertex with 520 in-neighbours of in-degree above 4,096 and 600
    out-neighbours of out-degree above it."""
    rng = np.random.default_rng(7)
    leaves, xs, ys = 5000, 520, 600
    s, d = [], []
    c, x0, y0, l1, l2 = 0, 1, 1 + xs, 1 + xs + ys, 1 + xs + ys + leaves
    for i in range(xs):
        pick = rng.permutation(leaves)[:4090 + i]
        s += [l1 + pick, [x0 + i]]
        d += [np.full(len(pick), x0 + i), [c]]
    for i in range(ys):
        pick = rng.permutation(leaves)[:4090 + i]
        s += [np.full(len(pick), y0 + i), [c]]
        d += [l2 + pick, [y0 + i]]
    return l2 + leaves, np.concatenate(s).astype(np.uint32), np.concatenate(d).astype(np.uint32)


GRAPHS = {
    "one_edge": lambda: (2, np.array([0], np.uint32), np.array([1], np.uint32)),
    "one_pair": lambda: (3, np.array([2, 0], np.uint32), np.array([0, 2], np.uint32)),
    "rmat9": lambda: rmat(9, 6),
    "rmat13": lambda: rmat(13, 24),
    "rmat14": lambda: rmat(14, 16),
    "uniform": lambda: (16384, *synth.er_edges(16384, 150001, 3)),
    "uniform_above": lambda: (16385, *synth.er_edges(16385, 150001, 4)),
    "rmat16": lambda: rmat(16, 12),
    "both_ways": both_ways,
    "two_hubs": two_hubs,
    "many_hubs": many_hubs,
    "heavy_rows": heavy_rows,
}


@pytest.mark.parametrize("graph", sorted(GRAPHS))
def test_whole_counts(graph):
    import paper_1802_03760_amd as gj
    n, src, dst = GRAPHS[graph]()
    ctx = gj.Context(0)
    G = gj.Graph(ctx, src, dst, n)
    O = oracle.Graph(n, src, dst)
    for kind in ("diamond", "cycle4"):
        want = oracle.twopath(O, kind, threads=8)
        got = gj.count(ctx, G, gj.Query(ctx, *QUERY[kind]))
        for k in ("matches", "prefixes", "extensions"):
            assert got[k] == want[k], (graph, kind, k, got[k], want[k])


def test_uniform_large():
    """2^22 vertices of 32 edges in no order: walks over all ids below a vertex
    would take 2.4 s for the diamond, so the dense counters count it in 0.8."""
    import time

    import torch
    import paper_1802_03760_amd as gj
    n, m = 1 << 22, 32 << 22
    gen = torch.Generator(device="cuda")
    gen.manual_seed(9)
    s, d = (torch.randint(0, n, (m,), dtype=torch.int32, device="cuda", generator=gen) for _ in range(2))
    torch.cuda.synchronize()
    ctx = gj.Context(0)
    G = gj.Graph(ctx, s, d, n)
    k = torch.unique(s.to(torch.int64) * n + d)
    del s, d
    k = k[k // n != k % n]
    out, into = torch.bincount(k // n, minlength=n), torch.bincount(k % n, minlength=n)
    # the prefixes as the degrees give them; a1 = a2 alone matches every 2-path
    pairs, paths = int((out * out).sum()), int((out * into).sum())
    del k, out, into
    q = gj.Query(ctx, *Q.DIAMOND)
    best = 1e9
    for _ in range(3):
        t = time.perf_counter()
        got = gj.count(ctx, G, q)
        best = min(best, time.perf_counter() - t)
        assert got["prefixes"][3] == got["extensions"][2] == pairs and got["matches"] >= paths
    assert best < 1.5, best
