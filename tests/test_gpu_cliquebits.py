"""Whole transitive 4-clique and 5-clique counts (counts and every counter)
against the oracle, on graphs that put a vertex at the edges of the bit-matrix
kernels' size classes, and beyond the largest (left to the edge-grouped
kernels)."""
import numpy as np
import pytest

import oracle
import synth
from tests import queries as Q

pytestmark = pytest.mark.gpu


def check(n, src, dst, **build):
    import paper_1802_03760_amd as gj
    ctx = gj.Context(0)
    G = gj.Graph(ctx, src, dst, n, **build)
    if build:
        src, dst, _ = oracle.relabel_by_degree(n, src, dst, undirected=build.get("undirected", False))
    O = oracle.Graph(n, src, dst)
    for q in (Q.CLIQUE4, Q.CLIQUE5):
        want = oracle.run(O, q, threads=8)
        got = gj.count(ctx, G, gj.Query(ctx, *q))
        for k in ("matches", "prefixes", "extensions"):
            assert got[k] == want[k], (q[0], k, got[k], want[k])


@pytest.mark.parametrize("k", [1, 2, 3, 63, 64, 65, 256, 257, 512, 513, 1056, 1057])
def test_members(k):
    """A vertex joined to k vertices of higher degree, in both directions and
    some both ways, with some 20 edges among them each."""
    rng = np.random.default_rng(k)
    hubs = 1 + np.arange(k)
    leaves = np.arange(k * (k + 8)) + 1 + k  # each hub's own, so that the first vertex has the least degree
    s, d = [np.repeat(hubs, k + 8)], [leaves]
    way = rng.integers(0, 3, k)  # out, in, both
    s += [np.zeros(int((way != 1).sum()), int), hubs[way != 0]]
    d += [hubs[way != 1], np.zeros(int((way != 0).sum()), int)]
    if k > 1:
        s.append(rng.integers(1, 1 + k, 20 * k))
        d.append(rng.integers(1, 1 + k, 20 * k))
    check(1 + k + len(leaves), np.concatenate(s).astype(np.uint32), np.concatenate(d).astype(np.uint32))


@pytest.mark.parametrize("build", [{}, {"degree_order": True}, {"degree_order": True, "undirected": True}])
def test_rmat(build):
    s, d = synth.rmat_draws(10, 12, seed=2)
    check(1 << 10, s, d, **build)


def test_complete():
    """Every ordered pair of 40 vertices: all members both ways."""
    n = 40
    s, d = np.nonzero(~np.eye(n, dtype=bool))
    check(n, s.astype(np.uint32), d.astype(np.uint32))


@pytest.mark.parametrize("oriented", [False, True])
def test_hub_bits(oriented):
    """Above 500,000 edges members among the 32,768 first vertices are tested by
    bits: 500 groups of 80 vertices, and one of 120, on either side of that."""
    rng = np.random.default_rng(5)
    n, at = 40000, rng.permutation(40000).astype(np.uint32)
    base = np.repeat(80 * np.arange(500), 1600)
    s = np.concatenate([at[base + rng.integers(0, 80, len(base))], at[rng.integers(0, 120, 8000)]])
    d = np.concatenate([at[base + rng.integers(0, 80, len(base))], at[rng.integers(0, 120, 8000)]])
    assert len(np.unique(s.astype(np.uint64) << np.uint64(32) | d)) > 600000
    check(n, s, d, **({"degree_order": True} if oriented else {}))


@pytest.mark.parametrize("k", [66, 130, 150])
@pytest.mark.parametrize("way", ["down", "up", "mixed"])
def test_dense_rows(way, k):
    """k vertices, nine in ten pairs joined one way: matrix rows of up to 64, of
    up to 128 and of more members, in the ids' order and against it (all members
    out-, or all in-neighbours) and in any; and ten pairs both ways."""
    rng = np.random.default_rng(k)
    i, j = np.tril_indices(k, -1)
    keep = rng.random(len(i)) < 0.9
    i, j = i[keep], j[keep]
    if way == "up":
        i, j = j, i
    if way == "mixed":
        p = rng.permutation(k)
        i, j = p[i], p[j]
        i, j = np.concatenate([i, j[:10]]), np.concatenate([j, i[:10]])
    check(k, i.astype(np.uint32), j.astype(np.uint32))
    if way == "down":
        check(k, i.astype(np.uint32), j.astype(np.uint32), degree_order=True)
