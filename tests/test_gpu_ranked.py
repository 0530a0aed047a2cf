"""Whole counts on graphs built with ids ascending by degree: as built, after
updates that change who is a hub, and after updates taken back; counts and every
counter against the oracle."""
import time

import numpy as np
import pytest

import oracle
import synth
from tests import queries as Q

pytestmark = pytest.mark.gpu

FOUR = {"clique4": Q.CLIQUE4, "clique5": Q.CLIQUE5, "diamond": Q.DIAMOND, "cycle4": Q.CYCLE4}


def check(gj, ctx, G, n, s, d, cliques=1 << 11):
    O = oracle.Graph(n, s, d)
    for name, q in FOUR.items():
        if name in ("clique4", "clique5") and n > cliques:  # the oracle's time
            continue
        want = (oracle.twopath(O, name, threads=8) if name in ("diamond", "cycle4") else oracle.run(O, q, threads=8))
        got = gj.count(ctx, G, gj.Query(ctx, *q))
        for k in ("matches", "prefixes", "extensions"):
            assert got[k] == want[k], (name, k, got[k], want[k])


@pytest.mark.parametrize("undirected", [False, True])
@pytest.mark.parametrize("scale", [9, 11, 14])
def test_built_and_updated(scale, undirected):
    """Updates against the order: R-MAT edges whose hubs are the ids of least
    degree, in either direction, some both ways."""
    import paper_1802_03760_amd as gj
    n = 1 << scale
    s, d = synth.rmat_draws(scale, 6, seed=scale)
    ctx = gj.Context(0)
    G = gj.Graph(ctx, s, d, n, degree_order=True, undirected=undirected)
    bs, bd, _ = oracle.relabel_by_degree(n, s, d, undirected=undirected)
    check(gj, ctx, G, n, bs, bd)
    us, ud = synth.rmat_draws(scale, 4, seed=scale + 1)
    k = len(us) // 8
    us, ud = np.concatenate([us, ud[:k]]), np.concatenate([ud, us[:k]])
    new = np.setdiff1d(us.astype(np.uint64) << np.uint64(32) | ud, bs.astype(np.uint64) << np.uint64(32) | bd)
    us, ud = (new >> np.uint64(32)).astype(np.uint32), new.astype(np.uint32)
    us, ud = us[us != ud], ud[us != ud]
    one = np.ones(len(us), np.int8)
    gj.apply_updates(ctx, G, us, ud, one, [])
    check(gj, ctx, G, n, np.concatenate([bs, us]), np.concatenate([bd, ud]))
    gj.apply_updates(ctx, G, us, ud, -one, [])
    check(gj, ctx, G, n, bs, bd)


@pytest.mark.parametrize("changes", [1, 400, 2000, 5000])
def test_few_changes(changes):
    """Few enough changes to keep the order, or just too many: all of them at the
    vertex of least degree, which they make a hub, in both directions (2,000:
    more members there than a bit matrix takes)."""
    import paper_1802_03760_amd as gj
    n = 1 << 13
    s, d = synth.rmat_draws(13, 12, seed=2)
    ctx = gj.Context(0)
    G = gj.Graph(ctx, s, d, n, degree_order=True)
    bs, bd, _ = oracle.relabel_by_degree(n, s, d)
    rng = np.random.default_rng(changes)
    x = 1 + rng.permutation(n - 1)[:changes].astype(np.uint32)
    way = rng.random(len(x)) < 0.5
    us, ud = np.where(way, 0, x).astype(np.uint32), np.where(way, x, 0).astype(np.uint32)
    gj.apply_updates(ctx, G, us, ud, np.ones(len(us), np.int8), [])
    check(gj, ctx, G, n, np.concatenate([bs, us]), np.concatenate([bd, ud]), n)


def test_updated_from_nothing():
    """A degree-ordered build of next to no edges, then all of them by updates:
    the ids say nothing of the degrees, and counts take about what they take on
    the same relation built without an order."""
    import paper_1802_03760_amd as gj
    scale, n = 18, 1 << 18
    s, d = synth.rmat_draws(scale, 8, seed=1)
    keys = np.unique(np.minimum(s, d).astype(np.uint64) << np.uint64(32) | np.maximum(s, d))
    us, ud = (keys >> np.uint64(32)).astype(np.uint32), keys.astype(np.uint32)
    us, ud = us[us != ud], ud[us != ud]
    ctx = gj.Context(0)
    G = gj.Graph(ctx, us[:1], ud[:1], n, degree_order=True)
    gj.apply_updates(ctx, G, [n - 2], [n - 1], np.array([-1], np.int8), [])
    gj.apply_updates(ctx, G, us, ud, np.ones(len(us), np.int8), [])
    H = gj.Graph(ctx, us, ud, n)
    for name in ("diamond", "cycle4"):
        q = gj.Query(ctx, *FOUR[name])
        t, got = [], []
        for graph in (G, H):
            got.append([gj.count(ctx, graph, q)[k] for k in ("matches", "prefixes", "extensions")])
            best = 1e9
            for _ in range(5):
                a = time.perf_counter()
                gj.count(ctx, graph, q)
                best = min(best, time.perf_counter() - a)
            t.append(best)
        assert got[0] == got[1], name
        assert t[0] < 2 * t[1], (name, t)
