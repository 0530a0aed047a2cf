"""Whole triangle listings (sorted rows and every counter) against the oracle,
with sets at the edges of the listing kernel's cases: sizes around a mask word
and around the LDS table's segments, on either side of the seed edge."""
import numpy as np
import pytest

import oracle
import synth
from tests import queries as Q

pytestmark = pytest.mark.gpu

SIZES = [1, 2, 63, 64, 65, 127, 128, 129, 192, 193, 300, 5000]


def check(n, src, dst, queries):
    import paper_1802_03760_amd as gj
    ctx = gj.Context(0)
    G = gj.Graph(ctx, src, dst, n)
    O = oracle.Graph(n, src, dst)
    for q in queries:
        want = oracle.run(O, q, collect=True, threads=4)
        Qh = gj.Query(ctx, q[0], q[1], q[2])
        st, rows = gj.enumerate_rows(ctx, G, Qh)
        for k in ("matches", "prefixes", "extensions"):
            assert st[k] == want[k], (q, k, st[k], want[k])
        assert np.array_equal(np.asarray(rows), want["rows"]), q
        if want["matches"]:
            with pytest.raises(gj.GJError) as e:
                gj.enumerate_rows(ctx, G, Qh, cap=want["matches"] - 1,
                                  out=np.empty((want["matches"], q[0]), np.uint32))
            assert e.value.status == gj.GJ_EOVERFLOW


@pytest.mark.parametrize("hub", [64, 65, 8191, 8192, 8193, 20000])
@pytest.mark.parametrize("out", [True, False])
def test_set_sizes(hub, out):
    """A vertex with `hub` neighbours, joined to vertices with sets of every
    size over the same ids; the hub at either end of the seed edge."""
    rng = np.random.default_rng(hub)
    ids = 100 + np.sort(rng.permutation(30000)[:hub])
    s, d = [np.full(hub, 50)], [ids]
    for i, size in enumerate(SIZES):
        v = 60 + i
        s += [np.array([50 if out else v]), np.full(size, v)]
        d += [np.array([v if out else 50]), 100 + rng.permutation(30000)[:size]]
    check(30100, np.concatenate(s).astype(np.uint32), np.concatenate(d).astype(np.uint32), [Q.TRIANGLE])


@pytest.mark.parametrize("scale", [6, 10, 13])
def test_rmat(scale):
    s, d = synth.rmat_draws(scale, 12, seed=scale)
    check(1 << scale, s, d, [Q.TRIANGLE, Q.CYCLIC_TRIANGLE, Q.with_order(Q.TRIANGLE, [2, 0, 1]),
                             Q.with_order(Q.TRIANGLE, [1, 2, 0])])


def test_no_matches():
    check(5, np.array([0, 1], np.uint32), np.array([1, 2], np.uint32), [Q.TRIANGLE])
    check(5, np.array([3], np.uint32), np.array([3], np.uint32), [Q.TRIANGLE])


# The listing kernel itself (run_stage_min 0: whatever the graph's size).


def listed(n, src, dst, queries, host=True):
    import torch
    import paper_1802_03760_amd as gj
    ctx = gj.Context(0)
    ctx.set_option("run_stage_min", 0)
    G = gj.Graph(ctx, src, dst, n)
    O = oracle.Graph(n, src, dst)
    for q in queries:
        want = oracle.run(O, q, collect=True, threads=4)
        k = want["matches"]
        Qh = gj.Query(ctx, q[0], q[1], q[2])
        for _ in range(2):  # the plan and the workspace of the first again
            if host:
                st, rows = gj.enumerate_rows(ctx, G, Qh)
                rows = np.asarray(rows)
            else:
                out = torch.full((k + 3, 3), -1, dtype=torch.int32, device="cuda")
                st, _ = gj.enumerate_rows(ctx, G, Qh, out=out)
                rows = out.cpu().numpy().view(np.uint32)
                assert (rows[k:] == 0xFFFFFFFF).all()
                rows = rows[:k]
            for c in ("matches", "prefixes", "extensions"):
                assert st[c] == want[c], (q, c, st[c], want[c])
            assert np.array_equal(rows, want["rows"]), q
        if k:
            with pytest.raises(gj.GJError) as e:
                gj.enumerate_rows(ctx, G, Qh, cap=k - 1, out=np.empty((k, q[0]), np.uint32))
            assert e.value.status == gj.GJ_EOVERFLOW
    return ctx


@pytest.mark.parametrize("hub", [63, 64, 65, 8191, 8192, 8193, 20000])
@pytest.mark.parametrize("out", [True, False])
def test_listed_set_sizes(hub, out):
    rng = np.random.default_rng(hub)
    ids = 100 + np.sort(rng.permutation(30000)[:hub])
    s, d = [np.full(hub, 50)], [ids]
    for i, size in enumerate(SIZES):
        v = 60 + i
        s += [np.array([50 if out else v]), np.full(size, v)]
        d += [np.array([v if out else 50]), 100 + rng.permutation(30000)[:size]]
    s, d = np.concatenate(s).astype(np.uint32), np.concatenate(d).astype(np.uint32)
    listed(30100, s, d, [Q.TRIANGLE])
    # the same sets as in-neighbours, and in both directions
    listed(30100, d, s, [Q.TRIANGLE], host=False)
    listed(30100, np.concatenate([s, d]), np.concatenate([d, s]), [Q.TRIANGLE, Q.CYCLIC_TRIANGLE])


@pytest.mark.parametrize("scale", [1, 3, 6, 10, 13])
@pytest.mark.parametrize("host", [True, False])
def test_listed_rmat(scale, host):
    s, d = synth.rmat_draws(scale, 12, seed=scale)
    qs = [Q.with_order(t, o) for t in (Q.TRIANGLE, Q.CYCLIC_TRIANGLE) for o in Q.valid_orders(t)]
    listed(1 << scale, s, d, qs if scale < 13 else qs[::3], host)


def test_listed_no_matches():
    a = np.arange(70, dtype=np.uint32)
    listed(80, a, a + 1, [Q.TRIANGLE, Q.CYCLIC_TRIANGLE])        # a path
    listed(80, a + 1, np.zeros(70, np.uint32), [Q.TRIANGLE])     # all into one vertex
    listed(80, np.zeros(70, np.uint32), a + 1, [Q.TRIANGLE])     # all out of it
    listed(5, np.array([3], np.uint32), np.array([3], np.uint32), [Q.TRIANGLE])


def test_listed_after_update():
    """The version an update wrote, and the one that takes it back."""
    import paper_1802_03760_amd as gj
    s, d = synth.rmat_draws(9, 12, seed=9)
    ctx = gj.Context(0)
    ctx.set_option("run_stage_min", 0)
    G = gj.Graph(ctx, s, d, 512)
    q = gj.Query(ctx, *Q.TRIANGLE)
    rng = np.random.default_rng(1)
    us, ud = (rng.integers(0, 512, 600).astype(np.uint32) for _ in range(2))
    s2, d2 = np.concatenate([s, us]), np.concatenate([d, ud])
    for S, D, sign in ((s, d, 0), (s2, d2, 1)):
        if sign:
            gj.apply_updates(ctx, G, us, ud, np.ones(600, np.int8), [])
        want = oracle.run(oracle.Graph(512, S, D), Q.TRIANGLE, collect=True)
        st, rows = gj.enumerate_rows(ctx, G, q)
        assert st["matches"] == want["matches"] and np.array_equal(np.asarray(rows), want["rows"])
