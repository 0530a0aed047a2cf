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
