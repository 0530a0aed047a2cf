"""Last stages bound by the two ends of an edge of the query, counted per edge
(the house and its variants), against the oracle: every direction of the two
atoms and of the edge that joins them, in one and in many batches."""
import pytest

import oracle
import synth
from tests import queries as Q

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("cap", [0, 1 << 14])
@pytest.mark.parametrize("way", range(8))
def test_directions(way, cap):
    import paper_1802_03760_amd as gj
    e, f, g = way & 1, way >> 1 & 1, way >> 2
    q = (4, [(0, 1), (2, 1) if e else (1, 2), (3, 1) if f else (1, 3), (3, 2) if g else (2, 3)], [0, 1, 2, 3])
    s, d = synth.rmat_draws(9, 16, seed=way)
    ctx = gj.Context(0)
    ctx.set_option("run_stage_min", 0)
    if cap:
        ctx.set_option("frontier_cap", cap)
    G = gj.Graph(ctx, s, d, 512)
    want = oracle.run(oracle.Graph(512, s, d), q, threads=8)
    got = gj.count(ctx, G, gj.Query(ctx, *q))
    for k in ("matches", "prefixes", "extensions"):
        assert got[k] == want[k], (q, k)


@pytest.mark.parametrize("lo,hi", [(0, None), (0, 1), (100, 3000)])
def test_house(lo, hi):
    import paper_1802_03760_amd as gj
    s, d = synth.rmat_draws(10, 12, seed=1)
    ctx = gj.Context(0)
    ctx.set_option("run_stage_min", 0)
    G = gj.Graph(ctx, s, d, 1024)
    want = oracle.run(oracle.Graph(1024, s, d), Q.HOUSE, seed_lo=lo, seed_hi=hi, threads=8)
    got = gj.count(ctx, G, gj.Query(ctx, *Q.HOUSE), lo, (1 << 64) - 1 if hi is None else hi)
    for k in ("matches", "prefixes", "extensions"):
        assert got[k] == want[k], k


@pytest.mark.parametrize("cap,seeds", [(1 << 18, 1 << 25), (1 << 20, 500)])
def test_batches(cap, seeds):
    """One table of edge counts for many batches, from the first that repays it:
    seeds of low degree first, whose batches are declined (of 30 batches of 500
    seeds the first eight have 0 to 0.5 times the candidates that a look at the
    edges needs, the others 1.2 to 5.6 times)."""
    import numpy as np
    import paper_1802_03760_amd as gj
    s, d = synth.rmat_draws(10, 20, seed=3)
    rank = np.argsort(np.argsort(np.bincount(s, minlength=1024) + np.bincount(d, minlength=1024)))
    s, d = rank[s].astype(np.uint32), rank[d].astype(np.uint32)  # ids ascend by degree
    ctx = gj.Context(0)
    for k, v in (("run_stage_min", 0), ("frontier_cap", cap), ("seed_chunk", seeds)):
        ctx.set_option(k, v)
    G = gj.Graph(ctx, s, d, 1024)
    want = oracle.run(oracle.Graph(1024, s, d), Q.HOUSE, threads=8)
    assert want["extensions"][4] > 60 * 256 * G.info()["edges"]
    got = gj.count(ctx, G, gj.Query(ctx, *Q.HOUSE))
    for k in ("matches", "prefixes", "extensions"):
        assert got[k] == want[k], (k, got[k], want[k])
