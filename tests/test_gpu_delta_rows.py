"""Row pointers of updated versions against the edge set, at the edges of the
waves' row ranges: changes in the first and last rows, in one row of a wave, in
every row, inserts and deletes that cancel."""
import numpy as np
import pytest

from tests.test_gpu_delta import check_index

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [2, 63, 64, 65, 4097, 524287, 524288, 600011])
@pytest.mark.parametrize("k", [1, 3, 5000])
def test_rows(n, k):
    import paper_1802_03760_amd as gj
    rng = np.random.default_rng(n + k)
    m = min(4 * n, 200000)
    loops = np.arange(n, dtype=np.uint64) * np.uint64((1 << 32) + 1)  # builds and updates drop them
    keys = np.unique(rng.integers(0, n, m).astype(np.uint64) << np.uint64(32) | rng.integers(0, n, m).astype(np.uint64))
    keys = np.setdiff1d(keys, loops)
    ctx = gj.Context(0)
    G = gj.Graph(ctx, (keys >> np.uint64(32)).astype(np.uint32), keys.astype(np.uint32), n)
    for step in range(3):  # the third version reuses the first one's buffers
        ends = rng.choice(np.array([0, 1 % n, n // 2, n - 1]), k)
        src = np.where(rng.random(k) < 0.5, ends, rng.integers(0, n, k))
        dst = np.where(rng.random(k) < 0.5, ends[::-1], rng.integers(0, n, k))
        new = np.setdiff1d(src.astype(np.uint64) << np.uint64(32) | dst.astype(np.uint64),
                           np.union1d(keys, loops))
        old = keys[rng.permutation(len(keys))[:k // 2]]
        b = np.concatenate([new, old])
        g = np.concatenate([np.ones(len(new), np.int8), -np.ones(len(old), np.int8)])
        gj.apply_updates(ctx, G, (b >> np.uint64(32)).astype(np.uint32), b.astype(np.uint32), g, [])
        keys = np.union1d(np.setdiff1d(keys, old), new)
        check_index(G, (keys >> np.uint64(32)).astype(np.uint32), keys.astype(np.uint32))
