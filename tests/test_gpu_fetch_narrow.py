"""Lists of narrow batches (one and four words per entity) where hub rows are cut into segments: rows at the edges of a
segment and of the classes, every hop level in one launch, pages, joined shards, and a recorded fetch."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

ROWS = [33, 1023, 1024, 2047, 2048, 2049, 4096, 4097, 9000, 20481]


@pytest.mark.parametrize("shards", [0, 3])
@pytest.mark.parametrize("hub_min", [0, 40, 3000])
@pytest.mark.parametrize("Q, k, masked", [(1, 3, False), (64, 0, False), (64, 2, True), (65, 3, False), (256, 3, True)])
def test_hub_rows_in_segments(Q, k, masked, hub_min, shards):
    import paper_2604_18913_amd as lkg
    rng = np.random.default_rng(Q + hub_min)
    E, R = 6007, 11
    o = np.concatenate([np.repeat(rng.permutation(E)[:len(ROWS)], ROWS), rng.integers(0, E, 9000)]).astype(np.int32)
    s = np.where(rng.random(o.size) < 0.2, rng.integers(0, 40, o.size), rng.integers(0, E, o.size)).astype(np.int32)
    p = rng.permutation(o.size)
    s, o = s[p], o[p]
    r = rng.integers(0, R, o.size).astype(np.int32)
    off = np.arange(Q + 1, dtype=np.int64)
    seeds = rng.integers(0, E, Q).astype(np.int32)
    mask = rng.integers(0, 2**R, (Q, 1)).astype(np.uint64) if masked else None
    g = lkg.Graph(s, r, o, E, R, hub_min_degree=hub_min, num_shards=shards)
    res = g.khop(off, seeds, k, mask, direction="pull")  # (a small search would not come by here)
    want = oracle.khop(E, s, r, o, off, seeds, k, mask)
    assert np.array_equal(res.offsets(), want[0])
    for q0, q1 in {(0, Q), (Q // 2, Q), (Q // 3, Q // 3 + 1)}:
        a, b = want[0][q0], want[0][q1]
        for got, w in zip(res.fetch(q0, q1), want[1:]):
            assert np.array_equal(got.cpu().numpy(), w[a:b])
    _, hop, pred = res.fetch(want_hop=False)
    assert hop is None and np.array_equal(pred.cpu().numpy(), want[3])
    res.close()
    g.close()


def test_more_threads_than_a_launch_takes():
    """Every row is a hub row and has a block per hop level: 66,100 rows x 254 hops x 256 threads pass 2^32."""
    import paper_2604_18913_amd as lkg
    n, d, k = 66_100, 33, 254
    s = np.repeat(np.arange(d, dtype=np.int32), n)
    o = np.tile(np.arange(d, d + n, dtype=np.int32), d)
    r = np.zeros(s.size, dtype=np.int32)
    off, seeds = np.array([0, 2], dtype=np.int64), np.array([3, 20], dtype=np.int32)
    g = lkg.Graph(s, r, o, d + n, 1, hub_min_degree=d)
    res = g.khop(off, seeds, k, direction="pull")
    want = oracle.khop(d + n, s, r, o, off, seeds, k)
    assert np.array_equal(res.offsets(), want[0])
    for got, w in zip(res.fetch(), want[1:]):
        assert np.array_equal(got.cpu().numpy(), w)
    res.close()
    g.close()


@pytest.mark.parametrize("Q, masked", [(40, False), (200, True)])
def test_a_recorded_fetch_of_rows_in_segments(Q, masked):
    """A capture takes no memory for the segments: the kernels run one by one, and a fetch behind them in one launch."""
    import paper_2604_18913_amd as lkg
    from test_gpu_capture import Arena, captured_fetch
    rng = np.random.default_rng(Q)
    E, R, k = 6007, 11, 3
    rows = [33, 1024, 2048, 2049, 4097, 8191]
    o = np.concatenate([np.repeat(rng.permutation(E)[:len(rows)], rows), rng.integers(0, E, 9000)]).astype(np.int32)
    s, r = rng.integers(0, E, o.size).astype(np.int32), rng.integers(0, R, o.size).astype(np.int32)
    s[rng.random(o.size) < 0.2] = 5
    off = np.arange(Q + 1, dtype=np.int64)
    seeds = rng.integers(0, E, Q).astype(np.int32)
    seeds[0] = 5
    mask = rng.integers(0, 2**R, (Q, 1)).astype(np.uint64) if masked else None
    want = oracle.khop(E, s, r, o, off, seeds, k, mask)
    arena = Arena(256 << 20)
    g = lkg.Graph(s, r, o, E, R, dev_alloc=arena.alloc, dev_free=arena.free)
    res = g.khop(off, seeds, k, mask, direction="pull")
    for q0, q1 in ((0, Q), (7, Q - 5)):
        for got in captured_fetch(res, arena, q0, q1):
            for x, y in zip(got, want[1:4]):
                assert np.array_equal(x, y[want[0][q0]:want[0][q1]])
        for x, y in zip(res.fetch(q0, q1), want[1:4]):
            assert np.array_equal(x.cpu().numpy(), y[want[0][q0]:want[0][q1]])
    res.close()
    g.close()
