"""Lists of 16-word batches on both sides of the share of reached pairs at which another kernel writes them: empty and full
words, queries that reach few and many entities of a tile, seeds, short and long rows, pages, ragged last words."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("hub_min", [0, 40])
@pytest.mark.parametrize("Q, k", [(257, 2), (1000, 3), (1024, 1), (1024, 0), (1024, 6)])
@pytest.mark.parametrize("allowed, popular", [(2, 0.0), (8, 0.3), (30, 0.8)])
def test_lists(Q, k, allowed, popular, hub_min):
    import paper_2604_18913_amd as lkg
    rng = np.random.default_rng(Q + allowed)
    E, R, T = 5003, 64, 24_000
    # a few objects that every query may reach, and objects with rows of 33 entries and more
    o = np.where(rng.random(T) < popular, rng.integers(0, 90, T), rng.integers(0, E, T)).astype(np.int32)
    o[:400], o[400:2600] = 4000, 4001
    s = rng.integers(0, E, T).astype(np.int32)
    r = rng.integers(0, R, T).astype(np.int32)
    off = np.concatenate([[0], np.cumsum(rng.integers(0, 9, Q))]).astype(np.int64)
    seeds = rng.integers(0, E, int(off[-1])).astype(np.int32)
    mask = np.zeros((Q, 1), dtype=np.uint64)
    for q in range(Q):
        for b in rng.integers(0, R, allowed):
            mask[q, 0] |= np.uint64(1) << np.uint64(b)
    g = lkg.Graph(s, r, o, E, R, hub_min_degree=hub_min)
    res = g.khop(off, seeds, k, mask)
    want = oracle.khop(E, s, r, o, off, seeds, k, mask)
    assert np.array_equal(res.offsets(), want[0])
    for q0, q1 in {(0, Q), (64, 128), (100, 101), (130, 250), (Q // 2, Q)}:
        a, b = want[0][q0], want[0][q1]
        for got, w in zip(res.fetch(q0, q1), want[1:]):
            assert np.array_equal(got.cpu().numpy(), w[a:b])
    ent, hop, pred = res.fetch(want_hop=False)
    assert hop is None and np.array_equal(ent.cpu().numpy(), want[1]) and np.array_equal(pred.cpu().numpy(), want[3])
    res.close()
    g.close()
