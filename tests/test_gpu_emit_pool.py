"""Lists of 16-word batches at the limits of what the list writer keeps in LDS: blocks whose edge ids and predecessor lines fit
together, whose lines do not fit beside the ids, whose ids do not fit, and last blocks of few tiles."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("E", [64, 1025, 3011])
@pytest.mark.parametrize("row, share_long", [(1, 0.0), (5, 0.2), (10, 0.5), (19, 0.0), (20, 0.1), (32, 0.0), (32, 0.05), (33, 0.0)])
def test_lists(row, share_long, E):
    import paper_2604_18913_amd as lkg
    rng = np.random.default_rng(E + row)
    Q, k, R = 300, 3, 5
    deg = np.where(rng.random(E) < share_long, 40, row)
    o = np.repeat(rng.permutation(E), deg).astype(np.int32)
    s = rng.integers(0, E, o.size).astype(np.int32)
    p = rng.permutation(o.size)
    s, o = s[p], o[p]
    r = rng.integers(0, R, o.size).astype(np.int32)
    off = np.arange(0, 30 * Q + 1, 30, dtype=np.int64)
    seeds = rng.integers(0, E, 30 * Q).astype(np.int32)
    g = lkg.Graph(s, r, o, E, R)
    res = g.khop(off, seeds, k)
    want = oracle.khop(E, s, r, o, off, seeds, k)
    assert np.array_equal(res.offsets(), want[0])
    for q0, q1 in ((0, Q), (70, 71), (0, 130)):
        a, b = want[0][q0], want[0][q1]
        for got, w in zip(res.fetch(q0, q1), want[1:]):
            assert np.array_equal(got.cpu().numpy(), w[a:b])
    res.close()
    g.close()


@pytest.mark.parametrize("allowed", [1, 4])
@pytest.mark.parametrize("row", [1, 2, 15, 16, 17, 18, 31, 32])
def test_rows_under_whitelists(row, allowed):
    """Object rows around the sixteen entries that a group holds from the start, with relations that most or few queries may
    follow."""
    import paper_2604_18913_amd as lkg
    rng = np.random.default_rng(row)
    E, R, Q, k = 1500, 5, 700, 3
    o = np.repeat(rng.permutation(E), row).astype(np.int32)
    s = rng.integers(0, E, o.size).astype(np.int32)
    p = rng.permutation(o.size)
    s, o = s[p], o[p]
    r = rng.integers(0, R, o.size).astype(np.int32)
    off = np.arange(0, 20 * Q + 1, 20, dtype=np.int64)
    seeds = rng.integers(0, E, 20 * Q).astype(np.int32)
    mask = np.zeros((Q, 1), dtype=np.uint64)
    for q in range(Q):
        for b in rng.permutation(R)[:allowed]:
            mask[q, 0] |= np.uint64(1) << np.uint64(b)
    g = lkg.Graph(s, r, o, E, R)
    want = oracle.khop(E, s, r, o, off, seeds, k, mask)
    for direction in ("push", "pull"):
        res = g.khop(off, seeds, k, mask, direction=direction)
        assert np.array_equal(res.offsets(), want[0])
        for q0, q1 in ((0, Q), (60, 500)):
            a, b = want[0][q0], want[0][q1]
            for got, w in zip(res.fetch(q0, q1), want[1:]):
                assert np.array_equal(got.cpu().numpy(), w[a:b])
        res.close()
    g.close()
