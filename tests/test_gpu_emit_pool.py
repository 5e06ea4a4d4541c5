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
