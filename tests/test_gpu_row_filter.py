"""Long object rows of 16-word batches under whitelists so narrow that few queries are left after a row's first steps: entries
are then left out by relation, up to the number of relations that the block's bits hold."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("R", [1, 63, 64, 65, 4095, 4096, 4097])
@pytest.mark.parametrize("allowed", [1, 3])
def test_rare_relations(R, allowed):
    import paper_2604_18913_amd as lkg
    rng = np.random.default_rng(R + allowed)
    E, Q, k = 12_000, 300, 2
    rows = (1024, 2049, 5000, 8193, 11_000)
    s = np.concatenate([rng.choice(E, d, replace=False) for d in rows] + [rng.integers(0, E, 20_000)]).astype(np.int32)
    o = np.concatenate([np.full(d, i) for i, d in enumerate(rows)] + [rng.integers(0, E, 20_000)]).astype(np.int32)
    r = (R * rng.random(len(s)) ** 3).astype(np.int32)  # the larger, the rarer
    p = rng.permutation(len(s))
    s, r, o = s[p], r[p], o[p]
    off = 40 * np.arange(Q + 1, dtype=np.int64)
    seeds = rng.integers(0, E, off[-1]).astype(np.int32)
    mask = np.zeros((Q, (R + 63) // 64), np.uint64)
    for q in range(Q):
        for x in rng.integers(0, R, allowed):
            mask[q, x >> 6] |= np.uint64(1) << np.uint64(x & 63)
    want = oracle.khop(E, s, r, o, off, seeds, k, mask)
    for opts in ({}, {"hub_min_degree": 9000}, {"num_shards": 2}):
        g = lkg.Graph(s, r, o, E, R, **opts)
        res = g.khop(off, seeds, k, mask)
        assert np.array_equal(res.offsets(), want[0])
        for got, w in zip(res.fetch(), want[1:4]):
            assert np.array_equal(got.cpu().numpy(), w)
        res.close()
        g.close()
