"""Predecessors of object rows that are cut into segments (8,192 entries and more), on every plane
width, deep searches, pages and sharded graphs."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


def giant_graph(rng, E, R, degrees):
    """Objects 0, 1, .. have the given numbers of entries; the rest is sparse and leads to their subjects."""
    o = np.concatenate([np.full(d, i) for i, d in enumerate(degrees)] + [rng.integers(len(degrees), E, 3 * E)])
    s = rng.integers(0, E, len(o))
    r = rng.integers(0, R, len(o))
    perm = rng.permutation(len(o))
    return s[perm].astype(np.int32), r[perm].astype(np.int32), o[perm].astype(np.int32)


@pytest.mark.parametrize("masked", [False, True])
@pytest.mark.parametrize("Q, k", [(40, 2), (200, 3), (1000, 2), (300, 7), (200, 0), (1000, 0)])
@pytest.mark.parametrize("shards", [0, 3])
def test_rows_of_several_segments(Q, k, shards, masked):
    import paper_2604_18913_amd as lkg
    rng = np.random.default_rng(Q + k)
    E, R = 5000, 40
    s, r, o = giant_graph(rng, E, R, (8191, 8192, 8193, 16384, 30001))
    off = np.concatenate([[0], np.cumsum(rng.integers(1, 3, Q))]).astype(np.int64)
    seeds = rng.integers(0, E, off[-1]).astype(np.int32)
    mask = None
    if masked:
        mask = np.zeros((Q, 1), np.uint64)
        for b in range(R):
            mask[:, 0] |= (rng.random(Q) < 0.15).astype(np.uint64) << np.uint64(b)
    want = oracle.khop(E, s, r, o, off, seeds, k, mask)
    for opts in ({}, {"max_resident_shards": 2}) if shards else ({}, {"hub_min_degree": 40}, {"hub_min_degree": 9000}):
        g = lkg.Graph(s, r, o, E, R, num_shards=shards, **opts)
        res = g.khop(off, seeds, k, mask)
        assert np.array_equal(res.offsets(), want[0])
        for q0, q1 in ((0, Q), (Q // 3, min(Q, Q // 3 + 30)), (Q - 1, Q)):
            ent, hop, pred = res.fetch(q0, q1)
            a, b = want[0][q0], want[0][q1]
            assert np.array_equal(ent.cpu().numpy(), want[1][a:b])
            assert np.array_equal(hop.cpu().numpy(), want[2][a:b])
            assert np.array_equal(pred.cpu().numpy(), want[3][a:b])
        res.close()
        g.close()
