"""Pages of a large batch on a result that lists so many entities that the page's words are packed first."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("masked", [False, True])
def test_pages_of_a_result_with_millions_of_listed_entities(masked):
    import paper_2604_18913_amd as lkg
    rng = np.random.default_rng(3)
    E, T, R, Q, k = 4_400_000, 12_000_000, 30, 300, 3
    s, o = rng.integers(0, E, T, dtype=np.int32), rng.integers(0, E, T, dtype=np.int32)
    r = rng.integers(0, R, T, dtype=np.int32)
    o[:200_000] = np.arange(200_000) % 9               # giant rows
    o[200_000:300_000] = 100 + np.arange(100_000) % 200  # mid rows
    lists = [rng.integers(0, E, 3) for _ in range(Q)]
    lists[7] = rng.permutation(E)[:4_300_000]          # one question seeds most of the graph: all of it is listed
    off = np.concatenate([[0], np.cumsum([len(x) for x in lists])]).astype(np.int64)
    seeds = np.concatenate(lists).astype(np.int32)
    mask = None
    if masked:
        mask = np.zeros((Q, 1), np.uint64)
        for b in range(R):
            mask[:, 0] |= (rng.random(Q) < 0.7).astype(np.uint64) << np.uint64(b)
    g = lkg.Graph(s, r, o, E, R)
    res = g.khop(off, seeds, k, mask)
    reached = res.offsets()
    for q0, q1 in ((64, 128), (130, 250), (70, 200), (299, 300)):  # one, two and four aligned words
        sub = lists[q0:q1]
        so = np.concatenate([[0], np.cumsum([len(x) for x in sub])]).astype(np.int64)
        want = oracle.khop(E, s, r, o, so, np.concatenate(sub).astype(np.int32), k, None if mask is None else mask[q0:q1])
        assert np.array_equal(reached[q0:q1 + 1] - reached[q0], want[0])
        ent, hop, pred = res.fetch(q0, q1)
        assert np.array_equal(ent.cpu().numpy(), want[1])
        assert np.array_equal(hop.cpu().numpy(), want[2])
        assert np.array_equal(pred.cpu().numpy(), want[3])
    res.close()
    g.close()
