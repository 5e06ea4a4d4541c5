"""Pulled hops on planes of one and four words: rows at the edges of the steps of a lane group, a wavefront and a segment,
queries that have nothing left to expand, and the bitmap and live words that the census makes, against the oracle."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

ROWS = [1, 2, 8, 15, 16, 17, 31, 32, 33, 64, 255, 256, 257, 1023, 1024, 1025, 2049, 5000]


def graph(E, rng):
    """Objects 0 .. len(ROWS) - 1 have rows of these lengths, the others of up to three entries; some subjects are hubs."""
    o = np.concatenate([np.repeat(np.arange(len(ROWS)), ROWS), rng.integers(len(ROWS), E, 3 * min(E, 4000))])
    s = np.where(rng.random(o.size) < 0.3, rng.integers(0, 5, o.size), rng.integers(0, min(E, 4000), o.size))
    p = rng.permutation(o.size)
    return s[p].astype(np.int32), rng.integers(0, 9, o.size).astype(np.int32), o[p].astype(np.int32)


@pytest.mark.parametrize("E", [4001, 4096, 1_100_003])  # the last: more entities than one turn of the census' grid
@pytest.mark.parametrize("Q, masked, walk", [(1, False, False), (3, False, True), (64, True, False), (65, False, False),
                                             (200, True, False), (256, True, True)])
def test_pulled_hops(E, Q, masked, walk):
    import paper_2604_18913_amd as lkg
    rng = np.random.default_rng(E + Q)
    s, r, o = graph(E, rng)
    k = 3
    off = np.concatenate([[0], np.cumsum(rng.integers(0, 4, Q - 1)), [0]]).astype(np.int64)
    off[-1] = off[-2] + 2 if Q > 1 else 2
    seeds = rng.integers(0, min(E, 4000), int(off[-1])).astype(np.int32)
    seeds[-1] = 2
    mask = rng.integers(0, 512, (Q, 1)).astype(np.uint64) if masked else None
    g = lkg.Graph(s, r, o, E, 9)
    res = g.khop(off, seeds, k, mask, direction="pull", walk_exact=walk)
    want = oracle.khop(E, s, r, o, off, seeds, k, mask)
    assert np.array_equal(res.offsets(), want[0])
    if walk:
        w_off, w_ent = oracle.walk_levels(E, s, r, o, off, seeds, k, mask)
        for h in range(k + 1):
            at, ent = res.level(h)
            a = w_off[h * Q:(h + 1) * Q + 1]
            assert np.array_equal(at, a - a[0]) and np.array_equal(ent.cpu().numpy(), w_ent[a[0]:a[-1]])
    else:
        for got, w in zip(res.fetch(), want[1:]):
            assert np.array_equal(got.cpu().numpy(), w)
    push = g.khop(off, seeds, k, mask, direction="push", walk_exact=walk)
    for a, b in zip(res.hop_stats(), push.hop_stats()):
        for name in ("active_rows", "frontier_edges", "entities_reached"):
            assert a[name] == b[name], name
    push.close()
    res.close()
    g.close()
