"""Pushed hops: first hops whose objects are seeds of the same query, of others, or both; lines of few and of many words; short
rows and segments at their edges; planes of all widths, whitelists, walk-exact levels, shards."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shards", [0, 3])
@pytest.mark.parametrize("walk_exact", [False, True])
@pytest.mark.parametrize("Q, per_query, masked", [(3, 1, False), (64, 40, True), (65, 3, False), (256, 9, True), (257, 1, True),
                                                  (1024, 2, False), (1024, 30, True)])
def test_pushed_hops(Q, per_query, masked, walk_exact, shards):
    import paper_2604_18913_amd as lkg
    rng = np.random.default_rng(Q + per_query)
    E, R, k = 700, 7, 3
    deg = rng.choice([0, 1, 7, 8, 9, 16, 17, 32, 33, 64, 65, 129], E)
    s = np.repeat(np.arange(E), deg).astype(np.int32)
    o = np.where(rng.random(s.size) < 0.5, s // 3, rng.integers(0, E, s.size)).astype(np.int32)  # (loops, and seeds as objects)
    r = rng.integers(0, R, s.size).astype(np.int32)
    off = np.arange(0, Q * per_query + 1, per_query, dtype=np.int64)
    seeds = rng.integers(0, 40 if per_query > 5 else E, Q * per_query).astype(np.int32)
    mask = rng.integers(0, 2**R, (Q, 1)).astype(np.uint64) if masked else None
    g = lkg.Graph(s, r, o, E, R, num_shards=shards)
    res = g.khop(off, seeds, k, mask, direction="push", walk_exact=walk_exact)
    if walk_exact:
        level_off, entity = oracle.walk_levels(E, s, r, o, off, seeds, k, mask)
        for h in range(k + 1):
            want = level_off[h * Q:(h + 1) * Q + 1]
            at, ent = res.level(h)
            assert np.array_equal(at, want - want[0]) and np.array_equal(ent.cpu().numpy(), entity[want[0]:want[-1]]), h
    else:
        want = oracle.khop(E, s, r, o, off, seeds, k, mask)
        assert np.array_equal(res.offsets(), want[0])
        for got, w in zip(res.fetch(), want[1:]):
            assert np.array_equal(got.cpu().numpy(), w)
        # an entity that the hop has pushed into for its seeds only is in no later level
        reached = [len(np.unique(want[1][want[2] == h])) for h in range(1, k + 1)]
        assert [x["entities_reached"] for x in res.hop_stats()][:k] == reached
    res.close()
    g.close()
