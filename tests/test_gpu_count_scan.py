"""Counts whose prefixes are made by the last blocks of the count kernels: one, several and just filled super and mega tiles
on every plane width, lists of active entities in one launch and in three, counts of levels behind counts of the reached."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("E", [1, 64, 1024, 1025, 65_536, 65_537, 200_001, 1 << 20, (1 << 20) + 1])
@pytest.mark.parametrize("Q", [3, 64, 200, 300, 1024])
def test_counts(E, Q):
    import paper_2604_18913_amd as lkg
    rng = np.random.default_rng(E + Q)
    T = min(4 * E, 60_000)
    s, o = (rng.integers(0, E, T).astype(np.int32) for _ in range(2))
    s[:T // 4] = s[0]  # a hub, so that a search reaches entities all over the graph
    r = np.zeros(T, dtype=np.int32)
    off = np.arange(Q + 1, dtype=np.int64)
    seeds = np.where(rng.random(Q) < 0.3, s[0], rng.integers(0, E, Q)).astype(np.int32)
    seeds[-1] = E - 1
    g = lkg.Graph(s, r, o, E, 1)
    want = oracle.khop(E, s, r, o, off, seeds, 2)
    for direction in ("auto", "pull"):  # twice: the tickets are put back
        res = g.khop(off, seeds, 2, direction=direction)
        assert np.array_equal(res.offsets(), want[0])
        for got, w in zip(res.fetch(), want[1:]):
            assert np.array_equal(got.cpu().numpy(), w)
        for h in range(3):
            at, ent = res.level(h)
            on = want[2] == h
            assert np.array_equal(ent.cpu().numpy(), want[1][on])
            assert np.array_equal(at, np.concatenate([[0], np.cumsum(on)])[want[0]])
        res.close()
    g.close()


@pytest.mark.parametrize("E", [64, 1000, 3 * 1024 + 70])
@pytest.mark.parametrize("Q", [64, 256, 700, 1024])
def test_counts_of_full_tiles(E, Q):
    """Every second query reaches every entity: all bits of a tile's counts."""
    import paper_2604_18913_amd as lkg
    s = np.concatenate([np.zeros(E), np.ones(E // 2)]).astype(np.int32)
    o = np.concatenate([np.arange(E), np.arange(E // 2) * 2 + 1]).astype(np.int32)
    r = np.zeros(s.size, dtype=np.int32)
    off = np.arange(Q + 1, dtype=np.int64)
    seeds = (np.arange(Q) % 5 % 2).astype(np.int32)
    g = lkg.Graph(s, r, o, E, 1)
    want = oracle.khop(E, s, r, o, off, seeds, 1)
    res = g.khop(off, seeds, 1)
    assert np.array_equal(res.offsets(), want[0])
    for got, w in zip(res.fetch(), want[1:]):
        assert np.array_equal(got.cpu().numpy(), w)
    res.close()
    g.close()
