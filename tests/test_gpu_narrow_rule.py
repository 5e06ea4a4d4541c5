"""Directions of narrow batches on graphs from which they pull earlier than at a twelfth of the triples: the rule, and lists and
levels against the oracle on both sides of it."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T", [(1 << 18) - 1, 1 << 18, 700_000])
@pytest.mark.parametrize("Q, masked", [(1, False), (50, False), (200, False), (200, True), (7, True)])
def test_rule(T, Q, masked):
    import paper_2604_18913_amd as lkg
    rng = np.random.default_rng(T + Q)
    E, R, k = 60_000, 6, 3
    hubs = rng.permutation(E)[:40]
    s = np.where(rng.random(T) < 0.3, hubs[rng.integers(0, 40, T)], rng.integers(0, E, T)).astype(np.int32)
    o = np.where(rng.random(T) < 0.2, hubs[rng.integers(0, 40, T)], rng.integers(0, E, T)).astype(np.int32)
    r = rng.integers(0, R, T).astype(np.int32)
    off = np.arange(Q + 1, dtype=np.int64)
    seeds = rng.integers(0, E, Q).astype(np.int32)
    seeds[::2] = hubs[0]  # a frontier of thousands of triples
    mask = rng.integers(1, 2**R, (Q, 1)).astype(np.uint64) if masked else None
    want = oracle.khop(E, s, r, o, off, seeds, k, mask)
    degree = np.bincount(s, minlength=E)
    few = T // 12
    if T >= 1 << 18:
        few = min(few, T * T >> 30) if not masked else 0 if Q > 64 else few
    g = lkg.Graph(s, r, o, E, R)
    res = g.khop(off, seeds, k, mask)
    assert np.array_equal(res.offsets(), want[0])
    for got, w in zip(res.fetch(), want[1:4]):
        assert np.array_equal(got.cpu().numpy(), w)
    for h, st in enumerate(res.hop_stats()):
        edges = int(degree[np.unique(want[1][want[2] == h])].sum())
        assert st["frontier_edges"] == edges
        if edges and (Q > 64 or edges > 2048):  # (smaller ones of up to 64 questions: one block, pushed)
            assert st["direction"] == lkg.binding.DIRECTIONS["pull" if edges > few else "push"], (h, edges, few)
    res.close()
    for walk in ((True,) if not masked else ()):
        w_off, w_ent = oracle.walk_levels(E, s, r, o, off, seeds, 2)
        res = g.khop(off, seeds, 2, walk_exact=True)
        for h in range(3):
            at, ent = res.level(h)
            a = w_off[h * Q:(h + 1) * Q + 1]
            assert np.array_equal(at, a - a[0]) and np.array_equal(ent.cpu().numpy(), w_ent[a[0]:a[-1]])
        res.close()
    g.close()


@pytest.mark.parametrize("T", [1 << 21, 3 << 20, 1 << 22, (1 << 22) + 1])
def test_whitelists_about_the_size_up_to_which_four_words_pull(T):
    import paper_2604_18913_amd as lkg
    E, R, Q, k = 600_000, 6, 65, 3
    rng = np.random.default_rng(T)
    s, o = rng.integers(0, E, (2, T)).astype(np.int32)
    r = rng.integers(0, R, T).astype(np.int32)
    off = np.arange(Q + 1, dtype=np.int64)
    seeds = rng.integers(0, E, Q).astype(np.int32)
    mask = rng.integers(1, 2**R, (Q, 1)).astype(np.uint64)
    want = oracle.khop(E, s, r, o, off, seeds, k, mask)
    degree = np.bincount(s, minlength=E)
    g = lkg.Graph(s, r, o, E, R)
    res = g.khop(off, seeds, k, mask)
    assert np.array_equal(res.offsets(), want[0])
    for got, w in zip(res.fetch(), want[1:4]):
        assert np.array_equal(got.cpu().numpy(), w)
    for h, st in enumerate(res.hop_stats()):
        edges = int(degree[np.unique(want[1][want[2] == h])].sum())
        line = 0 if T == 1 << 21 else T // 12 if T > 1 << 22 or h == k - 1 else 1024
        assert st["direction"] == lkg.binding.DIRECTIONS["pull" if edges > line else "push"], (h, edges)
    res.close()
    g.close()
