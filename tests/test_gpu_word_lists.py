"""Entity lists without hop numbers of 16-word batches, level lists among them: whole batches, pages of one word, parts of
words, numbers of active entities on both sides of a tile, of a block of tiles and of a super tile."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("E", [63, 64, 65, 1023, 1025, 4111])
@pytest.mark.parametrize("Q, walk", [(257, True), (1000, False), (1024, True)])
def test_entity_lists(E, Q, walk):
    import paper_2604_18913_amd as lkg
    rng = np.random.default_rng(E + Q)
    R, T, k = 5, 3 * E, 2
    s, o = rng.integers(0, E, (2, T)).astype(np.int32)
    r = rng.integers(0, R, T).astype(np.int32)
    off = np.concatenate([[0], np.cumsum(rng.integers(0, 4, Q))]).astype(np.int64)
    seeds = rng.integers(0, E, int(off[-1])).astype(np.int32)
    g = lkg.Graph(s, r, o, E, R)
    res = g.khop(off, seeds, k, walk_exact=walk)
    pages = [(0, Q), (0, 1), (63, 65), (64, 128), (100, 101), (130, 250), (Q - 1, Q)]
    want_off, want_ent = oracle.khop(E, s, r, o, off, seeds, k)[:2]
    if walk:
        level_off, level_ent = oracle.walk_levels(E, s, r, o, off, seeds, k)
        for h in range(k + 1):
            a = level_off[h * Q:(h + 1) * Q + 1]
            for q0, q1 in pages:
                got_off, got = res.level(h, q0, q1)
                assert np.array_equal(got_off, a - a[0])
                assert np.array_equal(got.cpu().numpy(), level_ent[a[q0]:a[q1]]), (h, q0, q1)
    assert np.array_equal(res.offsets(), want_off)
    for q0, q1 in [] if walk else pages:
        got, hop, pred = res.fetch(q0, q1, want_hop=False, want_pred=False)
        assert hop is None and pred is None
        assert np.array_equal(got.cpu().numpy(), want_ent[want_off[q0]:want_off[q1]]), (q0, q1)
    res.close()
    g.close()


@pytest.mark.parametrize("E, degree", [(700, 2), (700, 60), (140_000, 3)])
def test_pages_on_both_sides_of_the_rule(E, degree):
    """Four and five words; few tiles and many; nearly all pairs reached and few of them."""
    import paper_2604_18913_amd as lkg
    rng = np.random.default_rng(E + degree)
    Q, R, k = 1024, 3, 2
    s, o = rng.integers(0, E, (2, E * degree)).astype(np.int32)
    r = rng.integers(0, R, len(s)).astype(np.int32)
    off = np.arange(Q + 1, dtype=np.int64)
    seeds = rng.integers(0, E, Q).astype(np.int32)
    want_off, want_ent = oracle.khop(E, s, r, o, off, seeds, k)[:2]
    level_off, level_ent = oracle.walk_levels(E, s, r, o, off, seeds, k)
    a = level_off[k * Q:(k + 1) * Q + 1]
    g = lkg.Graph(s, r, o, E, R)
    res, walk = g.khop(off, seeds, k), g.khop(off, seeds, k, walk_exact=True)
    for q0, q1 in ((0, 256), (0, 257), (63, 257), (64, 320), (70, 390), (1, 1024)):
        got = res.fetch(q0, q1, want_hop=False, want_pred=False)[0]
        assert np.array_equal(got.cpu().numpy(), want_ent[want_off[q0]:want_off[q1]]), (q0, q1)
        got = walk.level(k, q0, q1)[1]
        assert np.array_equal(got.cpu().numpy(), level_ent[a[q0]:a[q1]]), (q0, q1)
    res.close()
    walk.close()
    g.close()
