"""Rows of distinct (subject, object) pairs, which calls without whitelists walk where a graph holds parallel triples."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


def parallel_graph(rng, E, R, rows, extra, share):
    """rows[i] distinct subjects for object i, and `extra` pairs elsewhere; of all triples a share repeats earlier pairs."""
    s = np.concatenate([rng.choice(E, d, replace=False) for d in rows] + [rng.integers(0, E, extra)])
    o = np.concatenate([np.full(d, i) for i, d in enumerate(rows)] + [rng.integers(len(rows), E, extra)])
    again = rng.integers(0, len(s), int(len(s) * share / (1 - share)))
    s, o = np.concatenate([s, s[again]]), np.concatenate([o, o[again]])
    perm = rng.permutation(len(s))
    return s[perm].astype(np.int32), rng.integers(0, R, len(s)).astype(np.int32), o[perm].astype(np.int32)


def seed_lists(lists):
    return np.concatenate([[0], np.cumsum([len(x) for x in lists])]).astype(np.int64), np.concatenate(lists).astype(np.int32)


def compare(g, E, s, r, o, off, seeds, k):
    want = oracle.khop(E, s, r, o, off, seeds, k)
    res = g.khop(off, seeds, k)
    assert np.array_equal(res.offsets(), want[0])
    Q = len(off) - 1
    for q0, q1 in ((0, Q), (Q // 2, min(Q, Q // 2 + 20))):
        a, b = want[0][q0], want[0][q1]
        for x, y in zip(res.fetch(q0, q1), want[1:4]):
            assert np.array_equal(x.cpu().numpy(), y[a:b])
    res.close()


# rows at the edges of the short ones (32), of segments (1,024, 2,048) and of giants (8,192), by distinct subjects; shares of
# parallel triples below, about and above the one from which they are taken out
@pytest.mark.parametrize("share", [0.02, 0.12, 0.4, 0.9])
@pytest.mark.parametrize("Q, k", [(3, 2), (200, 3), (700, 3), (300, 7)])
def test_parallel_triples(Q, k, share):
    import paper_2604_18913_amd as lkg
    rng = np.random.default_rng(Q + k)
    E, R = 12_000, 30
    s, r, o = parallel_graph(rng, E, R, (1, 31, 32, 33, 64, 65, 1023, 1024, 1025, 2047, 2049, 8191, 8192, 9000), 20_000, share)
    off, seeds = seed_lists([rng.integers(0, E, 1 + q % 3) for q in range(Q)])
    for opts in ({}, {"host_build": True, "hub_min_degree": 60}, {"num_shards": 3}, {"num_shards": 3, "max_resident_shards": 2}):
        g = lkg.Graph(s, r, o, E, R, **opts)
        compare(g, E, s, r, o, off, seeds, k)
        res = g.khop(off, seeds, 2, direction="pull")
        want = oracle.khop(E, s, r, o, off, seeds, 2)
        for x, y in zip(res.fetch(), want[1:4]):
            assert np.array_equal(x.cpu().numpy(), y)
        res.close()
        g.close()


@pytest.mark.parametrize("Q", [5, 130, 600])
def test_walk_levels_of_parallel_triples(Q):
    import paper_2604_18913_amd as lkg
    rng = np.random.default_rng(Q)
    E, R = 3_000, 9
    s, r, o = parallel_graph(rng, E, R, (33, 1025, 2500), 6_000, 0.5)
    off, seeds = seed_lists([rng.integers(0, E, 2) for _ in range(Q)])
    g = lkg.Graph(s, r, o, E, R)
    res = g.khop(off, seeds, 3, walk_exact=True, direction="pull")
    want_off, want = oracle.walk_levels(E, s, r, o, off, seeds, 3)
    for h in range(4):
        got_off, got = res.level(h)
        a = want_off[h * Q:(h + 1) * Q + 1]
        assert np.array_equal(got_off, a - a[0]) and np.array_equal(got.cpu().numpy(), want[a[0]:a[-1]])
    res.close()
    g.close()


@pytest.mark.parametrize("T, pairs", [(1, 1), (2, 1), (70, 1), (1000, 1000)])
def test_tiny_graphs(T, pairs):
    import paper_2604_18913_amd as lkg
    rng = np.random.default_rng(T)
    s, o = (np.arange(T) % pairs % 40).astype(np.int32), (np.arange(T) % pairs // 40 % 40).astype(np.int32)
    r = rng.integers(0, 3, T).astype(np.int32)
    off, seeds = seed_lists([[i % 40] for i in range(70)])
    g = lkg.Graph(s, r, o, 41, 3)
    compare(g, 41, s, r, o, off, seeds, 3)
    g.close()


@pytest.mark.parametrize("share, kept", [(0.02, False), (0.18, False), (0.22, True), (0.9, True)])
def test_which_graphs_hold_them(share, kept):
    """.. and that calls without whitelists then walk them: by the entries that a pulled hop reads in the counting mode."""
    import paper_2604_18913_amd as lkg
    rng = np.random.default_rng(int(100 * share))
    E, R = 12_000, 30
    s, r, o = parallel_graph(rng, E, R, (1, 31, 32, 33, 64, 65, 1023, 1024, 1025), 60_000, share)
    T, pairs = len(s), len(np.unique(s.astype(np.int64) * E + o))
    off, seeds = seed_lists([rng.integers(0, E, 2) for _ in range(300)])
    for opts, kept_here in (({}, kept), ({"num_shards": 3}, kept), ({"num_shards": 3, "max_resident_shards": 2}, False), ({"host_build": True}, False)):
        g, none = lkg.Graph(s, r, o, E, R, **opts), lkg.Graph(s[:0], r[:0], o[:0], E, R, **opts)
        if not opts:
            held = g.info()["device_bytes"] - none.info()["device_bytes"]
            assert (held > 20 * T + 6 * T + 12 * pairs) == kept, held / T
            assert kept or held < 23 * T
        g.khop(off, seeds, 1, direction="pull").close()  # (a cache holds every unit from here on)
        g.profile_enable(2)
        res = g.khop(off, seeds, 1, walk_exact=True, direction="pull")  # (every row is read to its end, or for what is live)
        read = res.hop_stats()[0]["edges_scanned"]
        assert read <= (pairs if kept_here else T), (opts, read, pairs, T)
        res.close()
        res = g.khop(off, seeds, 1, np.full((300, 1), (1 << R) - 1, np.uint64), walk_exact=True, direction="pull")
        read_all = res.hop_stats()[0]["edges_scanned"]
        assert (read < read_all) == kept_here, (opts, read, read_all)
        res.close()
        g.profile_enable(0)
        compare(g, E, s, r, o, off, seeds, 2)
        g.close()
        none.close()
