"""Searches that one block takes (up to 64 queries with small frontiers): the limits at which it hands over
to the general kernels, and its lists against the oracle."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


def check(E, s, r, o, R, off, seeds, k, mask=None, direction="auto"):
    import paper_2604_18913_amd as lkg
    g = lkg.Graph(s, r, o, E, R)
    res = g.khop(off, seeds, k, mask, direction=direction)
    want = oracle.khop(E, s, r, o, off, seeds, k, mask)
    assert np.array_equal(res.offsets(), want[0])
    Q = len(off) - 1
    for q0, q1 in {(0, Q), (Q // 2, Q), (Q // 3, Q // 3 + 1)}:
        ent, hop, pred = res.fetch(q0, q1)
        a, b = want[0][q0], want[0][q1]
        assert np.array_equal(ent.cpu().numpy(), want[1][a:b])
        assert np.array_equal(hop.cpu().numpy(), want[2][a:b])
        assert np.array_equal(pred.cpu().numpy(), want[3][a:b])
    ent, _, _ = res.fetch(0, Q, want_hop=False, want_pred=False)
    assert np.array_equal(ent.cpu().numpy(), want[1])
    if k and direction != "pull":
        pull = g.khop(off, seeds, k, mask, direction="pull")  # never takes the one-block path
        for a, b in zip(res.hop_stats(), pull.hop_stats()):
            for name in ("active_rows", "frontier_edges", "entities_reached"):
                assert a[name] == b[name], name
            if direction == "push":
                assert a["direction"] in (0, 1)
        pull.close()
    stats = res.hop_stats()
    res.close()
    g.close()
    return stats


def seed_lists(lists):
    off = np.concatenate([[0], np.cumsum([len(x) for x in lists])]).astype(np.int64)
    return off, np.concatenate(lists).astype(np.int32)


@pytest.mark.parametrize("masked", [False, True])
@pytest.mark.parametrize("Q, k, direction", [(1, 0, "auto"), (1, 2, "auto"), (64, 2, "push"), (63, 3, "auto"),
                                              (17, 5, "push"), (5, 16, "push"), (5, 17, "push"), (3, 40, "auto")])
def test_sparse_random_graphs(Q, k, direction, masked):
    rng = np.random.default_rng(100 * Q + k)
    E, T, R = 9001, 14000, 70
    s, o, r = (rng.integers(0, n, T).astype(np.int32) for n in (E, E, R))
    off, seeds = seed_lists([rng.integers(0, E, rng.integers(0, 4)) for _ in range(Q - 1)] + [np.array([5, 5, 7])])
    mask = None
    if masked:
        mask = rng.integers(0, 2**63, (Q, 2)).astype(np.uint64) | rng.integers(0, 2**63, (Q, 2)).astype(np.uint64)
        mask[:, 1] &= np.uint64(63)
    check(E, s, r, o, R, off, seeds, k, mask, direction)


@pytest.mark.parametrize("edges", [2047, 2048, 2049])
@pytest.mark.parametrize("hop", [1, 2])
def test_frontier_at_the_limit_of_one_block(edges, hop):
    # entity 0 (or 0 -> 1 .. 40) has `edges` out-triples in all; a tail behind their objects
    rng = np.random.default_rng(edges + hop)
    E, R, pad = 30000, 3, 40000
    first = np.zeros(40, np.int64) if hop == 2 else np.zeros(0, np.int64)
    src = 1 + np.arange(edges) % 40 if hop == 2 else np.zeros(edges, np.int64)
    dst = 100 + rng.permutation(12000)[:edges]
    s = np.concatenate([first, src, dst[:900], rng.integers(20000, E, pad)])
    o = np.concatenate([1 + np.arange(len(first)), dst, rng.integers(100, 12100, 900), rng.integers(20000, E, pad)])
    perm = rng.permutation(len(s))
    s, o = s[perm].astype(np.int32), o[perm].astype(np.int32)
    r = rng.integers(0, R, len(s)).astype(np.int32)
    off, seeds = seed_lists([np.array([0]), np.array([25000]), np.array([0, 3])])
    check(E, s, r, o, R, off, seeds, 4, direction="push")


@pytest.mark.parametrize("n_seeds", [1, 2047, 2048, 2049])
def test_many_seeds_and_more_reached_entities_than_the_list_holds(n_seeds):
    rng = np.random.default_rng(n_seeds)
    E, T, R = 20000, 30000, 2
    s, o, r = (rng.integers(0, n, T).astype(np.int32) for n in (E, E, R))
    off, seeds = seed_lists([rng.integers(0, E, n_seeds)])
    check(E, s, r, o, R, off, seeds, 3, direction="push")


def test_dense_words_and_hubs():
    # 64 queries on the same seeds (pairs above the limit), a subject of 60,000 triples, parallel triples
    rng = np.random.default_rng(9)
    E, R = 70000, 5
    s = np.concatenate([np.zeros(60000, np.int64), np.repeat(np.arange(1, 900), 2), rng.integers(1000, E, 300000)])
    o = np.concatenate([rng.integers(1000, E, 60000), rng.integers(1, 1000, 1798), rng.integers(1000, E, 300000)])
    r = rng.integers(0, R, len(s))
    o[60000:60050] = 0
    perm = rng.permutation(len(s))
    s, o, r = (x[perm].astype(np.int32) for x in (s, o, r))
    off, seeds = seed_lists([np.arange(1, 900) if q % 2 else np.array([q + 1]) for q in range(64)][:4])
    check(E, s, r, o, R, off, seeds, 3)
    off, seeds = seed_lists([np.array([1, 2, 3, 4, 5 + q]) for q in range(64)])
    check(E, s, r, o, R, off, seeds, 3)
    check(E, s, r, o, R, off, seeds, 3, direction="push")


def test_bad_seeds_are_refused():
    import paper_2604_18913_amd as lkg
    g = lkg.Graph([0, 1], [0, 0], [1, 2], 3, 1)
    for off, seeds in (([0, 1], [3]), ([0, 1], [-1]), ([0, 2], [0]), ([1, 1], [0]), ([0, 2, 1], [0])):
        with pytest.raises(lkg.LogosKGError) as err:
            g.khop(np.array(off, np.int64), np.array(seeds, np.int32), 1)
        assert err.value.status == 1
    res = g.khop(np.array([0, 1], np.int64), np.array([0], np.int32), 2)
    assert list(res.offsets()) == [0, 3]
    res.close()
    g.close()


def test_lists_of_a_host_built_graph_take_no_memory():
    import paper_2604_18913_amd as lkg
    rng = np.random.default_rng(3)
    E, T, R = 9001, 14000, 5
    s, o, r = (rng.integers(0, n, T).astype(np.int32) for n in (E, E, R))
    off, seeds = seed_lists([rng.integers(0, E, 2) for _ in range(30)])
    want = oracle.khop(E, s, r, o, off, seeds, 2)
    g = lkg.Graph(s, r, o, E, R, host_build=True)
    for triple_indices in (False, True):  # (the path listing builds them)
        if triple_indices:
            g.paths(res, np.zeros(1, np.int32), want[1][:1])
            res.close()
        res = g.khop(off, seeds, 2)
        assert np.array_equal(res.offsets(), want[0])
        held = g.info()["device_bytes"]
        for q0, q1 in ((0, 30), (4, 9)):
            got = res.fetch(q0, q1)
            assert g.info()["device_bytes"] == held
            for x, y in zip(got, want[1:4]):
                assert np.array_equal(x.cpu().numpy(), y[want[0][q0]:want[0][q1]])
    res.close()
    g.close()
