"""Path listing where it can go wrong: rows longer than a scan step, each number of wavefronts per
pair, the seeds' side with repeated seeds, too many seeds and more matches than its table holds."""
import numpy as np
import pytest

import kggen
import oracle

pytestmark = pytest.mark.gpu


def hub_graph(rng, E, R, T):
    """Half of the triples end in four hubs (rows of thousands of entries); entity 0 reaches hub 1 through
    300 relations."""
    s, r, o = rng.integers(0, E, T), rng.integers(0, R, T), rng.integers(0, E, T)
    o[: T // 2] = 1 + rng.integers(0, 4, T // 2)
    s[: T // 4] = 1 + rng.integers(0, 40, T // 4)
    s = np.concatenate([s, np.zeros(300, np.int64)])
    r = np.concatenate([r, np.arange(300)])
    o = np.concatenate([o, np.ones(300, np.int64)])
    perm = rng.permutation(s.shape[0])
    return s[perm].astype(np.int32), r[perm].astype(np.int32), o[perm].astype(np.int32)


@pytest.mark.parametrize("share", [None, 0.5, 0.02])  # of the relations on a query's whitelist
@pytest.mark.parametrize("max_paths", [16, 3])
def test_long_rows_every_width_and_both_sides(share, max_paths):
    import paper_2604_18913_amd as lkg
    rng = np.random.default_rng(11)
    E, R, T, Q, k = 3000, 600, 40000, 70, 3
    s, r, o = hub_graph(rng, E, R, T)
    lists = [np.array([0, 0, 7]), np.array([0])]                       # a repeated seed; the parallel triples
    lists += [rng.integers(0, E, 100) for _ in range(4)]               # more seeds than the seeds' side takes
    lists += [rng.integers(0, E, rng.integers(1, 4)) for _ in range(Q - len(lists))]
    off = np.concatenate([[0], np.cumsum([len(x) for x in lists])]).astype(np.int64)
    seeds = np.concatenate(lists).astype(np.int32)
    mask = None
    if share is not None:
        keep = rng.random((Q, R)) < share
        keep[:2, :300] = True
        mask = np.zeros((Q, (R + 63) // 64), np.uint64)
        for w in range(R):
            mask[:, w // 64] |= keep[:, w].astype(np.uint64) << np.uint64(w % 64)
    g = lkg.Graph(s, r, o, E, R)
    res = g.khop(off, seeds, k, mask)
    ent, _, _ = res.fetch()
    reached = res.offsets()
    pq, pt = kggen.sample_reached_pairs(3, reached, ent.cpu().numpy(), 1500)
    pq = np.concatenate([pq, [0, 0, 1, 1, 2, 3], rng.integers(0, Q, 200)]).astype(np.int32)
    pt = np.concatenate([pt, [1, 2, 1, 3, 1, 1], rng.integers(0, E, 200)]).astype(np.int32)
    cnt_o, edges_o = oracle.paths(E, s, r, o, off, seeds, k, pq, pt, max_paths, mask)
    for n in (5, 1024, len(pq), 65536 + 7):  # 16, 16, 4 and 1 wavefronts per pair
        at = np.arange(n) % len(pq)
        if n == 5:
            at = len(pq) - 201 - np.arange(5)
        cnt, edges = g.paths(res, pq[at], pt[at], max_paths)
        assert np.array_equal(cnt.cpu().numpy(), cnt_o[at])
        assert np.array_equal(edges.cpu().numpy(), edges_o[at])
    res.close()
    g.close()


@pytest.mark.parametrize("R", [1, 63, 64, 65, 2047, 2048, 2049])  # the LDS whitelist's words and its limit
def test_whitelist_in_lds_and_gathered(R):
    import paper_2604_18913_amd as lkg
    rng = np.random.default_rng(R)
    E, Q, k, rows = 400, 5, 2, (R - 1, R, R + 1, 3 * R + 7)  # triples ending in the entities 0 .. 3
    o = np.concatenate([np.full(n, v) for v, n in enumerate(rows)] + [rng.integers(4, E, 3000)]).astype(np.int32)
    s = rng.integers(4, 60, o.shape[0]).astype(np.int32)
    r = rng.integers(0, R, o.shape[0]).astype(np.int32)
    off = np.arange(0, 70 * Q + 1, 70).astype(np.int64)  # more seeds than the seeds' side takes: rows are scanned
    seeds = rng.integers(4, E, 70 * Q).astype(np.int32)
    keep = rng.random((Q, R)) < 0.3
    keep[:, -1] = True
    mask = np.zeros((Q, (R + 63) // 64), np.uint64)
    for w in range(R):
        mask[:, w // 64] |= keep[:, w].astype(np.uint64) << np.uint64(w % 64)
    pq = np.repeat(np.arange(Q), 5).astype(np.int32)
    pt = np.tile([0, 1, 2, 3, 4], Q).astype(np.int32)
    cnt_o, edges_o = oracle.paths(E, s, r, o, off, seeds, k, pq, pt, 16, mask)
    assert cnt_o.max() > 0
    g = lkg.Graph(s, r, o, E, R)
    res = g.khop(off, seeds, k, mask)
    cnt, edges = g.paths(res, pq, pt, 16)
    assert np.array_equal(cnt.cpu().numpy(), cnt_o)
    assert np.array_equal(edges.cpu().numpy(), edges_o)
    res.close()
    g.close()


@pytest.mark.parametrize("longest", [20, 127, 128, 129])  # up to 128 entries every pair is one wavefront's, four to a block
@pytest.mark.parametrize("shards", [1, 3])
@pytest.mark.parametrize("share", [None, 0.5])
def test_graphs_of_short_rows(longest, shards, share):
    import paper_2604_18913_amd as lkg
    rng = np.random.default_rng(longest)
    E, R, Q, k = 400, 70, 70, 4
    o = np.concatenate([np.repeat([0, 1], [longest, max(longest - 64, 1)]),
                        np.repeat(np.arange(2, E), rng.integers(0, 16, E - 2))]).astype(np.int32)
    s = rng.integers(0, E, o.shape[0]).astype(np.int32)
    r = rng.integers(0, R, o.shape[0]).astype(np.int32)
    perm = rng.permutation(o.shape[0])
    s, r, o = s[perm], r[perm], o[perm]
    off = np.arange(0, 3 * Q + 1, 3).astype(np.int64)
    seeds = rng.integers(0, E, 3 * Q).astype(np.int32)
    mask = None
    if share is not None:
        keep = rng.random((Q, R)) < share
        mask = np.zeros((Q, 2), np.uint64)
        for w in range(R):
            mask[:, w // 64] |= keep[:, w].astype(np.uint64) << np.uint64(w % 64)
    g = lkg.Graph(s, r, o, E, R, num_shards=shards)
    res = g.khop(off, seeds, k, mask)
    ent, _, _ = res.fetch()
    pq, pt = kggen.sample_reached_pairs(5, res.offsets(), ent.cpu().numpy(), 1200)
    pq = np.concatenate([pq, np.arange(Q), np.arange(Q), rng.integers(0, Q, 60), [-1, Q, 0, 0]]).astype(np.int32)
    pt = np.concatenate([pt, np.zeros(Q), np.ones(Q), rng.integers(0, E, 60), [0, 0, -1, E]]).astype(np.int32)
    inside = slice(0, len(pq) - 4)  # (the last four lie outside the batch or the graph: no paths)
    for max_paths in (1, 16):
        cnt_o, edges_o = oracle.paths(E, s, r, o, off, seeds, k, pq[inside], pt[inside], max_paths, mask)
        assert cnt_o.max() == max_paths or share is not None
        cnt_o = np.concatenate([cnt_o, np.zeros(4, cnt_o.dtype)])
        edges_o = np.concatenate([edges_o, np.full((4, max_paths, k), -1, edges_o.dtype)])
        for n in (1, 2, 3, 5, len(pq)):
            at = len(pq) - n + np.arange(n)
            cnt, edges = g.paths(res, pq[at], pt[at], max_paths)
            assert np.array_equal(cnt.cpu().numpy(), cnt_o[at])
            assert np.array_equal(edges.cpu().numpy().reshape(edges_o[at].shape), edges_o[at])
    res.close()
    g.close()


@pytest.mark.parametrize("share", [None, 0.3])
@pytest.mark.parametrize("exact", [False, True])
def test_seeds_with_rows_of_all_lengths(share, exact):
    """Rows of the seeds around the numbers of threads and matches of a block, long rows on levels 1, 2 and 3 above them."""
    import paper_2604_18913_amd as lkg
    rng = np.random.default_rng(5)
    degrees = [1, 63, 64, 65, 255, 256, 257, 300, 850, 1023, 1024, 1025, 4096, 4097, 16384, 16385]
    Q, R, mid, tops = len(degrees), 40, 50, 6
    m0, t0 = Q, Q + mid  # seeds | middles | tops
    E = t0 + tops + 200
    s = [np.repeat(np.arange(Q), degrees), m0 + rng.integers(0, mid, 2400), t0 + rng.integers(0, 3, 900), rng.integers(t0 + tops, E, 9000)]
    o = [m0 + rng.integers(0, mid, sum(degrees)), t0 + rng.integers(0, 3, 2400), t0 + 3 + rng.integers(0, 3, 900), rng.integers(m0, t0, 9000)]
    s, o = np.concatenate(s).astype(np.int32), np.concatenate(o).astype(np.int32)
    perm = rng.permutation(len(s))
    s, o = s[perm], o[perm]
    r = rng.integers(0, R, len(s)).astype(np.int32)
    mask = None
    if share is not None:
        mask = ((rng.random((Q, R)) < share).astype(np.uint64) << np.arange(R, dtype=np.uint64)).sum(1, dtype=np.uint64)[:, None]
    off, seeds = 2 * np.arange(Q + 1, dtype=np.int64), np.repeat(np.arange(Q), 2).astype(np.int32)  # (every seed twice)
    g = lkg.Graph(s, r, o, E, R)
    res = g.khop(off, seeds, 3, mask, walk_exact=exact)
    pq, pt = (x.ravel().astype(np.int32) for x in np.meshgrid(np.arange(Q), np.arange(m0, t0 + tops), indexing="ij"))
    length = np.where(pt < t0, 1, np.where(pt < t0 + 3, 2, 3)).astype(np.int32)
    for max_paths in (3, 16):
        if exact:
            cnt_o, edges_o = oracle.walk_paths(E, s, r, o, off, seeds, 3, pq, pt, length, max_paths, mask)
        else:
            cnt_o, edges_o = oracle.paths(E, s, r, o, off, seeds, 3, pq, pt, max_paths, mask)
        assert cnt_o.max() == max_paths
        for n in (len(pq), 1025, 65536 + 1):  # 16, 4 and 1 wavefronts per pair
            at = np.arange(n) % len(pq)
            cnt, edges = g.walks(res, pq[at], pt[at], length[at], max_paths) if exact else g.paths(res, pq[at], pt[at], max_paths)
            assert np.array_equal(cnt.cpu().numpy(), cnt_o[at])
            assert np.array_equal(edges.cpu().numpy(), edges_o[at])
    res.close()
    g.close()
