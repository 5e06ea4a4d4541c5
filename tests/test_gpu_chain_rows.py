"""Chain counts over object rows at the edges of the counting kernels: short rows, the turns of the four-
and sixteen-wavefront kernels, and sums past the limit."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

DEGREES = (1, 3, 4, 5, 31, 32, 33, 64, 511, 512, 513, 1025, 8191, 8192, 4097 * 3)


@pytest.mark.parametrize("masked", [False, True])
def test_rows_of_every_class(masked):
    import paper_2604_18913_amd as lkg
    rng = np.random.default_rng(5)
    N, R = 700, 9                                    # seed 0, subjects 1 .. N, then a target per degree
    E = 1 + N + len(DEGREES)
    sro = [(0, rr, m) for m in range(1, N + 1) for rr in range(1 + m % 3)]
    for i, d in enumerate(DEGREES):
        sro += [(int(rng.integers(1, N + 1)), int(rng.integers(0, R)), 1 + N + i) for _ in range(d)]
    sro = np.array(sro, np.int64)[rng.permutation(len(sro))]
    s, r, o = (np.ascontiguousarray(sro[:, i], dtype=np.int32) for i in range(3))
    allowed = np.ones(R, bool)
    if masked:
        allowed[[1, 5, 6]] = False
    mask = np.full((1, 1), sum(1 << i for i in range(R) if allowed[i]), np.uint64) if masked else None
    ok = allowed[r]
    first = {m: np.flatnonzero((o == m) & ok) for m in range(1, N + 1)}
    want_e, want_t = [], []
    for i in range(len(DEGREES)):
        for t2 in np.flatnonzero((o == 1 + N + i) & ok):
            f = first[int(s[t2])]
            want_e.append(np.stack([f, np.full(len(f), t2)], 1))
            want_t.append(np.full(len(f), 1 + N + i))
    want_e, want_t = np.concatenate(want_e), np.concatenate(want_t)
    g = lkg.Graph(s, r, o, E, R)
    res = g.khop(np.array([0, 1], np.int64), np.zeros(1, np.int32), 2, mask, walk_exact=True)
    assert res.walks_count(0, 2) == len(want_t)
    edges, target = res.walks_fetch(0, 2, 0, len(want_t))
    assert np.array_equal(edges.cpu().numpy(), want_e) and np.array_equal(target.cpu().numpy(), want_t)
    res.close()
    g.close()


@pytest.mark.parametrize("parallel, last_that_fits", [(32, 11), (4096, 4), (9000, 4)])
def test_too_many_chains_are_refused_whatever_the_row(parallel, last_that_fits):
    import paper_2604_18913_amd as lkg
    # two entities joined by `parallel` triples each way: parallel^h chains of h triples
    r = np.concatenate([np.arange(parallel)] * 2).astype(np.int32)
    s = np.repeat(np.array([0, 1], np.int32), parallel)
    g = lkg.Graph(s, r, 1 - s, 2, parallel)
    res = g.khop(np.array([0, 1], np.int64), np.zeros(1, np.int32), last_that_fits + 1, walk_exact=True)
    assert res.walks_count(0, last_that_fits) == parallel ** last_that_fits
    with pytest.raises(lkg.LogosKGError) as err:
        res.walks_count(0, last_that_fits + 1)
    assert err.value.status == 4
    res.close()
    g.close()


@pytest.mark.parametrize("parallel, hops, last", [(8192, 4, 16), (4096, 4, 256), (1 << 14, 3, 1 << 14)])
@pytest.mark.parametrize("missing", [0, 1])
def test_the_sum_of_a_row_at_the_limit(parallel, hops, last, missing):
    import paper_2604_18913_amd as lkg
    # entities 0 .. hops, neighbours joined by `parallel` triples, then a row of `last` triples from the last of
    # them: parallel^hops * last = 2^56 chains end in it, which is one entry too many
    assert parallel ** hops * last == 1 << 56
    n = last - missing
    s = np.concatenate([np.repeat(np.arange(hops), parallel), np.full(n, hops)]).astype(np.int32)
    r = np.concatenate([np.tile(np.arange(parallel), hops), np.arange(n)]).astype(np.int32)
    g = lkg.Graph(s, r, s + 1, hops + 2, max(parallel, last))
    res = g.khop(np.array([0, 1], np.int64), np.zeros(1, np.int32), hops + 1, walk_exact=True)
    if missing:
        assert res.walks_count(0, hops + 1) == parallel ** hops * n
        edges, target = res.walks_fetch(0, hops + 1, parallel ** hops * n - 3, 3)
        assert np.array_equal(target.cpu().numpy(), np.full(3, hops + 1))
        assert edges.cpu().numpy()[:, -1].tolist() == [parallel * hops + n - 1] * 3
    else:
        with pytest.raises(lkg.LogosKGError) as err:
            res.walks_count(0, hops + 1)
        assert err.value.status == 4
    res.close()
    g.close()
