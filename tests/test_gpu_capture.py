"""A fetch recorded into a graph: it takes no memory, and every replay writes what an eager fetch writes."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


class Arena:
    """Device memory for a graph's pool, handed out once; counts the requests."""

    def __init__(self, nbytes):
        import torch
        self.block = torch.empty(nbytes, dtype=torch.uint8, device="cuda")
        self.at = (self.block.data_ptr() + 255) // 256 * 256
        self.end = self.block.data_ptr() + nbytes
        self.requests = 0

    def alloc(self, nbytes):
        self.requests += 1
        p = self.at
        if p + nbytes > self.end:
            return 0
        self.at = p + (nbytes + 255) // 256 * 256
        return p

    def free(self, address):
        pass


def captured_fetch(res, arena, q0, q1):
    """-> the lists of three replays, with eager work on the graph's pool between them."""
    import torch
    off = res.offsets()
    n = int(off[q1] - off[q0])
    out = (torch.empty(n, dtype=torch.int32, device="cuda"), torch.empty(n, dtype=torch.uint8, device="cuda"),
           torch.empty(n, dtype=torch.int32, device="cuda"))
    torch.cuda.synchronize()
    before = arena.requests
    rec = torch.cuda.CUDAGraph()
    with torch.cuda.graph(rec):
        res.fetch(q0, q1, out=out)
    assert arena.requests == before
    lists = []
    for _ in range(3):
        for x in out:
            x.fill_(77)
        rec.replay()
        torch.cuda.synchronize()
        lists.append([x.cpu().numpy() for x in out])
        res.fetch(q0, q1)
        torch.cuda.synchronize()
    return lists


@pytest.mark.parametrize("masked", [False, True])
@pytest.mark.parametrize("Q, overlap", [(40, False), (40, True), (200, False), (200, True)])
def test_giant_rows_on_narrow_planes(Q, overlap, masked, monkeypatch):
    import paper_2604_18913_amd as lkg
    if overlap:
        monkeypatch.setenv("LOGOSKG_OVERLAP_FETCH", "1")
    rng = np.random.default_rng(Q)
    E, T, R, k = 5000, 40_000, 40, 3
    s, o, r = (rng.integers(0, n, T).astype(np.int32) for n in (E, E, R))
    o[:9000], o[9000:26_000], o[26_000:28_000] = 1, 2, rng.integers(10, 20, 2000)
    off = np.arange(Q + 1, dtype=np.int64) * 3
    seeds = rng.integers(0, E, 3 * Q).astype(np.int32)
    mask = None
    if masked:
        mask = np.zeros((Q, 1), np.uint64)
        for b in range(R):
            mask[:, 0] |= (rng.random(Q) < 0.3).astype(np.uint64) << np.uint64(b)
    want = oracle.khop(E, s, r, o, off, seeds, k, mask)
    arena = Arena(256 << 20)
    g = lkg.Graph(s, r, o, E, R, dev_alloc=arena.alloc, dev_free=arena.free)
    res = g.khop(off, seeds, k, mask)
    for q0, q1 in ((0, Q), (7, Q - 5)):
        for got in captured_fetch(res, arena, q0, q1):
            for x, y in zip(got, want[1:4]):
                assert np.array_equal(x, y[want[0][q0]:want[0][q1]])
    res.close()
    g.close()


def test_a_page_whose_words_an_eager_fetch_packs():
    import paper_2604_18913_amd as lkg
    rng = np.random.default_rng(4)
    E, T, Q = 4_400_000, 9_000_000, 300
    s, o = rng.integers(0, E, T, dtype=np.int32), rng.integers(0, E, T, dtype=np.int32)
    r = np.zeros(T, np.int32)
    o[:30_000] = np.arange(30_000) % 3
    lists = [rng.integers(0, E, 3) for _ in range(Q)]
    lists[7] = rng.permutation(E)[:4_300_000]  # one question seeds most of the graph: all of it is listed
    off = np.concatenate([[0], np.cumsum([len(x) for x in lists])]).astype(np.int64)
    arena = Arena(6 << 30)
    g = lkg.Graph(s, r, o, E, 1, dev_alloc=arena.alloc, dev_free=arena.free)
    res = g.khop(off, np.concatenate(lists).astype(np.int32), 2)
    res.fetch()  # the buffers that the first fetch of more than 256 queries makes; five words of the lines: not packed
    for q0, q1 in ((64, 128), (130, 250)):
        lists = captured_fetch(res, arena, q0, q1)
        want = [x.cpu().numpy() for x in res.fetch(q0, q1)]
        for got in lists:
            assert all(np.array_equal(x, y) for x, y in zip(got, want))
    res.close()
    g.close()


def test_levels_resolved_from_the_subject_side():
    import kggen
    import paper_2604_18913_amd as lkg
    w = kggen.config2(0.01, num_queries=300)
    want = oracle.khop(w.num_entities, w.subj, w.rel, w.obj, w.seed_off, w.seeds, w.k)
    arena = Arena(1 << 30)
    g = lkg.Graph(w.subj, w.rel, w.obj, w.num_entities, w.num_relations, hub_min_degree=100, dev_alloc=arena.alloc,
                  dev_free=arena.free)
    res = g.khop(w.seed_off, w.seeds, w.k)
    assert any(4 * h["frontier_edges"] <= w.num_triples for h in res.hop_stats())
    res.fetch()
    for q0, q1 in ((0, 300), (60, 140)):
        for got in captured_fetch(res, arena, q0, q1):
            for x, y in zip(got, want[1:4]):
                assert np.array_equal(x, y[want[0][q0]:want[0][q1]])
    res.close()
    g.close()
