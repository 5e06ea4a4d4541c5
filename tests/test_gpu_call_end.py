"""How a k-hop call ends: what a call that fails behind its hops leaves to the next one, and that its stream is idle."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

E, T, R = 4_000_000, 40_000_000, 5  # (a hop of some hundred microseconds)


@pytest.fixture(scope="module")
def triples():
    rng = np.random.default_rng(11)
    s, o = rng.integers(0, E, T).astype(np.int32), rng.integers(0, E, T).astype(np.int32)
    s[:20_000_000], s[20_000_000:20_003_000], o[30_000_000:30_050_000] = 7, 8, 9
    return s, rng.integers(0, R, T).astype(np.int32), o


def batch(rng, Q, few):
    off = np.arange(Q + 1, dtype=np.int64) * 2
    seeds = rng.integers(0, E, 2 * Q).astype(np.int32)
    seeds[0 if few else slice(0, None, 4)] = 8 if few else 7  # (more than a small search takes)
    return off, seeds


class Refusing:
    """Device memory by torch; turns requests down while `refuse` says so."""

    def __init__(self):
        self.held, self.refuse, self.refused, self.calls = {}, None, 0, 0

    def alloc(self, nbytes):
        import torch
        self.calls += 1
        if self.refuse is not None and self.calls > self.refuse:
            self.refused += 1
            return 0
        t = torch.empty(nbytes, dtype=torch.uint8, device="cuda:0")
        self.held[t.data_ptr()] = t
        return t.data_ptr()

    def free(self, address):
        del self.held[address]


@pytest.mark.parametrize("k", [2, 3])
@pytest.mark.parametrize("Q, direction", [(3, "auto"), (200, "auto"), (200, "pull"), (400, "auto")])
def test_a_call_behind_one_without_room_for_its_counts(triples, Q, direction, k):
    """The first call runs all its hops and finds no room for the tables of the counts; the second follows at once, on
    the same stream and on another one, and reads nothing of the first one's counters (the last level's are written
    to the words of level 0 where k is even)."""
    import torch
    import paper_2604_18913_amd as lkg
    s, r, o = triples
    rng = np.random.default_rng(Q + k)
    mem = Refusing()
    g = lkg.Graph(s, r, o, E, R, dev_alloc=mem.alloc, dev_free=mem.free)
    first, second = batch(rng, Q, False), batch(rng, Q, True)
    want = oracle.khop(E, s, r, o, *second, k)
    seed_degree = np.bincount(s, minlength=E)[np.unique(second[1])]
    inputs = [torch.from_numpy(x).cuda() for x in (*first, *second)]  # (nothing but the calls between the two)
    other = torch.cuda.Stream()
    torch.cuda.synchronize()
    for stream in (None, other):
        res = g.khop(*inputs[:2], k, direction=direction, counts=False)  # the planes and the seeds are in the pool
        res.close()
        torch.cuda.synchronize()
        mem.refuse, mem.refused = mem.calls, 0
        with pytest.raises(lkg.LogosKGError) as err:
            g.khop(*inputs[:2], k, direction=direction)
        assert err.value.status == 2 and mem.refused >= 2  # (once more behind a trim)
        mem.refuse = None
        res = g.khop(*inputs[2:], k, direction=direction, stream=stream)
        assert np.array_equal(res.offsets(), want[0])
        reached = [len(np.unique(want[1][want[2] == h])) for h in range(1, k + 1)]
        stats = res.hop_stats()
        assert [x["entities_reached"] for x in stats] == reached
        assert (stats[0]["active_rows"], stats[0]["frontier_edges"]) == (np.count_nonzero(seed_degree), seed_degree.sum())
        torch.cuda.synchronize()
        for got, w in zip(res.fetch(), want[1:]):
            assert np.array_equal(got.cpu().numpy(), w)
        res.close()
        torch.cuda.synchronize()
        g.close()
        g = lkg.Graph(s, r, o, E, R, dev_alloc=mem.alloc, dev_free=mem.free)
    g.close()


@pytest.mark.parametrize("shards", [0, 3])
@pytest.mark.parametrize("Q, direction, walk", [(1, "auto", False), (3, "auto", False), (3, "pull", True), (64, "push", False),
                                                (200, "auto", False), (200, "auto", True), (200, "pull", False),
                                                (400, "auto", False), (400, "pull", True)])
def test_a_call_without_counts_leaves_its_stream_idle(Q, direction, walk, shards):
    """... and its levels to whoever reads them on another stream."""
    import torch
    import paper_2604_18913_amd as lkg
    rng = np.random.default_rng(Q)
    E, T, R, k = 1_000_003, 3_000_000, 4, 3
    s, r, o = (rng.integers(0, n, T).astype(np.int32) for n in (E, R, E))
    s[:T // 2] = rng.integers(0, 5, T // 2)  # (some hubs: the first hops pull)
    off, seeds = np.arange(Q + 1, dtype=np.int64), rng.integers(0, E, Q).astype(np.int32)
    seeds[0] = 3
    if walk:
        w_off, w_ent = oracle.walk_levels(E, s, r, o, off, seeds, k)
    else:
        want = oracle.khop(E, s, r, o, off, seeds, k)
    g = lkg.Graph(s, r, o, E, R, num_shards=shards)
    inputs = [torch.from_numpy(x).cuda() for x in (off, seeds)]
    one, other = torch.cuda.Stream(), torch.cuda.Stream()
    torch.cuda.synchronize()
    for h in range(k, -1, -1):
        res = g.khop(*inputs, k, direction=direction, counts=False, walk_exact=walk, stream=one)
        assert one.query()
        at, ent = res.level(h, stream=other)
        other.synchronize()
        if walk:
            a = w_off[h * Q:(h + 1) * Q + 1]
            assert np.array_equal(at, a - a[0]) and np.array_equal(ent.cpu().numpy(), w_ent[a[0]:a[-1]])
        else:
            on = want[2] == h
            assert np.array_equal(at, np.concatenate([[0], np.cumsum(on)])[want[0]])
            assert np.array_equal(ent.cpu().numpy(), want[1][on])
        res.close()
    g.close()
