"""How a k-hop call ends: what a call that fails behind its hops leaves to the next one."""
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
