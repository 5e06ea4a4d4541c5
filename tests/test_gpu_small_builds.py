"""Builds about the sizes where the rows are classified on the host or on the device, the arrays are one allocation or eight and
the distinct pairs go by id or by in-degree: searches in both directions, and builds on the host, which hold no pairs."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


def graph(rng, E, T):  # rows of all lengths, half of the triples repeat others' subject and object
    n = T - T // 2
    s, o = rng.integers(0, E, n), (E * rng.random(n) ** 4).astype(np.int64)
    again = rng.integers(0, n, T // 2)
    p = rng.permutation(T)
    return np.concatenate([s, s[again]])[p].astype(np.int32), rng.integers(0, 9, T).astype(np.int32), np.concatenate([o, o[again]])[p].astype(np.int32)


@pytest.mark.parametrize("E, T", [(1, 3), (63, 900), (1 << 14, 100_000), ((1 << 14) + 1, 100_000), (30_000, 830_000), (30_000, 850_000),
                                  (50_000, 1 << 21), (50_000, (1 << 21) + 1)])
def test_build(E, T):
    import paper_2604_18913_amd as lkg
    rng = np.random.default_rng(E + T)
    s, r, o = graph(rng, E, T)
    pairs = len(np.unique(s.astype(np.int64) * E + o))
    degree = np.bincount(o, minlength=E)
    for opts in ({}, {"hub_min_degree": 50}, {"host_build": True}):
        g = lkg.Graph(s, r, o, E, 9, **opts)
        info = g.info()
        hub = opts.get("hub_min_degree", 1024)
        assert info["num_in_rows"] == np.count_nonzero(degree) and info["num_in_hubs"] == np.count_nonzero(degree >= hub)
        assert info["num_out_rows"] == len(np.unique(s)) and info["num_out_hubs"] == np.count_nonzero(np.bincount(s) >= hub)
        if T > 1000:
            kept = info["device_bytes"] > 20 * T + 6 * T + 12 * pairs
            assert kept == ("host_build" not in opts), info["device_bytes"] / T
        for Q, k in ((3, 3), (100, 2), (300, 2)):
            off, seeds = np.arange(Q + 1, dtype=np.int64), rng.integers(0, E, Q).astype(np.int32)
            want = oracle.khop(E, s, r, o, off, seeds, k)
            for direction in ("auto", "pull"):
                res = g.khop(off, seeds, k, direction=direction)
                assert np.array_equal(res.offsets(), want[0])
                for x, y in zip(res.fetch(), want[1:4]):
                    assert np.array_equal(x.cpu().numpy(), y)
                res.close()
        g.close()
