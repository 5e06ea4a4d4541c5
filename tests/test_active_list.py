"""The list of active entities: which graphs and searches make it in one launch, whose blocks read all bitmaps in front of them,
and lists of deep searches on both sides of that rule."""
import numpy as np
import pytest

import oracle
from test_wavefront_order import between, run, text


def test_what_the_blocks_of_one_launch_read(tmp_path):
    run(tmp_path, between(text("result.hip"), "constexpr long long kActiveOneLaunch", "constexpr int kActiveListThreads") + """
int main() {
    int bad = 0, taken = 0;
    for (long long E = 64; E <= (1 << 21); E += 64 + E / 16 / 64 * 64)
        for (int levels = 1; levels <= 255; ++levels) {
            if (!active_in_one_launch(E, levels)) continue;
            ++taken;
            const long long words = E / 32, blocks = (words + 255) / 256, together = levels * words * blocks / 2;
            bad += together * 4 > 8 << 20;  // bytes: a few microseconds of a cache's rate, however the search is shaped
        }
    printf("%d shapes, %d too large\\n", taken, bad);
    return bad != 0 || taken < 1000;
}
""")


@pytest.mark.gpu
@pytest.mark.parametrize("E, k", [(64, 254), (2_000, 254), (2_048, 254), (2_112, 248), (8_190, 63), (8_192, 64), (65_536, 7),
                                  (65_537, 7), (262_144, 1), (262_145, 1), (300_000, 30), (1 << 20, 12)])
@pytest.mark.parametrize("Q", [2, 200, 300])
def test_deep_searches(E, k, Q):
    """A chain through the graph and a few triples across it: every level holds something."""
    import paper_2604_18913_amd as lkg
    rng = np.random.default_rng(E + k)
    step = max(1, E // 300)
    at = np.arange(0, E - step, step)
    s = np.concatenate([at, rng.integers(0, E, 200)]).astype(np.int32)
    o = np.concatenate([at + step, rng.integers(0, E, 200)]).astype(np.int32)
    r = np.zeros(s.size, np.int32)
    off = np.arange(Q + 1, dtype=np.int64)
    seeds = rng.choice(s, Q).astype(np.int32)
    seeds[0] = 0
    want = oracle.khop(E, s, r, o, off, seeds, k)
    g = lkg.Graph(s, r, o, E, 1)
    res = g.khop(off, seeds, k, direction="pull")
    assert np.array_equal(res.offsets(), want[0])
    for got, w in zip(res.fetch(), want[1:]):
        assert np.array_equal(got.cpu().numpy(), w)
    res.close()
    g.close()


@pytest.mark.gpu
@pytest.mark.parametrize("E", [300_000, 1 << 20, (1 << 20) + 2_049])
@pytest.mark.parametrize("Q", [2, 200, 300])
@pytest.mark.parametrize("sum_chunks", [0, 512, 1 << 20])
def test_prefixes_by_a_scan_or_by_the_blocks(monkeypatch, E, Q, sum_chunks):
    """512 chunks hold 1,048,576 entities: both sides of the rule, and either form for all."""
    import paper_2604_18913_amd as lkg
    monkeypatch.setenv("LOGOSKG_ACTIVE_SUM_CHUNKS", str(sum_chunks))
    rng = np.random.default_rng(E + Q)
    s, o = rng.integers(0, E, (2, 60_000)).astype(np.int32)
    o[:40_000] = np.sort(rng.choice(E, 40_000, replace=False))
    s[:40_000] = rng.integers(0, 40, 40_000)
    r = np.zeros(s.size, np.int32)
    off = np.arange(Q + 1, dtype=np.int64)
    seeds = rng.integers(0, 40, Q).astype(np.int32)
    want = oracle.khop(E, s, r, o, off, seeds, 2)
    g = lkg.Graph(s, r, o, E, 1)
    res = g.khop(off, seeds, 2)
    assert np.array_equal(res.offsets(), want[0])
    for got, w in zip(res.fetch(), want[1:]):
        assert np.array_equal(got.cpu().numpy(), w)
    res.close()
    g.close()
