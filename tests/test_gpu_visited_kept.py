"""Searches on 16-word planes that keep the visited plane in their hops (deep ones, small graphs, graphs whose last result was
asked for it) and searches that do not: lists and the plane itself, on both sides of each line."""
import numpy as np
import pytest

import oracle
from test_gpu_visited import plane

pytestmark = pytest.mark.gpu


def problem(seed, E, T, Q=300):
    rng = np.random.default_rng(seed)
    s = np.where(rng.random(T) < 0.6, rng.integers(0, 3_000, T), rng.integers(0, E, T)).astype(np.int32)
    # object rows of every class: short ones, single segments and several of them
    o = np.where(rng.random(T) < 0.5, rng.integers(0, 12, T), rng.integers(0, 3_000, T)).astype(np.int32)
    r = rng.integers(0, 8, T).astype(np.int32)
    off = np.concatenate([[0], np.cumsum(rng.integers(1, 3, Q))]).astype(np.int64)
    return s, r, o, off, rng.integers(0, 3_000, off[-1]).astype(np.int32)


@pytest.mark.parametrize("E", [4_000, (1 << 18) - 64, 1 << 18])
@pytest.mark.parametrize("direction, opts", [("auto", {}), ("pull", {}), ("push", {}), ("pull", {"num_shards": 3, "max_resident_shards": 2})])
def test_lists_and_plane(E, direction, opts):
    import paper_2604_18913_amd as lkg
    s, r, o, off, seeds = problem(E, E, 40_000)
    g = lkg.Graph(s, r, o, E, 8, **opts)
    n = (E + 63) // 64 * 64 * 16
    for k, asked in ((3, False), (3, True), (4, False), (5, False), (1, True), (2, False)):
        want = oracle.khop(E, s, r, o, off, seeds, k)
        res = g.khop(off, seeds, k, direction=direction)  # (the search before it was asked for its plane or not)
        assert np.array_equal(res.offsets(), want[0]), (k, asked)
        for x, y in zip(res.fetch(), want[1:4]):
            assert np.array_equal(x.cpu().numpy(), y), (k, asked)
        if not asked:
            info = res._info()
            levels = plane(info.levels, n * (k + 1)).reshape(k + 1, n)
            assert np.array_equal(plane(info.visited, n), np.bitwise_or.reduce(levels, 0)), k
        res.close()
    g.close()


@pytest.mark.parametrize("E", [(1 << 15) - 64, 1 << 15])
@pytest.mark.parametrize("direction", ["auto", "push", "pull"])
def test_walk_exact(E, direction):
    import paper_2604_18913_amd as lkg
    s, r, o, off, seeds = problem(E + 1, E, 30_000)
    g = lkg.Graph(s, r, o, E, 8)
    Q, k, n = len(off) - 1, 3, (E + 63) // 64 * 64 * 16
    w_off, w_ent = oracle.walk_levels(E, s, r, o, off, seeds, k)
    for asked in (False, True, False):
        res = g.khop(off, seeds, k, walk_exact=True, direction=direction)
        for h in range(k + 1):
            at, ent = res.level(h)
            a = w_off[h * Q:(h + 1) * Q + 1]
            assert np.array_equal(at, a - a[0]) and np.array_equal(ent.cpu().numpy(), w_ent[a[0]:a[-1]])
        if not asked:
            info = res._info()
            levels = plane(info.levels, n * (k + 1)).reshape(k + 1, n)
            assert np.array_equal(plane(info.visited, n), np.bitwise_or.reduce(levels, 0))
        res.close()
    g.close()


def test_lists_without_predecessors_and_a_recorded_fetch():
    """On a graph that does not keep the plane: the first such list makes it, the next search keeps it, the one behind does not."""
    import torch
    import paper_2604_18913_amd as lkg
    E, k = 1 << 18, 3
    s, r, o, off, seeds = problem(9, E, 40_000)
    g = lkg.Graph(s, r, o, E, 8)
    want = oracle.khop(E, s, r, o, off, seeds, k)
    for turn in range(4):
        res = g.khop(off, seeds, k)
        if turn != 2:
            ent, hop, _ = res.fetch(want_pred=False)
            assert np.array_equal(ent.cpu().numpy(), want[1]) and np.array_equal(hop.cpu().numpy(), want[2])
        else:
            for x, y in zip(res.fetch(), want[1:4]):
                assert np.array_equal(x.cpu().numpy(), y)
        res.close()
    for x in g.khop(off, seeds, k).fetch():  # (nothing asks)
        assert x.numel() == want[0][-1]
    res = g.khop(off, seeds, k, direction="pull")
    out = [torch.zeros(want[0][-1], dtype=t, device="cuda") for t in (torch.int32, torch.uint8)] + [None]
    torch.cuda.synchronize()
    stream, graph = torch.cuda.Stream(), torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream):
        res.fetch(out=out, stream=stream, want_pred=False)
    for _ in range(3):
        out[0].zero_()
        out[1].zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert np.array_equal(out[0].cpu().numpy(), want[1]) and np.array_equal(out[1].cpu().numpy(), want[2])
    del graph
    streams = [torch.cuda.Stream() for _ in range(3)]
    outs = [[torch.zeros(want[0][-1], dtype=t, device="cuda") for t in (torch.int32, torch.uint8)] + [None] for _ in streams]
    with torch.cuda.stream(streams[0]):
        torch.cuda._sleep(20_000_000)
    for out, stream in zip(outs, streams):  # (held back on the first stream, the others wait for the plane)
        res.fetch(out=out, stream=stream, want_pred=False)
    torch.cuda.synchronize()
    for out in outs:
        assert np.array_equal(out[0].cpu().numpy(), want[1]) and np.array_equal(out[1].cpu().numpy(), want[2])
    res.close()
    g.close()


@pytest.mark.parametrize("overlap", ["0", "1"])
def test_get_info_while_a_fetch_is_recorded(monkeypatch, overlap):
    import torch
    import paper_2604_18913_amd as lkg
    monkeypatch.setenv("LOGOSKG_OVERLAP_FETCH", overlap)
    E, k = 1 << 18, 3
    s, r, o, off, seeds = problem(13, E, 40_000)
    g = lkg.Graph(s, r, o, E, 8)
    want = oracle.khop(E, s, r, o, off, seeds, k)
    g.khop(off, seeds, k).fetch()
    res = g.khop(off, seeds, k)  # (its plane is not kept)
    out = [torch.zeros(want[0][-1], dtype=t, device="cuda") for t in (torch.int32, torch.uint8, torch.int32)]
    torch.cuda.synchronize()
    stream, graph = torch.cuda.Stream(), torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream):
        res.fetch(out=out, stream=stream)
        info = res._info()
    n = (E + 63) // 64 * 64 * 16
    levels = plane(info.levels, n * (k + 1)).reshape(k + 1, n)
    assert np.array_equal(plane(info.visited, n), np.bitwise_or.reduce(levels, 0))
    for _ in range(3):
        for x in out:
            x.zero_()
        graph.replay()
        torch.cuda.synchronize()
        for x, y in zip(out, want[1:4]):
            assert np.array_equal(x.cpu().numpy(), y)
    del graph
    res.close()
    g.close()
