"""The visited plane of 16-word batches: what get_info hands out, lists that ask for it, and that a block given back cleared is
clear.  (Hops keep it on graphs of this size; where they do not, on larger ones, it is made where it is asked
for: test_gpu_visited_kept.py.)"""
import ctypes

import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


def problem(seed, E=4_000, T=30_000, Q=400):
    rng = np.random.default_rng(seed)
    s, r = rng.integers(0, E, T).astype(np.int32), rng.integers(0, 8, T).astype(np.int32)
    o = np.where(rng.random(T) < 0.5, rng.integers(0, 40, T), rng.integers(0, E // 2, T)).astype(np.int32)
    off = np.concatenate([[0], np.cumsum(rng.integers(1, 3, Q))]).astype(np.int64)
    return E, s, r, o, off, rng.integers(0, E, off[-1]).astype(np.int32)


def plane(ptr, words):
    import torch
    torch.cuda.synchronize()
    out = np.zeros(words, np.uint64)
    hip = ctypes.CDLL("libamdhip64.so.7")
    assert hip.hipMemcpy(out.ctypes.data_as(ctypes.c_void_p), ctypes.c_void_p(ptr), ctypes.c_size_t(8 * words), 2) == 0
    return out


@pytest.mark.parametrize("walk_exact", [False, True])
@pytest.mark.parametrize("direction", ["auto", "push", "pull"])
@pytest.mark.parametrize("k", [0, 1, 3, 9])
def test_the_plane_of_get_info_is_the_union_of_the_levels(k, direction, walk_exact):
    import paper_2604_18913_amd as lkg
    E, s, r, o, off, seeds = problem(k)
    for opts in ({}, {"num_shards": 3}):
        g = lkg.Graph(s, r, o, E, 8, **opts)
        for counts in (True, False):
            res = g.khop(off, seeds, k, direction=direction, walk_exact=walk_exact, counts=counts)
            info = res._info()
            n = info.padded_entities * 16
            levels = plane(info.levels, n * (k + 1)).reshape(k + 1, n)
            assert np.array_equal(plane(info.visited, n), np.bitwise_or.reduce(levels, 0))
            assert info.total_reached == res.total_reached
            res.close()
        g.close()


@pytest.mark.parametrize("opts", [{}, {"num_shards": 3, "max_resident_shards": 2}])
def test_lists_that_ask_for_it_and_blocks_given_back(opts):
    import paper_2604_18913_amd as lkg
    E, s, r, o, off, seeds = problem(77)
    g = lkg.Graph(s, r, o, E, 8, **opts)
    for turn, k in enumerate((3, 3, 2, 8, 3)):
        want = oracle.khop(E, s, r, o, off, seeds, k)
        res = g.khop(off, seeds, k, direction=("auto", "pull", "push", "pull", "auto")[turn])
        assert np.array_equal(res.offsets(), want[0])
        ent, hop, _ = res.fetch(want_pred=False)
        assert np.array_equal(ent.cpu().numpy(), want[1]) and np.array_equal(hop.cpu().numpy(), want[2])
        for x, y in zip(res.fetch(), want[1:4]):
            assert np.array_equal(x.cpu().numpy(), y)
        if turn % 2:
            res._info()
        res.close()
    g.close()


def test_a_recorded_fetch_makes_it_at_every_replay():
    import torch
    import paper_2604_18913_amd as lkg
    E, s, r, o, off, seeds = problem(5)
    g = lkg.Graph(s, r, o, E, 8)
    want = oracle.khop(E, s, r, o, off, seeds, 3)
    res = g.khop(off, seeds, 3, direction="pull")
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
    res.close()
    res = g.khop(off[:301], seeds[:off[300]], 3, direction="push")  # a block that the replays have written
    for x, y in zip(res.fetch(), oracle.khop(E, s, r, o, off[:301], seeds[:off[300]], 3)[1:4]):
        assert np.array_equal(x.cpu().numpy(), y)
    res.close()
    g.close()


def test_calls_on_other_streams_wait_for_the_plane():
    """Lists without predecessors make the plane on their stream, held back here; the next ones, on other streams, read it."""
    import torch
    import paper_2604_18913_amd as lkg
    E, s, r, o, off, seeds = problem(6)
    g = lkg.Graph(s, r, o, E, 8)
    want = oracle.khop(E, s, r, o, off, seeds, 3)
    outs = [[torch.zeros(want[0][-1], dtype=t, device="cuda") for t in (torch.int32, torch.uint8)] + [None] for _ in range(3)]
    res = g.khop(off, seeds, 3, direction="pull")
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream() for _ in outs]
    with torch.cuda.stream(streams[0]):
        torch.cuda._sleep(20_000_000)
    for out, stream in zip(outs, streams):
        res.fetch(out=out, stream=stream, want_pred=False)
    info = res._info()  # (synchronises by itself)
    levels = plane(info.levels, info.padded_entities * 64).reshape(4, -1)
    assert np.array_equal(plane(info.visited, levels.shape[1]), np.bitwise_or.reduce(levels, 0))
    for out in outs:
        assert np.array_equal(out[0].cpu().numpy(), want[1]) and np.array_equal(out[1].cpu().numpy(), want[2])
    res.close()
    res = g.khop(off, seeds, 3, direction="pull")  # the block, given back cleared
    for x, y in zip(res.fetch(), want[1:4]):
        assert np.array_equal(x.cpu().numpy(), y)
    res.close()
    g.close()
