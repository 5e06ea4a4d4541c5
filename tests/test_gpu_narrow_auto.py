"""Searches of narrow batches that choose their own directions: a hop behind a pulled one is launched before the host has read its
frontier, and kernels of a hop that is not pulled after all return at once.  Layered graphs make the order of the
directions; lists or levels, directions and counters against the oracle."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

SHARE = {"push": 0.02, "pull": 0.12, "dense": 0.62, "end": 0.0}  # of the triples that leave a layer
PLANS = [["push", "pull", "push", "pull"], ["pull", "push", "push", "pull"], ["pull", "pull", "push", "push", "pull"],
         ["dense", "pull", "push", "pull", "end"], ["pull", "dense", "push", "end", "end"], ["push", "push", "dense", "end", "end", "end"],
         ["pull", "end", "end"], ["dense", "end"], ["pull", "pull", "pull"], ["push", "dense", "push", "pull"]]


def layered(plan, rng, back, T=60_000, R=6):
    """Layer 0: three subjects; every layer's triples go to the next one, its first objects having long rows, and some back
    (one question reaches a whole layer at once; of several, some would come to the rest of it a hop later)."""
    sizes = [3] + [int(rng.integers(200, 600)) for _ in plan]
    first = np.concatenate([[0], np.cumsum(sizes)])
    s, o = [], []
    for i, kind in enumerate(plan):
        m = int(SHARE[kind] * T)
        if m == 0:
            break
        src, dst = first[i] + np.arange(sizes[i]), first[i + 1] + np.arange(sizes[i + 1])
        to = np.where(rng.random(m) < 0.4, dst[rng.integers(0, 3, m)], dst[rng.integers(0, sizes[i + 1], m)])
        if i > 0 and back:
            to = np.where(rng.random(m) < 0.05, first[i - 1] + rng.integers(0, sizes[i - 1], m), to)
        to[:dst.size] = dst  # (the whole layer is reached)
        s.append(np.concatenate([src, src[rng.integers(0, sizes[i], m)]])[:m])
        o.append(to)
    rest = T - sum(x.size for x in s)  # triples that no search follows
    E = int(first[-1]) + 1000
    s.append(rng.integers(first[-1], E, rest))
    o.append(rng.integers(0, E, rest))
    p = rng.permutation(T)
    return (E, R, np.concatenate(s)[p].astype(np.int32), rng.integers(0, R, T).astype(np.int32),
            np.concatenate(o)[p].astype(np.int32))


@pytest.mark.parametrize("walk", [False, True])
@pytest.mark.parametrize("Q, masked", [(1, False), (3, True), (64, False), (65, True), (256, False)])
@pytest.mark.parametrize("plan", PLANS, ids="-".join)
def test_directions(plan, Q, masked, walk):
    import paper_2604_18913_amd as lkg
    rng = np.random.default_rng(len(plan) * 1000 + Q)
    E, R, s, r, o = layered(plan, rng, Q == 1)
    T, k = s.size, len(plan)
    counts = np.concatenate([[3], rng.integers(1, 4, Q - 1)])
    off = np.concatenate([[0], np.cumsum(counts)]).astype(np.int64)
    seeds = np.concatenate([rng.permutation(3)[:n] for n in counts]).astype(np.int32)
    mask = rng.integers(1, 2**R, (Q, 1)).astype(np.uint64) if masked else None
    if masked:
        mask[0] = 2**R - 1
    want = oracle.khop(E, s, r, o, off, seeds, k, mask)
    if walk:
        w_off, w_ent = oracle.walk_levels(E, s, r, o, off, seeds, k, mask)
        frontier = [np.unique(w_ent[w_off[h * Q]:w_off[(h + 1) * Q]]) for h in range(k + 1)]
    else:
        frontier = [np.unique(want[1][want[2] == h]) for h in range(k + 1)]
    degree = np.bincount(s, minlength=E)
    g = lkg.Graph(s, r, o, E, R)
    for _ in range(2):
        res = g.khop(off, seeds, k, mask, walk_exact=walk)
        assert np.array_equal(res.offsets(), want[0])
        stats = res.hop_stats()
        for h, (kind, st) in enumerate(zip(plan, stats)):
            edges = int(degree[frontier[h]].sum())
            direction = 0 if edges == 0 else lkg.binding.DIRECTIONS["pull" if edges * 12 > T else "push"]
            assert (st["direction"], st["frontier_edges"]) == (direction, edges), h
            assert st["active_rows"] == np.count_nonzero(degree[frontier[h]]) and st["entities_reached"] == frontier[h + 1].size, h
            if not walk and not masked:
                assert direction == {"push": 1, "pull": 2, "dense": 2, "end": 0}[kind], h
        if walk:
            for h in range(k + 1):
                at, ent = res.level(h)
                a = w_off[h * Q:(h + 1) * Q + 1]
                assert np.array_equal(at, a - a[0]) and np.array_equal(ent.cpu().numpy(), w_ent[a[0]:a[-1]]), h
        else:
            for got, w in zip(res.fetch(), want[1:]):
                assert np.array_equal(got.cpu().numpy(), w)
        res.close()
    g.close()
