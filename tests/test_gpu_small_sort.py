"""Order of the entities of a small search: ids spread evenly, ids that crowd (more than a bucket of the sort takes), runs
of neighbours, the ends of the id range, and numbers of entities around the block's threads."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 2, 63, 64, 65, 1023, 1024, 1025, 2047])
@pytest.mark.parametrize("how", ["even", "run", "crowd", "ends", "two runs"])
def test_order(n, how):
    import paper_2604_18913_amd as lkg
    rng = np.random.default_rng(n)
    E = 300_000
    if how == "even":
        objects = rng.choice(np.arange(1, E), n, replace=False)
    elif how == "run":
        objects = 77_000 + np.arange(n)
    elif how == "crowd":  # half of the ids next to each other, half far apart
        objects = np.unique(np.concatenate([5_000 + np.arange(n // 2 + 1), rng.choice(np.arange(10_000, E), n // 2 + 1)]))[:n]
    elif how == "ends":
        objects = np.unique(np.concatenate([np.arange(1, n // 2 + 1), E - 1 - np.arange(n - n // 2)]))
    else:
        objects = np.concatenate([np.arange(1_000, 1_000 + n // 2), 200_000 + 3 * np.arange(n - n // 2)])
    objects = rng.permutation(objects).astype(np.int32)
    s = np.full(objects.size, 500, dtype=np.int32)
    objects[objects == 500] = 501
    r = np.zeros(objects.size, dtype=np.int32)
    off, seeds = np.array([0, 1, 2], dtype=np.int64), np.array([500, 299_000], dtype=np.int32)
    g = lkg.Graph(s, r, objects, E, 1)
    res = g.khop(off, seeds, 1, direction="push")
    want = oracle.khop(E, s, r, objects, off, seeds, 1)
    assert np.array_equal(res.offsets(), want[0])
    for got, w in zip(res.fetch(), want[1:]):
        assert np.array_equal(got.cpu().numpy(), w)
    res.close()
    g.close()
