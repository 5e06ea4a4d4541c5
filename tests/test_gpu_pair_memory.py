"""Memory of the rows of distinct (subject, object) pairs, which a graph can do without: what is counted for them, and calls that
find no room but theirs.  Each test is a process of its own, with hip_memory.cpp or hip_limit.cpp in front of the runtime."""
import os
import subprocess
import sys

import pytest

pytestmark = pytest.mark.gpu

HERE = os.path.dirname(os.path.abspath(__file__))

HEAD = """
import ctypes, sys
sys.path[:0] = [sys.argv[2], sys.argv[3]]
import numpy as np
import torch
torch.cuda.init()
mem = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
for f in ("memory_watch", "memory_limit"):
    if hasattr(mem, f):
        getattr(mem, f).argtypes = [ctypes.c_size_t]
for f in ("memory_peak", "memory_live"):
    if hasattr(mem, f):
        getattr(mem, f).restype = ctypes.c_size_t
import oracle
import paper_2604_18913_amd as lkg

def graph(E, T, seed, share=0.5):  # a share of the triples repeats others' subject and object
    rng = np.random.default_rng(seed)
    n = int(T * (1 - share))
    s, o = rng.integers(0, E, n), (E * rng.random(n) ** 4).astype(np.int64)  # rows of all lengths
    again = rng.integers(0, n, T - n)
    p = rng.permutation(T)
    return rng, np.concatenate([s, s[again]])[p].astype(np.int32), rng.integers(0, 9, T).astype(np.int32), np.concatenate([o, o[again]])[p].astype(np.int32)

def batch(rng, E, Q):
    return np.arange(Q + 1, dtype=np.int64), rng.integers(0, E, Q).astype(np.int32)

def same(res, want):
    assert np.array_equal(res.offsets(), want[0])
    assert all(np.array_equal(x.cpu().numpy(), y) for x, y in zip(res.fetch(), want[1:4]))
"""


def run(tmp_path, shim_source, code):
    shim = tmp_path / "shim.so"
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-o", str(shim), os.path.join(HERE, shim_source), "-ldl"],
                   check=True, timeout=120)
    p = subprocess.run([sys.executable, "-c", HEAD + code, str(shim), os.path.dirname(HERE), HERE], capture_output=True,
                       text=True, timeout=110)
    assert p.returncode == 0, p.stdout[-2000:] + p.stderr[-4000:]


def test_device_bytes_follow_them(tmp_path):
    run(tmp_path, "hip_memory.cpp", """
E, T, Q, k = 70_000, 700_000, 300, 2
rng, s, r, o = graph(E, T, 1)
off, seeds = batch(rng, E, Q)
want = oracle.khop(E, s, r, o, off, seeds, k)
lkg.Graph(s, r, o, E, 9).close()
mem.memory_watch(0)
live = mem.memory_live()
g = lkg.Graph(s, r, o, E, 9)
held, counted = mem.memory_live() - live, g.info()["device_bytes"]
assert 30 * T < counted <= held < counted + 64 * 1024, (held, counted)
pairs = len(np.unique(s.astype(np.int64) * E + o))
assert counted > 20 * T + 6 * T + 12 * pairs
before = g.info()["device_bytes"]
res = g.khop(off, seeds, k)
pool = g.info()["device_bytes"]
res.fetch()
assert g.info()["device_bytes"] == pool + 4 * E  # their index
same(res, want)
res.close()
g.close()
# their work lists turned down: none of their bytes is left in what is counted
hist = np.bincount(np.unique(s.astype(np.int64) * E + o) % E, minlength=E)
seg, long_rows, multi = int(np.ceil(hist[hist > 32] / 1024).sum()), int((hist > 32).sum()), int((hist > 1024).sum())
giant = hist[hist >= 8192]
hubs = hist[hist >= 1024]
table = 1 + len(giant) + 1 + (int(np.ceil(giant.max() / 8192)) if len(giant) else 0) + 1 + len(hubs)
up = lambda b: (max(b, 4) + 15) // 16 * 16
bytes_ = up(16 * seg) + up(4 * table) + up(4 * multi) + up(4 * long_rows) + 12 * int(((hist > 0) & (hist <= 32)).sum())
mem.memory_watch(bytes_)
live = mem.memory_live()
g = lkg.Graph(s, r, o, E, 9)
assert mem.memory_refusals() > 0, bytes_
held, counted = mem.memory_live() - live, g.info()["device_bytes"]
assert counted <= held < counted + 64 * 1024, (held, counted)
same(g.khop(off, seeds, k), want)
""")


LIMITED = """
E, T, k = 60_000, 1_200_000, 3
rng, s, r, o = graph(E, T, 2)
"""


@pytest.mark.parametrize("Q", [40, 200, 300])
def test_calls_that_find_no_room_but_theirs(tmp_path, Q):
    run(tmp_path, "hip_limit.cpp", f"Q = {Q}" + LIMITED + """
off, seeds = batch(rng, E, Q)
want = oracle.khop(E, s, r, o, off, seeds, k)
out = [torch.empty(want[0][-1], dtype=t, device="cuda") for t in (torch.int32, torch.uint8, torch.int32)]
off, seeds = torch.from_numpy(off).cuda(), torch.from_numpy(seeds).cuda()
pairs = 6 * T + 12 * len(np.unique(s.astype(np.int64) * E + o))

def search_and_fetch(g):
    res = g.khop(off, seeds, k)
    res.fetch(out=out)
    torch.cuda.synchronize()
    assert np.array_equal(res.offsets(), want[0])
    assert all(np.array_equal(x.cpu().numpy(), y) for x, y in zip(out, want[1:4]))
    res.close()

g = lkg.Graph(s, r, o, E, 9)
mem.memory_limit(0)
live = mem.memory_live()
search_and_fetch(g)
needs = mem.memory_peak() - live
g.close()
for short in (1 << 16, min(pairs, needs) * 3 // 4):
    g = lkg.Graph(s, r, o, E, 9)
    held = g.info()["device_bytes"]
    assert held > 20 * T + pairs
    mem.memory_limit(mem.memory_live() + needs - short)
    for _ in range(3):
        search_and_fetch(g)
    mem.memory_limit(0)
    g.close()
""")


def test_recorded_fetches_keep_them(tmp_path):
    run(tmp_path, "hip_limit.cpp", LIMITED + """
Q = 300
off, seeds = batch(rng, E, Q)
want = oracle.khop(E, s, r, o, off, seeds, k)
g = lkg.Graph(s, r, o, E, 9)
res = g.khop(off, seeds, k)
same(res, want)
out = [torch.zeros(want[0][-1], dtype=t, device="cuda") for t in (torch.int32, torch.uint8, torch.int32)]
torch.cuda.synchronize()
stream, recorded = torch.cuda.Stream(), torch.cuda.CUDAGraph()
with torch.cuda.graph(recorded, stream=stream):
    res.fetch(out=out, stream=stream)
held = g.info()["device_bytes"]
mem.memory_limit(mem.memory_live() + (1 << 20))
try:
    g.khop(off, seeds, k)
    raise SystemExit("a second result had no room")
except lkg.LogosKGError as e:
    assert e.status == 2, e
mem.memory_limit(0)
assert g.info()["device_bytes"] > 20 * T + 12 * T // 2
for _ in range(3):
    for x in out:
        x.zero_()
    recorded.replay()
    torch.cuda.synchronize()
    assert all(np.array_equal(x.cpu().numpy(), y) for x, y in zip(out, want[1:4]))
""")


def test_builds_on_a_small_device(tmp_path):
    run(tmp_path, "hip_limit.cpp", """
E, T, Q, k = 100_000, 6_000_000, 100, 2
rng, s, r, o = graph(E, T, 3)
off, seeds = batch(rng, E, Q)
want = oracle.khop(E, s, r, o, off, seeds, k)
for per_triple, kept in ((70, False), (400, True)):   # the sorts and the arrays need fifty bytes per triple
    mem.memory_limit(mem.memory_live() + per_triple * T)
    g = lkg.Graph(s, r, o, E, 9)
    assert (g.info()["device_bytes"] > 26 * T) == kept, g.info()["device_bytes"] / T
    same(g.khop(off, seeds, k), want)
    g.close()
    mem.memory_limit(0)
""")


@pytest.mark.parametrize("opts", [{}, {"num_shards": 2}])
def test_no_room_for_their_index(tmp_path, opts):
    """The last thing that the first fetch of a large batch takes: it then goes by all triples."""
    run(tmp_path, "hip_limit.cpp", f"opts = {opts!r}" + LIMITED + """
Q = 300
off, seeds = batch(rng, E, Q)
want = oracle.khop(E, s, r, o, off, seeds, k)
out = [torch.zeros(want[0][-1], dtype=t, device="cuda") for t in (torch.int32, torch.uint8, torch.int32)]
off, seeds = torch.from_numpy(off).cuda(), torch.from_numpy(seeds).cuda()
for limited in (False, True):
    g = lkg.Graph(s, r, o, E, 9, **opts)
    g.khop(off, seeds, k, direction="pull").close()  # (a cache holds every unit from here on)
    res = g.khop(off, seeds, k)
    live, held = mem.memory_live(), g.info()["device_bytes"]
    assert held > 26 * T
    if limited:
        mem.memory_limit(live + needs - 1024)
    res.fetch(out=out)
    torch.cuda.synchronize()
    mem.memory_limit(0)
    needs = mem.memory_live() - live
    assert g.info()["device_bytes"] == held + (0 if limited else 4 * E), (g.info()["device_bytes"] - held, E)
    assert all(np.array_equal(x.cpu().numpy(), y) for x, y in zip(out, want[1:4]))
    res.fetch(out=out)
    assert all(np.array_equal(x.cpu().numpy(), y) for x, y in zip(out, want[1:4]))
    res.close()
    g.close()
""")


def test_a_fetch_that_does_without_memory_has_them_go_with_the_next_search(tmp_path):
    run(tmp_path, "hip_limit.cpp", LIMITED + """
Q = 200
o[:90_000] = 7  # object rows that are cut into segments
o[90_000:120_000] = 8
off, seeds = batch(rng, E, Q)
want = oracle.khop(E, s, r, o, off, seeds, k)
out = [torch.zeros(want[0][-1], dtype=t, device="cuda") for t in (torch.int32, torch.uint8, torch.int32)]
off, seeds = torch.from_numpy(off).cuda(), torch.from_numpy(seeds).cuda()
pairs = 6 * T + 12 * len(np.unique(s.astype(np.int64) * E + o))
g = lkg.Graph(s, r, o, E, 9)
held = g.info()["device_bytes"]
assert held > 20 * T + pairs
res = g.khop(off, seeds, k)
pool = g.info()["device_bytes"] - held
mem.memory_limit(mem.memory_live() + 256)
for _ in range(2):
    for x in out:
        x.zero_()
    res.fetch(out=out)
    torch.cuda.synchronize()
    assert all(np.array_equal(x.cpu().numpy(), y) for x, y in zip(out, want[1:4]))
assert g.info()["device_bytes"] == held + pool
res.close()
for _ in range(2):
    res = g.khop(off, seeds, k)
    res.fetch(out=out)
    torch.cuda.synchronize()
    assert all(np.array_equal(x.cpu().numpy(), y) for x, y in zip(out, want[1:4]))
    assert g.info()["device_bytes"] < held + pool - pairs // 2
    res.close()
""")


def test_a_build_without_room_for_the_classification_on_the_device(tmp_path):
    run(tmp_path, "hip_memory.cpp", """
E, T, Q, k = 70_001, 400_000, 90, 2
rng, s, r, o = graph(E, T, 5)
off, seeds = batch(rng, E, Q)
want = oracle.khop(E, s, r, o, off, seeds, k)
degree = np.bincount(o, minlength=E)
mem.memory_watch((4 * E + 255) // 256 * 256)  # a word per row
g = lkg.Graph(s, r, o, E, 9, host_build=True)
assert mem.memory_refusals() > 0
mem.memory_watch(0)  # (a search's planes may have the size)
info = g.info()
assert info["num_in_rows"] == np.count_nonzero(degree) and info["num_in_hubs"] == np.count_nonzero(degree >= 1024)
same(g.khop(off, seeds, k), want)
""")
