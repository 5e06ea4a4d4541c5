"""What the library takes from the runtime: peaks and calls, and what a call does when a block that it can do
without is turned down.  Each test is a process of its own, with hip_memory.cpp in front of the runtime."""
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
mem.memory_watch.argtypes = [ctypes.c_size_t]
mem.memory_peak.restype = mem.memory_live.restype = ctypes.c_size_t
import oracle
import paper_2604_18913_amd as lkg

def graph(E, T, R, seed):
    rng = np.random.default_rng(seed)
    return rng, *(rng.integers(0, n, T).astype(np.int32) for n in (E, R, E))
"""


def run(tmp_path, code):
    shim = tmp_path / "hip_memory.so"
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-o", str(shim), os.path.join(HERE, "hip_memory.cpp"),
                    "-ldl"], check=True, timeout=120)
    p = subprocess.run([sys.executable, "-c", HEAD + code, str(shim), os.path.dirname(HERE), HERE], capture_output=True,
                       text=True, timeout=110)
    assert p.returncode == 0, p.stdout[-2000:] + p.stderr[-4000:]


def test_build_needs_no_more_than_its_arrays_and_five_columns_of_scratch(tmp_path):
    run(tmp_path, """
E, T, R = 100_000, 4_000_000, 20
_, s, r, o = graph(E, T, R, 1)
mem.memory_watch(0)
before = mem.memory_live()
g = lkg.Graph(s, r, o, E, R)
peak, kept = mem.memory_peak() - before, mem.memory_live() - before
print(peak / T, kept / T, mem.memory_device_calls())
# kept: objects, relation ids and triple indices of SUB's rows, subjects, relation ids and triple indices of OBJ's;
# beside them during the sorts: the triples, the keys and the indices that are sorted, and the sort's own buffers
assert kept < (20 + 2) * T, kept
assert peak < (20 + 20 + 10) * T, peak
res = g.khop(np.array([0, 2], np.int64), np.array([5, 7], np.int32), 2)
want = oracle.khop(E, s, r, o, np.array([0, 2], np.int64), np.array([5, 7], np.int32), 2)
assert all(np.array_equal(x.cpu().numpy(), y) for x, y in zip(res.fetch(), want[1:4]))
""")


def test_a_resident_graph_takes_one_block_of_pinned_memory(tmp_path):
    run(tmp_path, """
E, T, R = 10_000, 50_000, 20
_, s, r, o = graph(E, T, R, 2)
lkg.Graph(s, r, o, E, R).close()
mem.memory_watch(0)
g = lkg.Graph(s, r, o, E, R)
print(mem.memory_host_calls(), mem.memory_device_calls())
assert mem.memory_host_calls() == 1
""")


def test_no_room_for_the_triple_indices_of_a_host_built_graph(tmp_path):
    run(tmp_path, """
E, T, R = 9_000, 60_011, 7
rng, s, r, o = graph(E, T, R, 3)
o[:20_000] = rng.integers(0, 300, 20_000)      # object rows of more than 32 entries
for Q in (20, 300):                            # one- and sixteen-word planes
    off = np.arange(Q + 1, dtype=np.int64)
    seeds = rng.integers(0, E, Q).astype(np.int32)
    want = oracle.khop(E, s, r, o, off, seeds, 2)
    g = lkg.Graph(s, r, o, E, R, host_build=True)
    mem.memory_watch(4 * T)
    res = g.khop(off, seeds, 2)
    assert all(np.array_equal(x.cpu().numpy(), y) for x, y in zip(res.fetch(), want[1:4]))
    q, t = np.zeros(1, np.int32), want[1][want[0][1] - 1:want[0][1]]
    count, edges = g.paths(res, q, t)
    assert mem.memory_refusals() > 0
    mem.memory_watch(0)
    assert all(np.array_equal(x.cpu().numpy(), y) for x, y in zip(res.fetch(), want[1:4]))
    count2, edges2 = g.paths(res, q, t)
    assert int(count[0]) > 0 and torch.equal(count, count2) and torch.equal(edges, edges2)
    res.close()
    g.close()
""")
