"""Blocks that come back from the device pool as cleared: only a request that the zeros cover may go without a fill.  The pool's
own text runs on the CPU with host memory behind it; on the GPU searches of many shapes take turns on one graph, on
memory that holds anything but zeros."""
import numpy as np
import pytest

import oracle
from test_wavefront_order import between, definition, run, text

RUNTIME = """
#include <map>
#include <memory>
#include <unordered_map>
typedef void *hipStream_t; typedef int *hipEvent_t; enum hipError_t { hipSuccess, hipFailed };
enum logoskg_status { LOGOSKG_OK, LOGOSKG_EDEVICE, LOGOSKG_ENOMEM };
enum { hipEventDisableTiming };
hipError_t hipMalloc(void **p, size_t n) { *p = memset(malloc(n), 0xAA, n); return hipSuccess; }
hipError_t hipFree(void *p) { free(p); return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
const char *hipGetErrorString(hipError_t) { return ""; }
hipError_t hipEventCreateWithFlags(hipEvent_t *e, int) { *e = new int; return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, int) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
void set_error(const char *, ...) {}
"""

MAIN = """
int main() {
    unsigned long long rng = 1;
    auto next = [&](unsigned n) { rng = rng * 6364136223846793005ull + 1442695040888963407ull; return (unsigned)(rng >> 33) % n; };
    DevPool pool;
    struct Held { char *p; size_t n; bool clear; };
    std::vector<Held> held;
    int skipped = 0;
    for (int turn = 0; turn < 20000; ++turn) {
        if (held.size() < 6 && next(2)) {
            Held h = {nullptr, 1 + next(3) * 100 + next(900), next(2) != 0};
            bool zeroed = false;
            if (pool.alloc((void **)&h.p, h.n, (hipStream_t)(size_t)next(2), &zeroed) != LOGOSKG_OK) return 2;
            for (size_t i = 0; zeroed && i < h.n; ++i)
                if (h.p[i]) { printf("turn %d: byte %zu of %zu is not zero\\n", turn, i, h.n); return 1; }
            skipped += zeroed;
            memset(h.p, h.clear ? 0 : 0x55, h.n);
            held.push_back(h);
        } else if (!held.empty()) {
            const size_t i = next((unsigned)held.size());
            void *p = held[i].p;
            const bool clear = held[i].clear;
            if (!clear && next(2)) pool.release(p);
            else pool.release_after(&p, &clear, 1, (hipStream_t)(size_t)next(2));
            held.erase(held.begin() + i);
        }
    }
    printf("%d requests of cleared blocks\\n", skipped);
    return skipped < 100;
}
"""


def test_cleared_blocks_cover_the_request(tmp_path):
    build = text("build.hip")
    run(tmp_path, RUNTIME + definition(text("common.h"), "class DevPool {")
        + between(build, "logoskg_status DevPool::alloc(", "const char *const kKernelNames") + MAIN)


@pytest.mark.gpu
def test_searches_of_many_shapes_on_one_graph():
    import torch
    import paper_2604_18913_amd as lkg
    rng = np.random.default_rng(5)
    E, T, R = 6_001, 20_000, 3
    s, r, o = (rng.integers(0, n, T).astype(np.int32) for n in (E, R, E))
    held = {}

    def dev_alloc(nbytes):
        t = torch.full((nbytes,), 0xA5, dtype=torch.uint8, device="cuda")
        torch.cuda.synchronize()
        held[t.data_ptr()] = t
        return t.data_ptr()

    g = lkg.Graph(s, r, o, E, R, dev_alloc=dev_alloc, dev_free=held.__delitem__)
    for turn in range(60):
        Q, k = int(rng.choice([1, 60, 65, 200, 300, 1000])), int(rng.choice([0, 1, 2, 3, 7, 15, 23, 40]))
        off, seeds = np.arange(Q + 1, dtype=np.int64), rng.integers(0, E, Q).astype(np.int32)
        want = oracle.khop(E, s, r, o, off, seeds, k)
        res = g.khop(off, seeds, k, direction=str(rng.choice(["auto", "push", "pull"])))
        assert np.array_equal(res.offsets(), want[0]), (turn, Q, k)
        for got, w in zip(res.fetch(), want[1:]):
            assert np.array_equal(got.cpu().numpy(), w), (turn, Q, k)
        res.close()
    g.close()
