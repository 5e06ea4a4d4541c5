// Runs the text of a device kernel on the CPU: one fiber per lane, 64 lanes per wavefront.  A wavefront
// runs until all of its lanes wait at the block's barrier (or have ended) before the next one starts, in the
// order of `waves`, so that whatever a kernel leaves unordered between two barriers is met in the order that
// the caller picks.  Cross-lane operations work on the lanes of a wavefront that wait at one together.
#pragma once

#include <ucontext.h>

#include <algorithm>
#include <climits>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <functional>
#include <memory>
#include <numeric>
#include <vector>

#define __device__
#define __global__
#define __forceinline__ inline
#define __restrict__
#define __shared__ static
#define __launch_bounds__(...)
using std::max;
using std::min;

namespace fibers {

enum State { kRuns, kAtLanes, kAtBarrier, kEnded };
struct Lane {
    ucontext_t ctx;
    State state;
    unsigned long long value, seen[64], present;
    std::vector<char> stack = std::vector<char>(128 << 10);
};
static std::vector<std::unique_ptr<Lane>> lanes;
static ucontext_t scheduler;
static int current;
static std::function<void()> body;

static void pause_in(State s) {
    Lane &l = *lanes[current];
    l.state = s;
    swapcontext(&l.ctx, &scheduler);
}

static void lane_main() {
    body();
    pause_in(kEnded);
}

// every waiting lane of the wavefront sees the values of all of them
static const Lane &exchange(unsigned long long value) {
    lanes[current]->value = value;
    pause_in(kAtLanes);
    return *lanes[current];
}

}  // namespace fibers

struct Index { unsigned x, y, z; };
static Index threadIdx, blockIdx, blockDim, gridDim;

// one block: wavefronts in the order of `waves`
static void run_block(int n, const std::vector<int> &waves, const std::function<void()> &kernel) {
    using namespace fibers;
    body = kernel;
    while ((int)lanes.size() < n) lanes.emplace_back(new Lane);
    for (int i = 0; i < n; ++i) {
        Lane &l = *lanes[i];
        l.state = kRuns;
        getcontext(&l.ctx);
        l.ctx.uc_stack.ss_sp = l.stack.data();
        l.ctx.uc_stack.ss_size = l.stack.size();
        l.ctx.uc_link = nullptr;
        makecontext(&l.ctx, lane_main, 0);
    }
    for (;;) {
        for (int w : waves)
            for (;;) {
                for (int i = w * 64; i < w * 64 + 64; ++i)
                    if (lanes[i]->state == kRuns) {
                        current = i;
                        threadIdx = {(unsigned)i, 0, 0};
                        swapcontext(&scheduler, &lanes[i]->ctx);
                    }
                unsigned long long present = 0, values[64];
                for (int i = 0; i < 64; ++i) {
                    values[i] = lanes[w * 64 + i]->value;
                    if (lanes[w * 64 + i]->state == kAtLanes) present |= 1ull << i;
                }
                if (!present) break;
                for (int i = 0; i < 64; ++i)
                    if ((present >> i) & 1) {
                        Lane &l = *lanes[w * 64 + i];
                        memcpy(l.seen, values, sizeof(values));
                        l.present = present;
                        l.state = kRuns;
                    }
            }
        bool any = false;
        for (int i = 0; i < n; ++i)
            if (lanes[i]->state == kAtBarrier) {
                lanes[i]->state = kRuns;
                any = true;
            }
        if (!any) return;  // all have ended
    }
}

static void run_grid(unsigned blocks, int threads, const std::vector<int> &waves, const std::function<void()> &kernel) {
    gridDim = {blocks, 1, 1};
    blockDim = {(unsigned)threads, 1, 1};
    for (unsigned b = 0; b < blocks; ++b) {
        blockIdx = {b, 0, 0};
        run_block(threads, waves, kernel);
    }
}

// ---- what the kernels call
static inline void __syncthreads() { fibers::pause_in(fibers::kAtBarrier); }
static inline unsigned __lane_id() { return fibers::current & 63; }
static inline unsigned long long __ballot(bool p) {
    const fibers::Lane &l = fibers::exchange(p);
    unsigned long long m = 0;
    for (int i = 0; i < 64; ++i)
        if (((l.present >> i) & 1) && l.seen[i]) m |= 1ull << i;
    return m;
}
static inline int __shfl(int v, int from) { return (int)fibers::exchange((unsigned)v).seen[from & 63]; }
static inline int __shfl_xor(int v, int m) { const int at = (int)__lane_id() ^ m; return __shfl(v, at); }
static inline int __shfl_up(int v, int d) { const int at = (int)__lane_id() - d; return __shfl(v, at < 0 ? at + d : at); }
static inline void wave_fence() { fibers::exchange(0); }
#define __builtin_amdgcn_wave_barrier wave_fence
#define __hip_atomic_load(p, order, scope) (*(p))
static inline int __popcll(unsigned long long x) { return __builtin_popcountll(x); }
static inline int __ffsll(long long x) { return __builtin_ffsll(x); }
template <class T, class U> static inline T atomicAdd(T *p, U v) { const T old = *p; *p = (T)(old + (T)v); return old; }
template <class T, class U> static inline T atomicOr(T *p, U v) { const T old = *p; *p = (T)(old | (T)v); return old; }
template <class T, class U> static inline T atomicMin(T *p, U v) { const T old = *p; *p = min(old, (T)v); return old; }
