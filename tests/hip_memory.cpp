// hipMalloc / hipFree / hipHostMalloc in front of the runtime's own (loaded with RTLD_GLOBAL ahead of the library
// under test): counts device bytes and calls, and can turn down device allocations of one size, which the runtime is
// then asked for in a size that it refuses itself, so that its error state is the real one.
#include <dlfcn.h>

#include <cstddef>
#include <mutex>
#include <unordered_map>

namespace {
std::mutex lock;
std::unordered_map<void *, size_t> sizes;
size_t live, peak, refused_size;
int device_calls, host_calls, refusals;

template <typename F>
F real(const char *name) {
    static void *lib = dlopen("libamdhip64.so.7", RTLD_LAZY | RTLD_NOLOAD);
    return lib ? reinterpret_cast<F>(dlsym(lib, name)) : nullptr;
}
}  // namespace

extern "C" {

int hipMalloc(void **p, size_t n) {
    static auto fn = real<int (*)(void **, size_t)>("hipMalloc");
    bool refuse;
    {
        std::lock_guard<std::mutex> g(lock);
        refuse = refused_size && n == refused_size;
        refusals += refuse;
        ++device_calls;
    }
    const int e = fn(p, refuse ? (size_t)1 << 50 : n);
    if (e == 0) {
        std::lock_guard<std::mutex> g(lock);
        sizes[*p] = n;
        live += n;
        if (live > peak) peak = live;
    }
    return e;
}

int hipFree(void *p) {
    static auto fn = real<int (*)(void *)>("hipFree");
    {
        std::lock_guard<std::mutex> g(lock);
        auto it = sizes.find(p);
        if (it != sizes.end()) {
            live -= it->second;
            sizes.erase(it);
        }
    }
    return fn(p);
}

int hipHostMalloc(void **p, size_t n, unsigned flags) {
    static auto fn = real<int (*)(void **, size_t, unsigned)>("hipHostMalloc");
    {
        std::lock_guard<std::mutex> g(lock);
        ++host_calls;
    }
    return fn(p, n, flags);
}

void memory_watch(size_t refuse) {  // counters from zero; device allocations of exactly `refuse` bytes fail (0: none)
    std::lock_guard<std::mutex> g(lock);
    peak = live;
    refused_size = refuse;
    device_calls = host_calls = refusals = 0;
}

size_t memory_peak() { return peak; }
size_t memory_live() { return live; }
int memory_device_calls() { return device_calls; }
int memory_host_calls() { return host_calls; }
int memory_refusals() { return refusals; }
}
