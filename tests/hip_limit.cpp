// hipMalloc / hipFree / hipMemGetInfo in front of the runtime's own (loaded with RTLD_GLOBAL ahead of the library under test): a
// device of few bytes.  An allocation that would pass them is asked of the runtime in a size that it refuses itself, so
// that its error state is the real one.
#include <dlfcn.h>

#include <cstddef>
#include <mutex>
#include <unordered_map>

namespace {
std::mutex lock;
std::unordered_map<void *, size_t> sizes;
size_t live, peak, most;  // most: 0 is no limit

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
        refuse = most && live + n > most;
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

int hipMemGetInfo(size_t *free_bytes, size_t *all_bytes) {
    static auto fn = real<int (*)(size_t *, size_t *)>("hipMemGetInfo");
    const int e = fn(free_bytes, all_bytes);
    std::lock_guard<std::mutex> g(lock);
    if (e == 0 && most) {
        *all_bytes = most;
        *free_bytes = live < most ? most - live : 0;
    }
    return e;
}

void memory_limit(size_t bytes) {  // (the peak starts again)
    std::lock_guard<std::mutex> g(lock);
    most = bytes;
    peak = live;
}

size_t memory_peak() { return peak; }
size_t memory_live() { return live; }
}
